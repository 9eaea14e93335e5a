// multigrid.hip -- geometric multigrid Helmholtz solver on one uniform
// cell-centred grid and the reaction-diffusion time steps built on it
// (declared in include/amrv_mg.h; the method's multigrid of Sec. 1.4 and the
// reaction-diffusion schemes of Sec. 2.5).
//
// Layout in the caller's workspace (every array 256-byte aligned):
//   phi[field][level], f[field][level]   n_l^d doubles each, n_l = n >> l,
//                                         level 0 is the grid; x fastest, or in
//                                         3D above the tail (constant
//                                         coefficient) in split order
//                                         (mg_internal.hpp)
//   tmp[4]                                n^d doubles (reaction-diffusion
//                                         temporaries; between explicit steps
//                                         tmp[2 + field] holds the coarse
//                                         matrix, k_mg_coarse_matrix)
//   par                                   lambda per field, 1/diagonal per
//                                         field and level, 1/h^2 per level
// plus pinned host memory for the per-block residual maxima, folded on the
// host after each cycle.
//
// A V-cycle: on each level above the tail, `pre` red-black sweeps and a
// launch that forms the residual on the 2^d children of every coarse cell,
// averages it into the coarse right-hand side and zeroes the coarse
// correction (in 2D both in one tiled launch, k_mg_down2d); the coarse
// levels of at most 4,096 cells are solved by one workgroup per field with
// every level resident in LDS (k_mg_tail: the whole descent and ascent in one
// launch, with the levels of at most 64 cells, down to the exact solve on the
// 2-per-side grid, as one product with the coarse matrix; with a cell
// coefficient k_mg_tail_var, level by level); back up, a launch adds the
// bi/trilinear interpolation of the coarse correction, then `post` sweeps
// (again one tiled launch in 2D, the finest one also folding the residual
// norms).  Fields (u and v of the reaction-diffusion steps) are solved by the
// same launches (grid y = field).  These grids are small (a 256^2 field is
// 512 KiB), so the cycle is bound by launch and synchronisation latency, not
// by HBM: a solve enqueues several cycles before its first host check, and
// each cycle can be replayed from a captured HIP graph (use_graph).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>

#include "../../include/amrv_mg.h"
#include "errors.hpp"
#include "mg_internal.hpp"

namespace {

using amrv::split_idx;

constexpr int MG_MAXL = 14;   // n <= 8192: 13 levels down to 2 cells per side
constexpr int NFMAX = 2;
constexpr int TAIL_CELLS = 4096;
constexpr int TAIL_THREADS = 1024;  // the variable-coefficient tail
// threads of the tail: in 3D 512, whose 256 registers hold a restriction's reads
// (1,024 threads spilled, and the first touch of scratch memory cost 3 us)
template <int ND>
constexpr int tail_threads() {
  return ND == 3 ? 512 : 1024;
}
constexpr int COARSE_CELLS = 64;  // the tail's levels of at most this many cells: one matrix product
constexpr int PAR_LAM = 0;
constexpr int PAR_IDIAG = NFMAX;                       // + field * MG_MAXL + level
constexpr int PAR_IH2 = NFMAX + NFMAX * MG_MAXL;       // + level
constexpr int PAR_COUNT = PAR_IH2 + MG_MAXL;

struct MgDev {
  int nd, bc, nlev, nf;
  int n[MG_MAXL];
  int lg[MG_MAXL];              // log2(n[l])
  int cells[MG_MAXL];
  int loffv[MG_MAXL];           // LDS offset (doubles) of the variable-coefficient tail's phi_l, f_l, eps_l
  const double* eps[MG_MAXL];   // cell coefficient per level (variable-coefficient solves)
  double* phi[NFMAX][MG_MAXL];
  double* f[NFMAX][MG_MAXL];
  double* phi2[NFMAX][MG_MAXL]; // 2D levels above the tail: the tiled launches'
                                // second buffer (down writes it, up reads it)
  const double* par;
  double* cmat[NFMAX];        // [64 columns][64 cells]: the coarse matrix (null: grids below TAIL_CELLS)
  int split0;                 // level 0 (and every level above the tail) in split order
  unsigned long long* hpart;  // pinned host slots of per-block maxima: [2][NFMAX][maxb]
  int maxb;
};

struct MgPar {
  double v[PAR_COUNT];
};

struct RdK {
  int model;
  double Du, Dv, p1, p2, p3;
};

// neighbours with the boundary rule: periodic wrap, or (Neumann) the cell
// itself, whose value is the mirrored ghost
__device__ __forceinline__ int im(int i, int n, int bc) { return i > 0 ? i - 1 : (bc == AMRV_MG_PERIODIC ? n - 1 : 0); }
__device__ __forceinline__ int ip(int i, int n, int bc) { return i < n - 1 ? i + 1 : (bc == AMRV_MG_PERIODIC ? 0 : n - 1); }

// cell t of a level with n = 2^lg cells per side
template <int ND>
__device__ __forceinline__ void decode(int t, int n, int lg, int& x, int& y, int& z) {
  x = t & (n - 1);
  const int r = t >> lg;
  y = ND == 3 ? (r & (n - 1)) : r;
  z = ND == 3 ? (r >> lg) : 0;
}

// Laplacian: per direction ((w- + w+) - 2 w) * (1/h^2), added x, y, z
template <int ND>
__device__ __forceinline__ double lap_at(const double* a, int x, int y, int z, int n, int bc, double ih2) {
  const int row = (z * n + y) * n;
  const double w = a[row + x];
  double out = ((a[row + im(x, n, bc)] + a[row + ip(x, n, bc)]) - 2.0 * w) * ih2;
  out = out + ((a[(z * n + im(y, n, bc)) * n + x] + a[(z * n + ip(y, n, bc)) * n + x]) - 2.0 * w) * ih2;
  if constexpr (ND == 3)
    out = out + ((a[(im(z, n, bc) * n + y) * n + x] + a[(ip(z, n, bc) * n + y) * n + x]) - 2.0 * w) * ih2;
  return out;
}

// Gauss-Seidel update of one cell: phi = (sum of neighbours / h^2 - f) / (2 d / h^2 + lambda)
template <int ND>
__device__ __forceinline__ void gs_cell(double* p, const double* rhs, int x, int y, int z, int n, int bc, double ih2,
                                        double idiag) {
  const int row = (z * n + y) * n;
  double s = (p[row + im(x, n, bc)] + p[row + ip(x, n, bc)]) +
             (p[(z * n + im(y, n, bc)) * n + x] + p[(z * n + ip(y, n, bc)) * n + x]);
  if constexpr (ND == 3) s = s + (p[(im(z, n, bc) * n + y) * n + x] + p[(ip(z, n, bc) * n + y) * n + x]);
  p[row + x] = (s * ih2 - rhs[row + x]) * idiag;
}

// cell t of colour c among the cells with (x + y + z) % 2 == c
template <int ND>
__device__ __forceinline__ void colour_cell(int t, int n, int lg, int c, int& x, int& y, int& z) {
  const int xh = t & ((n >> 1) - 1);
  const int r = t >> (lg - 1);
  y = ND == 3 ? (r & (n - 1)) : r;
  z = ND == 3 ? (r >> lg) : 0;
  x = 2 * xh + ((y + z + c) & 1);
}

// residual f - (lap(phi) - lambda phi) of one fine cell
template <int ND>
__device__ __forceinline__ double resid(const double* p, const double* rhs, int x, int y, int z, int n, int bc,
                                        double ih2, double lam) {
  const int i = (z * n + y) * n + x;
  return rhs[i] - (lap_at<ND>(p, x, y, z, n, bc, ih2) - lam * p[i]);
}

// coarse cell (xc, yc, zc): mean of the children's residuals
template <int ND>
__device__ __forceinline__ double restrict_cell(const double* p, const double* rhs, int xc, int yc, int zc, int n,
                                                int bc, double ih2, double lam) {
  double s = 0.0;
#pragma unroll
  for (int dz = 0; dz < (ND == 3 ? 2 : 1); dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++) s += resid<ND>(p, rhs, 2 * xc + dx, 2 * yc + dy, 2 * zc + dz, n, bc, ih2, lam);
  return s * (ND == 3 ? 0.125 : 0.25);
}

// ---- variable coefficient: div(eps grad phi) - lambda phi, face coefficient
// the mean of the two cells; a neighbour that is the cell itself (a Neumann
// face) contributes no flux -----------------------------------------------

template <int ND>
__device__ __forceinline__ void nbr_list(int x, int y, int z, int n, int bc, int* j) {
  const int row = (z * n + y) * n;
  j[0] = row + im(x, n, bc);
  j[1] = row + ip(x, n, bc);
  j[2] = (z * n + im(y, n, bc)) * n + x;
  j[3] = (z * n + ip(y, n, bc)) * n + x;
  if constexpr (ND == 3) {
    j[4] = (im(z, n, bc) * n + y) * n + x;
    j[5] = (ip(z, n, bc) * n + y) * n + x;
  }
}

template <int ND>
__device__ __forceinline__ void gs_cell_var(double* p, const double* rhs, const double* e, int x, int y, int z, int n,
                                            int bc, double ih2, double lam) {
  const int i = (z * n + y) * n + x;
  int j[2 * ND];
  nbr_list<ND>(x, y, z, n, bc, j);
  double num = 0.0, den = 0.0;
#pragma unroll
  for (int k = 0; k < 2 * ND; k++)
    if (j[k] != i) {
      const double ef = 0.5 * (e[i] + e[j[k]]);
      num += ef * p[j[k]];
      den += ef;
    }
  p[i] = (num * ih2 - rhs[i]) / (den * ih2 + lam);
}

template <int ND>
__device__ __forceinline__ double resid_var(const double* p, const double* rhs, const double* e, int x, int y, int z,
                                            int n, int bc, double ih2, double lam) {
  const int i = (z * n + y) * n + x;
  int j[2 * ND];
  nbr_list<ND>(x, y, z, n, bc, j);
  double a = 0.0;
#pragma unroll
  for (int k = 0; k < 2 * ND; k++)
    if (j[k] != i) a += 0.5 * (e[i] + e[j[k]]) * (p[j[k]] - p[i]);
  return rhs[i] - (a * ih2 - lam * p[i]);
}

template <int ND>
__device__ __forceinline__ double restrict_cell_var(const double* p, const double* rhs, const double* e, int xc, int yc,
                                                    int zc, int n, int bc, double ih2, double lam) {
  double s = 0.0;
#pragma unroll
  for (int dz = 0; dz < (ND == 3 ? 2 : 1); dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++)
        s += resid_var<ND>(p, rhs, e, 2 * xc + dx, 2 * yc + dy, 2 * zc + dz, n, bc, ih2, lam);
  return s * (ND == 3 ? 0.125 : 0.25);
}

// bi/trilinear interpolation of the coarse correction at fine cell (x, y, z):
// weight 3/4 on the parent and 1/4 on the parent's neighbour on the side of
// the fine cell, per direction (boundary rule as for the stencil)
template <int ND>
__device__ __forceinline__ double prolong_cell(const double* e, int x, int y, int z, int nc, int bc) {
  const int xc = x >> 1, yc = y >> 1, zc = z >> 1;
  const int xn = (x & 1) ? ip(xc, nc, bc) : im(xc, nc, bc);
  const int yn = (y & 1) ? ip(yc, nc, bc) : im(yc, nc, bc);
  auto plane = [&](int zz) {
    const double a = 0.75 * e[(zz * nc + yc) * nc + xc] + 0.25 * e[(zz * nc + yc) * nc + xn];
    const double b = 0.75 * e[(zz * nc + yn) * nc + xc] + 0.25 * e[(zz * nc + yn) * nc + xn];
    return 0.75 * a + 0.25 * b;
  };
  if constexpr (ND == 2) {
    return plane(0);
  } else {
    const int zn = (z & 1) ? ip(zc, nc, bc) : im(zc, nc, bc);
    return 0.75 * plane(zc) + 0.25 * plane(zn);
  }
}

__device__ __forceinline__ double par_ih2(const MgDev& g, int l) { return g.par[PAR_IH2 + l]; }
__device__ __forceinline__ double par_idiag(const MgDev& g, int f, int l) { return g.par[PAR_IDIAG + f * MG_MAXL + l]; }
__device__ __forceinline__ double par_lam(const MgDev& g, int f) { return g.par[PAR_LAM + f]; }

// ---- level kernels (HBM levels above the tail) ---------------------------

template <int ND, bool VAR>
__global__ void __launch_bounds__(256) k_mg_smooth(MgDev g, int l, int c) {
  const int f = blockIdx.y;
  const int n = g.n[l];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (g.cells[l] >> 1)) return;
  int x, y, z;
  colour_cell<ND>(t, n, g.lg[l], c, x, y, z);
  if constexpr (VAR)
    gs_cell_var<ND>(g.phi[f][l], g.f[f][l], g.eps[l], x, y, z, n, g.bc, par_ih2(g, l), par_lam(g, f));
  else
    gs_cell<ND>(g.phi[f][l], g.f[f][l], x, y, z, n, g.bc, par_ih2(g, l), par_idiag(g, f, l));
}

template <int ND, bool VAR>
__global__ void __launch_bounds__(256) k_mg_restrict(MgDev g, int l) {
  const int f = blockIdx.y;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[l + 1]) return;
  int x, y, z;
  decode<ND>(t, g.n[l + 1], g.lg[l + 1], x, y, z);
  if constexpr (VAR)
    g.f[f][l + 1][t] = restrict_cell_var<ND>(g.phi[f][l], g.f[f][l], g.eps[l], x, y, z, g.n[l], g.bc, par_ih2(g, l),
                                             par_lam(g, f));
  else
    g.f[f][l + 1][t] =
        restrict_cell<ND>(g.phi[f][l], g.f[f][l], x, y, z, g.n[l], g.bc, par_ih2(g, l), par_lam(g, f));
  g.phi[f][l + 1][t] = 0.0;
}

// coefficient of level l + 1: the mean of the 2^d children
template <int ND>
__global__ void __launch_bounds__(256) k_mg_eps_restrict(MgDev g, int l, double* out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[l + 1]) return;
  int x, y, z;
  decode<ND>(t, g.n[l + 1], g.lg[l + 1], x, y, z);
  const int n = g.n[l];
  const double* e = g.eps[l];
  double s = 0.0;
  for (int dz = 0; dz < (ND == 3 ? 2 : 1); dz++)
    for (int dy = 0; dy < 2; dy++)
      for (int dx = 0; dx < 2; dx++) s += e[((2 * z + dz) * n + 2 * y + dy) * n + 2 * x + dx];
  out[t] = s * (ND == 3 ? 0.125 : 0.25);
}

template <int ND>
__global__ void __launch_bounds__(256) k_mg_prolong(MgDev g, int l) {
  const int f = blockIdx.y;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[l]) return;
  int x, y, z;
  decode<ND>(t, g.n[l], g.lg[l], x, y, z);
  g.phi[f][l][t] += prolong_cell<ND>(g.phi[f][l + 1], x, y, z, g.n[l + 1], g.bc);
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

// Block maxima of non-negative doubles as bit patterns (NaN sorts above every
// number), written by each block into its own slot of the pinned host buffer
// (the residual maxima of field f in row f, the |f| maxima in row NFMAX + f);
// the host folds the launch's slots once it has completed.  No atomics: many
// blocks folding into one address serialise.
__device__ void fold_norms(const MgDev& g, int f, unsigned long long a, unsigned long long b, int with_f) {
  __shared__ unsigned long long sr[16], sf[16];
  a = wave_max_u64(a);
  b = wave_max_u64(b);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sr[w] = a;
    sf[w] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x >> 6); i++) {
      a = sr[i] > a ? sr[i] : a;
      b = sf[i] > b ? sf[i] : b;
    }
    g.hpart[(size_t)f * g.maxb + blockIdx.x] = a;
    if (with_f) g.hpart[(size_t)(NFMAX + f) * g.maxb + blockIdx.x] = b;
  }
}

// max |residual| (and with with_f, max |f|) of level 0 per field
template <int ND, bool VAR>
__global__ void __launch_bounds__(256) k_mg_resnorm(MgDev g, int with_f) {
  const int f = blockIdx.y;
  unsigned long long br = 0, bf = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < g.cells[0]; t += gridDim.x * blockDim.x) {
    int x, y, z;
    decode<ND>(t, g.n[0], g.lg[0], x, y, z);
    double r;
    if constexpr (VAR)
      r = resid_var<ND>(g.phi[f][0], g.f[f][0], g.eps[0], x, y, z, g.n[0], g.bc, par_ih2(g, 0), par_lam(g, f));
    else
      r = resid<ND>(g.phi[f][0], g.f[f][0], x, y, z, g.n[0], g.bc, par_ih2(g, 0), par_lam(g, f));
    const unsigned long long a = (unsigned long long)__double_as_longlong(fabs(r));
    const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(g.f[f][0][t]));
    br = a > br ? a : br;
    bf = b > bf ? b : bf;
  }
  fold_norms(g, f, br, bf, with_f);
}


__global__ void k_mg_set(double* dst, MgPar v) {
  const int i = threadIdx.x;
  if (i < PAR_COUNT) dst[i] = v.v[i];
}

// ---- tiled 2D level kernels ---------------------------------------------
// One workgroup per 32x32 tile of a level above the tail: the tile and a halo
// ring of H cells (clipped at Neumann domain faces, wrapped on periodic ones)
// are staged in LDS and the red-black sweeps are repeated over the whole
// staged region; a cell whose neighbours are not all staged (the open edge
// of the halo) is never updated, so after k half-sweeps every cell at least
// k cells from the open edge holds exactly the value the global sweeps give
// it (same neighbours, same arithmetic).  `down` sweeps pre times, forms the
// residual on the tile, restricts it and clears the coarse correction (H =
// 2 pre + 1); `up` adds the interpolated coarse correction over the region,
// sweeps post times (H = 2 post, + 1 when it also folds the residual norm
// of the finest level).  A launch never writes the array it stages from
// (blocks that start late would read a neighbour's new tile): down reads phi
// and writes phi2, up reads phi2 and writes phi.

constexpr int TS = 32;                 // tile side
constexpr int TT = 1024;               // threads per tile: a phase (half-sweep) is bound by its instructions per
                                       // thread; 256 threads took four rows each where these take one or two
                                       // (finest up 14.4 -> 7.9 us, down 8.3 -> 6.2 us at 256^2, two fields)
constexpr int RP = 64;                 // LDS row pitch of a staged region
constexpr int HMAX = 9;                // largest halo: pre, post <= 4
constexpr int RMAX = TS + 2 * HMAX;    // largest staged rows and columns

struct Region {
  int gx0, gy0, w, h;
  bool open[4];  // x-, x+, y-, y+ edges that cut the domain (not a Neumann face)
};

__device__ __forceinline__ Region region2d(int x0, int y0, int n, int H, int bc) {
  Region r;
  if (bc == AMRV_MG_PERIODIC) {
    r.gx0 = x0 - H;
    r.gy0 = y0 - H;
    r.w = r.h = TS + 2 * H;
    r.open[0] = r.open[1] = r.open[2] = r.open[3] = true;
  } else {
    r.gx0 = max(x0 - H, 0);
    r.gy0 = max(y0 - H, 0);
    const int x1 = min(x0 + TS + H, n), y1 = min(y0 + TS + H, n);
    r.w = x1 - r.gx0;
    r.h = y1 - r.gy0;
    r.open[0] = r.gx0 > 0;
    r.open[1] = x1 < n;
    r.open[2] = r.gy0 > 0;
    r.open[3] = y1 < n;
  }
  return r;
}

__device__ __forceinline__ int wrapn(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// The coarse cells a region's interpolation reads: parents (gx >> 1 of the
// unwrapped fine coordinate) and their neighbours, staged with the boundary
// rule applied (wrap, or the mirrored cell at a Neumann face) in an
// EP-pitched LDS block, so each fine cell interpolates from LDS with the
// weights and order of prolong_cell.
constexpr int EP = 32;
constexpr int EMAX = RMAX / 2 + 3;

struct CoarseWin {
  int cx0, cy0;
};

__device__ __forceinline__ CoarseWin stage_coarse(double* E, const Region& r, int nc, const double* e, int bc) {
  CoarseWin c;
  c.cx0 = (r.gx0 >> 1) - 1;
  c.cy0 = (r.gy0 >> 1) - 1;
  const int cw = ((r.gx0 + r.w - 1) >> 1) - c.cx0 + 2, ch = ((r.gy0 + r.h - 1) >> 1) - c.cy0 + 2;
  constexpr int K = (EMAX * EP + TT - 1) / TT;
  double v[K];
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int i = threadIdx.x + TT * k;
    const int lx = i & (EP - 1), ly = i >> 5;
    v[k] = 0.0;
    if (lx < cw && ly < ch) {
      int gx = c.cx0 + lx, gy = c.cy0 + ly;
      if (bc == AMRV_MG_PERIODIC) {
        gx = wrapn(gx, nc);
        gy = wrapn(gy, nc);
      } else {
        gx = min(max(gx, 0), nc - 1);
        gy = min(max(gy, 0), nc - 1);
      }
      v[k] = e[gy * nc + gx];
    }
  }
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int i = threadIdx.x + TT * k;
    const int lx = i & (EP - 1), ly = i >> 5;
    if (lx < cw && ly < ch) E[ly * EP + lx] = v[k];
  }
  return c;
}

// prolong_cell's interpolation at the unwrapped fine cell (ux, uy) from the
// staged coarse block
__device__ __forceinline__ double prolong_lds(const double* E, const CoarseWin& c, int ux, int uy) {
  const int xc = (ux >> 1) - c.cx0, yc = (uy >> 1) - c.cy0;
  const int xn = (ux & 1) ? xc + 1 : xc - 1, yn = (uy & 1) ? yc + 1 : yc - 1;
  const double a = 0.75 * E[yc * EP + xc] + 0.25 * E[yc * EP + xn];
  const double b = 0.75 * E[yn * EP + xc] + 0.25 * E[yn * EP + xn];
  return 0.75 * a + 0.25 * b;
}

// stage phi (+ the interpolated coarse correction when E != null) and f of
// the region into LDS (row pitch RP); every global load is issued before the
// first one is waited for
__device__ __forceinline__ void stage_region(double* P, double* F, const Region& r, int n, const double* phi,
                                             const double* rhs, const double* E, const CoarseWin& cw) {
  constexpr int K = (RMAX * RP + TT - 1) / TT;
  double pv[K], fv[K];
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int i = threadIdx.x + TT * k;
    const int lx = i & (RP - 1), ly = i >> 6;
    pv[k] = fv[k] = 0.0;
    if (lx < r.w && ly < r.h) {
      const int gx = wrapn(r.gx0 + lx, n), gy = wrapn(r.gy0 + ly, n);
      pv[k] = phi[gy * n + gx];
      fv[k] = rhs[gy * n + gx];
    }
  }
  if (E) {
#pragma unroll
    for (int k = 0; k < K; k++) {
      const int i = threadIdx.x + TT * k;
      const int lx = i & (RP - 1), ly = i >> 6;
      if (lx < r.w && ly < r.h) pv[k] = pv[k] + prolong_lds(E, cw, r.gx0 + lx, r.gy0 + ly);
    }
  }
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int i = threadIdx.x + TT * k;
    const int lx = i & (RP - 1), ly = i >> 6;
    if (lx < r.w && ly < r.h) {
      P[i] = pv[k];
      F[i] = fv[k];
    }
  }
}

// one half-sweep of colour c over the staged region: 32 lanes per row take
// the row's cells of that colour; every new value is computed before any is
// stored (a half-sweep reads only the other colour, so no barrier is needed
// between the two passes).  A cell with a neighbour beyond an open edge is
// left alone.
__device__ __forceinline__ void tile_halfsweep(double* P, const double* F, const Region& r, int c, double ih2,
                                               double idiag) {
  constexpr int RR = TT / 32, K = (RMAX + RR - 1) / RR;
  const int j = threadIdx.x & 31, r0 = threadIdx.x >> 5;
  double nv[K];
  bool ok[K];
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int ly = r0 + RR * k;
    const int lx = 2 * j + ((c + r.gx0 + r.gy0 + ly) & 1);
    const int i = ly * RP + lx;
    ok[k] = ly < r.h && lx < r.w && !(lx == 0 && r.open[0]) && !(lx == r.w - 1 && r.open[1]) &&
            !(ly == 0 && r.open[2]) && !(ly == r.h - 1 && r.open[3]);
    nv[k] = 0.0;
    if (ok[k]) {
      const int xm = lx == 0 ? i : i - 1, xp = lx == r.w - 1 ? i : i + 1;
      const int ym = ly == 0 ? i : i - RP, yp = ly == r.h - 1 ? i : i + RP;
      const double sum = (P[xm] + P[xp]) + (P[ym] + P[yp]);
      nv[k] = (sum * ih2 - F[i]) * idiag;
    }
  }
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int ly = r0 + RR * k;
    const int lx = 2 * j + ((c + r.gx0 + r.gy0 + ly) & 1);
    if (ok[k]) P[ly * RP + lx] = nv[k];
  }
}

// residual at a staged cell whose neighbours are all staged
__device__ __forceinline__ double tile_resid(const double* P, const double* F, const Region& r, int lx, int ly,
                                             double ih2, double lam) {
  const int i = ly * RP + lx;
  const int xm = lx == 0 ? i : i - 1, xp = lx == r.w - 1 ? i : i + 1;
  const int ym = ly == 0 ? i : i - RP, yp = ly == r.h - 1 ? i : i + RP;
  const double w = P[i];
  double lap = ((P[xm] + P[xp]) - 2.0 * w) * ih2;
  lap = lap + ((P[ym] + P[yp]) - 2.0 * w) * ih2;
  return F[i] - (lap - lam * w);
}

__global__ void __launch_bounds__(TT) k_mg_down2d(MgDev g, int l, int pre) {
  __shared__ double P[RMAX * RP], F[RMAX * RP];
  const int f = blockIdx.y, n = g.n[l], nt = n / TS;
  const int x0 = (blockIdx.x % nt) * TS, y0 = (blockIdx.x / nt) * TS;
  const Region r = region2d(x0, y0, n, 2 * pre + 1, g.bc);
  stage_region(P, F, r, n, g.phi[f][l], g.f[f][l], nullptr, CoarseWin{0, 0});
  __syncthreads();
  const double ih2 = par_ih2(g, l), idg = par_idiag(g, f, l), lam = par_lam(g, f);
  for (int s = 0; s < pre; s++)
    for (int c = 0; c < 2; c++) {
      tile_halfsweep(P, F, r, c, ih2, idg);
      __syncthreads();
    }
  if (threadIdx.x < TS * TS / 4) {
    const int cx = threadIdx.x & (TS / 2 - 1), cy = threadIdx.x >> 4;
    const int bx = x0 - r.gx0 + 2 * cx, by = y0 - r.gy0 + 2 * cy;
    double sum = 0.0;
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++) sum += tile_resid(P, F, r, bx + dx, by + dy, ih2, lam);
    const int nc = n >> 1;
    const int ci = (y0 / 2 + cy) * nc + (x0 / 2 + cx);
    g.f[f][l + 1][ci] = sum * 0.25;
    g.phi[f][l + 1][ci] = 0.0;
  }
  double* out = g.phi2[f][l];  // other blocks of this launch still stage phi
#pragma unroll
  for (int k = 0; k < TS * TS / TT; k++) {
    const int tx = threadIdx.x & (TS - 1), ty = (threadIdx.x >> 5) + (TT / TS) * k;
    out[(y0 + ty) * n + x0 + tx] = P[(y0 + ty - r.gy0) * RP + (x0 + tx - r.gx0)];
  }
}

__global__ void __launch_bounds__(TT) k_mg_up2d(MgDev g, int l, int post, int norm) {
  __shared__ double P[RMAX * RP], F[RMAX * RP], E[EMAX * EP];
  const int f = blockIdx.y, n = g.n[l], nt = n / TS;
  const int x0 = (blockIdx.x % nt) * TS, y0 = (blockIdx.x / nt) * TS;
  const Region r = region2d(x0, y0, n, 2 * post + (norm ? 1 : 0), g.bc);
  const CoarseWin cw = stage_coarse(E, r, n >> 1, g.phi[f][l + 1], g.bc);
  __syncthreads();
  stage_region(P, F, r, n, g.phi2[f][l], g.f[f][l], E, cw);
  __syncthreads();
  const double ih2 = par_ih2(g, l), idg = par_idiag(g, f, l), lam = par_lam(g, f);
  for (int s = 0; s < post; s++)
    for (int c = 0; c < 2; c++) {
      tile_halfsweep(P, F, r, c, ih2, idg);
      __syncthreads();
    }
  double* out = g.phi[f][l];
  unsigned long long br = 0;
#pragma unroll
  for (int k = 0; k < TS * TS / TT; k++) {
    const int tx = threadIdx.x & (TS - 1), ty = (threadIdx.x >> 5) + (TT / TS) * k;
    const int lx = x0 + tx - r.gx0, ly = y0 + ty - r.gy0;
    out[(y0 + ty) * n + x0 + tx] = P[ly * RP + lx];
    if (norm) {
      const unsigned long long a =
          (unsigned long long)__double_as_longlong(fabs(tile_resid(P, F, r, lx, ly, ih2, lam)));
      br = a > br ? a : br;
    }
  }
  if (norm) fold_norms(g, f, br, 0ull, 0);
}

// ---- the coarse tail: every level from `top` down, one workgroup per field,
// all levels in LDS -------------------------------------------------------

// exact solve on the coarsest grid (2 cells per side): per direction the
// operator couples the two cells as c [[-1, 1], [1, -1]] (c = 1/h^2 with the
// mirrored Neumann ghost, 2/h^2 with the periodic wrap), so the 2^d Walsh
// patterns (-1)^popcount(k & cell) are its eigenvectors, with eigenvalue
// -2c per set bit of k, minus lambda.  For lambda = 0 the constant pattern
// has eigenvalue 0 and the correction gets no constant part.
// One wave: lane k forms the coefficient of pattern k, then cell k's sum.
template <int ND>
__device__ __forceinline__ void coarse_exact(double* P, const double* F, int bc, double ih2, double lam) {
  constexpr int C = 1 << ND;
  const int k = threadIdx.x & (C - 1);
  const double c2 = 2.0 * (bc == AMRV_MG_PERIODIC ? 2.0 : 1.0) * ih2;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < C; c++) s += (__popc(k & c) & 1) ? -F[c] : F[c];
  double mu = -lam;
#pragma unroll
  for (int d = 0; d < ND; d++)
    if ((k >> d) & 1) mu -= c2;
  const double hat = mu == 0.0 ? 0.0 : s / (mu * C);
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < C; q++) {
    const double h = __shfl(hat, q, 64);
    v += (__popc(q & k) & 1) ? -h : h;
  }
  if (threadIdx.x < C) P[k] = v;
}

// A tail level in LDS holds its two colours in two halves (mg_internal.hpp: the
// cells of one colour are then consecutive; two doubles apart, as in the natural
// order, they meet two-way bank conflicts).

// LDS indices of a thread's pairs and right-hand sides, formed once per level
// and kept in registers over its sweeps, so that a cell update is its
// neighbour reads, six operations and a store
template <int ND, int K>
struct TailPairs {
  bool ok[K];
  int p[K];
  int nb[2][K][2 * ND - 1];  // per colour: the outer x neighbour, then -y, +y, -z, +z (the inner x neighbour is p)
  double f[2][K];
};

template <int ND, int K>
__device__ __forceinline__ TailPairs<ND, K> tail_pairs(const double* F, int lg, int bc, int t0) {
  constexpr int NT = tail_threads<ND>();
  const int n = 1 << lg, nh = n >> 1, half = 1 << (ND * lg - 1);
  const bool per = bc == AMRV_MG_PERIODIC;
  TailPairs<ND, K> T;
#pragma unroll
  for (int k = 0; k < K; k++) {
    T.ok[k] = t0 + k * NT < half;
    const int p = T.ok[k] ? t0 + k * NT : 0;
    const int xh = p & (nh - 1), r = p >> (lg - 1), y = ND == 3 ? r & (n - 1) : r, z = ND == 3 ? r >> lg : 0;
    T.p[k] = p;
    T.f[0][k] = F[p];
    T.f[1][k] = F[half + p];
    // index of a neighbour for colour 0 and colour 1: in the other half, or (a
    // Neumann wall) the cell itself
    auto both = [&](bool edge, int in, int wrap, int& a0, int& a1) {
      const bool wall = edge && !per;
      const int q = wall ? p : (edge ? wrap : in);
      a0 = wall ? q : q + half;
      a1 = wall ? q + half : q;
    };
    int l0, l1, r0, r1;
    both(xh == 0, p - 1, p + nh - 1, l0, l1);
    both(xh == nh - 1, p + 1, p - nh + 1, r0, r1);
    const bool right = (y + z) & 1;  // the cell of colour 0 is the pair's right one
    T.nb[0][k][0] = right ? r0 : l0;
    T.nb[1][k][0] = right ? l1 : r1;
    both(y == 0, p - nh, p + ((n - 1) << (lg - 1)), T.nb[0][k][1], T.nb[1][k][1]);
    both(y == n - 1, p + nh, p - ((n - 1) << (lg - 1)), T.nb[0][k][2], T.nb[1][k][2]);
    if constexpr (ND == 3) {
      const int zs = 1 << (2 * lg - 1);
      both(z == 0, p - zs, p + half - zs, T.nb[0][k][3], T.nb[1][k][3]);
      both(z == n - 1, p + zs, p - half + zs, T.nb[0][k][4], T.nb[1][k][4]);
    }
  }
  return T;
}

// `sweeps` red-black sweeps on a level, without the first half-sweep when the
// level's values already include it
template <int ND, int K>
__device__ __forceinline__ void tail_sweeps(const TailPairs<ND, K>& T, double* P, int half, int sweeps,
                                            bool first_done, double ih2, double idg) {
  auto half_sweep = [&](auto colour) {
    constexpr int c = decltype(colour)::value;
    double* own = P + (c ? half : 0);
    const double* other = P + (c ? 0 : half);
    double nv[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
      const int* b = T.nb[c][k];
      double sum = (other[T.p[k]] + P[b[0]]) + (P[b[1]] + P[b[2]]);
      if constexpr (ND == 3) sum = sum + (P[b[3]] + P[b[4]]);
      nv[k] = (sum * ih2 - T.f[c][k]) * idg;
    }
    // a half-sweep reads the other colour (and a wall cell its own value): no
    // barrier before the stores
#pragma unroll
    for (int k = 0; k < K; k++)
      if (T.ok[k]) own[T.p[k]] = nv[k];
    __syncthreads();
  };
  for (int s = 0; s < sweeps; s++) {
    if (s || !first_done) half_sweep(std::integral_constant<int, 0>{});
    half_sweep(std::integral_constant<int, 1>{});
  }
}

// the coarse right-hand side (the children's mean residual, restrict_cell's
// arithmetic with each value read once) and, for the zero initial guess, the
// coarse level after its first half-sweep: colour 0 at -f / diag, colour 1 at
// 0; the matrix level (SPLIT false, natural order) takes the right-hand side only
template <int ND, bool SPLIT>
__device__ __forceinline__ void tail_restrict(const double* P, const double* F, double* Pc, double* Fc, int t, int lg,
                                              int bc, double ih2, double lam, double idgc) {
  int xc, yc, zc;
  const int n = 1 << lg, nc = n >> 1, half = 1 << (ND * lg - 1), lgc = lg - 1;
  const bool per = bc == AMRV_MG_PERIODIC;
  decode<ND>(t, nc, lgc, xc, yc, zc);
  constexpr int NZ = ND == 3 ? 2 : 1;
  const int zs = 1 << (2 * lg - 1);  // pairs of a plane
  const int p00 = ND == 3 ? (((2 * zc << lg) + 2 * yc) << lgc) + xc : (2 * yc << lgc) + xc;
  double w[NZ][2][2];
#pragma unroll
  for (int dz = 0; dz < NZ; dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++) w[dz][dy][dx] = P[p00 + dy * nc + dz * zs + (((dx + dy + dz) & 1) ? half : 0)];
  double s = 0.0;
#pragma unroll
  for (int dz = 0; dz < NZ; dz++) {
    // the neighbours outside the 2^d children: the other colour, or (a Neumann
    // wall) the cell itself
    double fv[2][2], ex[2][2], ey[2][2], ez[2][2];
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++) {
        const int p = p00 + dy * nc + dz * zs, oo = ((dx + dy + dz) & 1) ? 0 : half;  // other half
        const int os = half - oo;                                                     // own half
        auto out = [&](bool edge, int in, int wrap) { return P[!edge ? oo + in : (per ? oo + wrap : os + p)]; };
        fv[dy][dx] = F[os + p];
        ex[dy][dx] = dx ? out(xc == nc - 1, p + 1, p - nc + 1) : out(xc == 0, p - 1, p + nc - 1);
        ey[dy][dx] = dy ? out(yc == nc - 1, p + nc, p - ((n - 1) << lgc)) : out(yc == 0, p - nc, p + ((n - 1) << lgc));
        if constexpr (ND == 3)
          ez[dy][dx] = dz ? out(zc == nc - 1, p + zs, p - half + zs) : out(zc == 0, p - zs, p + half - zs);
      }
#pragma unroll
    for (int dy = 0; dy < 2; dy++)
#pragma unroll
      for (int dx = 0; dx < 2; dx++) {
        const double v = w[dz][dy][dx];
        double lap = ((ex[dy][dx] + w[dz][dy][1 - dx]) - 2.0 * v) * ih2;
        lap = lap + ((ey[dy][dx] + w[dz][1 - dy][dx]) - 2.0 * v) * ih2;
        if constexpr (ND == 3) lap = lap + ((ez[dy][dx] + w[NZ - 1 - dz][dy][dx]) - 2.0 * v) * ih2;
        s += fv[dy][dx] - (lap - lam * v);
      }
    }
  const double fc = s * (ND == 3 ? 0.125 : 0.25);
  if constexpr (SPLIT) {
    const int i = split_idx<ND>(xc, yc, zc, lgc);
    Fc[i] = fc;
    Pc[i] = ((xc + yc + zc) & 1) ? 0.0 : (0.0 - fc) * idgc;
  } else {
    Fc[t] = fc;
  }
}

// the interpolated correction (prolong_cell's weights and order) added to the
// colour-1 cell of pair p and, with both, to its colour-0 cell; coarse level in
// split or natural order
template <int ND, bool SPLIT>
__device__ __forceinline__ void prolong_pair(double* P, const double* Pc, int p, int lg, int bc, bool both) {
  const int n = 1 << lg, half = 1 << (ND * lg - 1), lgc = lg - 1, nc = n >> 1;
  const int xc = p & (nc - 1), r = p >> lgc, y = ND == 3 ? r & (n - 1) : r, z = ND == 3 ? r >> lg : 0;
  const bool odd = (y + z) & 1;  // the cell of colour 1 is the pair's left one
  const int xl = im(xc, nc, bc), xr = ip(xc, nc, bc);
  const int xa = odd ? xl : xr, xb = odd ? xr : xl;  // toward the cell of colour 1, of colour 0
  auto row = [&](int yy, int zz, double& a, double& b) {
    const int base = ND == 3 ? ((zz << lgc) + yy) << lgc : yy << lgc;
    const int s = (yy + zz) & 1;
    auto e = [&](int x) {
      if constexpr (SPLIT) return Pc[((base + x) >> 1) + (((x + s) & 1) << (ND * lgc - 1))];
      return Pc[base + x];
    };
    const double c = 0.75 * e(xc);
    a = c + 0.25 * e(xa);
    b = both ? c + 0.25 * e(xb) : 0.0;
  };
  const int yc = y >> 1, yn = (y & 1) ? ip(yc, nc, bc) : im(yc, nc, bc);
  auto plane = [&](int zz, double& a, double& b) {
    double a0, b0, a1, b1;
    row(yc, zz, a0, b0);
    row(yn, zz, a1, b1);
    a = 0.75 * a0 + 0.25 * a1;
    b = 0.75 * b0 + 0.25 * b1;
  };
  double d1, d0;
  if constexpr (ND == 2) {
    plane(0, d1, d0);
  } else {
    const int zc = z >> 1, zn = (z & 1) ? ip(zc, nc, bc) : im(zc, nc, bc);
    double a0, b0, a1, b1;
    plane(zc, a0, b0);
    plane(zn, a1, b1);
    d1 = 0.75 * a0 + 0.25 * a1;
    d0 = 0.75 * b0 + 0.25 * b1;
  }
  P[half + p] += d1;
  if (both) P[p] += d0;
}

// on a tail level where the half-sweep of colour 0 that follows reads it: every
// cell of colour 1 and, with Neumann walls (a cell at one sums its own old
// value), both cells of every pair, which share their coarse rows; the others
// of colour 0 are recomputed without their old values
template <int ND, int K, bool SPLIT>
__device__ __forceinline__ void tail_prolong(double* P, const double* Pc, int t0, int lg, int bc) {
  constexpr int NT = tail_threads<ND>();
#pragma unroll
  for (int k = 0; k < K; k++) {
    const int p = t0 + k * NT;
    if (p < (1 << (ND * lg - 1))) prolong_pair<ND, SPLIT>(P, Pc, p, lg, bc, bc != AMRV_MG_PERIODIC);
  }
}

// a V-cycle on a grid of at most 64 cells by one wave (phi at P, f after it, the
// levels below after that, natural order in LDS): the coarse matrix's columns and grids with
// no larger level
template <int ND>
__device__ void wave_cycle(double* P, int lg0, int lev0, const MgDev& g, int f, int bc, int pre, int post,
                           double lam) {
  const int l = threadIdx.x;
  auto sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
  };
  auto level = [&](double* base, int lg) {  // start of level lg: 2 cells doubles per level above it
    for (int q = lg0; q > lg; q--) base += 2 << (ND * q);
    return base;
  };
  auto sweeps = [&](double* p, const double* r, int lg, int lev, int count) {
    const int n = 1 << lg, half = 1 << (ND * lg - 1);
    const double ih2 = par_ih2(g, lev), idg = par_idiag(g, f, lev);
    for (int s = 0; s < 2 * count; s++) {
      if (l < half) {
        int x, y, z;
        colour_cell<ND>(l, n, lg, s & 1, x, y, z);
        gs_cell<ND>(p, r, x, y, z, n, bc, ih2, idg);
      }
      sync();
    }
  };
  sync();  // the lanes' phi and f
  for (int lg = lg0, lev = lev0; lg > 1; lg--, lev++) {
    double* p = level(P, lg);
    double* r = p + (1 << (ND * lg));
    double* pc = level(P, lg - 1);
    sweeps(p, r, lg, lev, pre);
    if (l < (1 << (ND * (lg - 1)))) {
      int x, y, z;
      decode<ND>(l, 1 << (lg - 1), lg - 1, x, y, z);
      pc[(1 << (ND * (lg - 1))) + l] = restrict_cell<ND>(p, r, x, y, z, 1 << lg, bc, par_ih2(g, lev), lam);
      pc[l] = 0.0;
    }
    sync();
  }
  {
    double* p = level(P, 1);
    coarse_exact<ND>(p, p + (1 << ND), bc, par_ih2(g, lev0 + lg0 - 1), lam);
    sync();
  }
  for (int lg = 2, lev = lev0 + lg0 - 2; lg <= lg0; lg++, lev--) {
    double* p = level(P, lg);
    double* r = p + (1 << (ND * lg));
    const double* pc = level(P, lg - 1);
    if (l < (1 << (ND * lg))) {
      int x, y, z;
      decode<ND>(l, 1 << lg, lg, x, y, z);
      p[l] += prolong_cell<ND>(pc, x, y, z, 1 << (lg - 1), bc);
    }
    sync();
    sweeps(p, r, lg, lev, post);
  }
}

template <int ND>
__device__ void tail_sweeps_var(const MgDev& g, double* P, const double* F, const double* E, int l, int sweeps,
                                double ih2, double lam) {
  const int n = g.n[l], lg = g.lg[l], half = g.cells[l] >> 1;
  for (int s = 0; s < sweeps; s++)
    for (int c = 0; c < 2; c++) {
      for (int t = threadIdx.x; t < half; t += blockDim.x) {
        int x, y, z;
        colour_cell<ND>(t, n, lg, c, x, y, z);
        gs_cell_var<ND>(P, F, E, x, y, z, n, g.bc, ih2, lam);
      }
      __syncthreads();
    }
}

// exact solve on the 2-per-side grid with a coefficient: the 2^d x 2^d
// system of the operator, strictly diagonally dominant (lambda > 0), by
// Gaussian elimination without pivoting in one thread
template <int ND>
__device__ void coarse_exact_var(const MgDev& g, double* P, const double* F, const double* E, double ih2, double lam) {
  constexpr int C = 1 << ND;
  if (threadIdx.x == 0) {
    double A[C][C + 1];
    for (int r = 0; r < C; r++) {
      for (int c = 0; c <= C; c++) A[r][c] = 0.0;
      const int x = r & 1, y = (r >> 1) & 1, z = ND == 3 ? (r >> 2) & 1 : 0;
      int j[2 * ND];
      nbr_list<ND>(x, y, z, 2, g.bc, j);
      double diag = -lam;
      for (int k = 0; k < 2 * ND; k++)
        if (j[k] != r) {
          const double ef = 0.5 * (E[r] + E[j[k]]) * ih2;
          A[r][j[k]] += ef;
          diag -= ef;
        }
      A[r][r] += diag;
      A[r][C] = F[r];
    }
    for (int k = 0; k < C; k++)
      for (int r = k + 1; r < C; r++) {
        const double m = A[r][k] / A[k][k];
        for (int c = k; c <= C; c++) A[r][c] -= m * A[k][c];
      }
    for (int r = C - 1; r >= 0; r--) {
      double s = A[r][C];
      for (int c = r + 1; c < C; c++) s -= A[r][c] * P[c];
      P[r] = s / A[r][r];
    }
  }
  __syncthreads();
}

// The coarse matrix: a V-cycle from zero on the level of 64 cells (8^2 or 4^3)
// and everything below is a fixed linear map of its right-hand side, 64 x 64
// per field (32 KiB, in the two temporaries that only the explicit midpoint
// step uses: grids of fewer than 4,096 cells have no room for it there, and one
// wave runs the cycle).  Column j (one wave each) is the cycle's answer to a unit
// right-hand side at cell j; formed whenever the parameters (lambda) are set.
// As a product it replaces the last two or three levels' ~25 dependent phases,
// which kept one wave busy for 10 us of each cycle's tail.
template <int ND>
__global__ void __launch_bounds__(64) k_mg_coarse_matrix(MgDev g, int lev, int pre, int post) {
  __shared__ double lds[2 * (64 + 16 + 8)];
  const int j = blockIdx.x, f = blockIdx.y, l = threadIdx.x;
  lds[l] = 0.0;
  lds[64 + l] = l == j ? 1.0 : 0.0;
  __syncthreads();
  wave_cycle<ND>(lds, ND == 2 ? 3 : 2, lev, g, f, g.bc, pre, post, par_lam(g, f));
  __syncthreads();
  g.cmat[f][j * 64 + l] = lds[l];
}

// a grid of at most 64 cells: one V-cycle by one wave
template <int ND>
__global__ void __launch_bounds__(64) k_mg_small(MgDev g, int pre, int post) {
  __shared__ double lds[2 * (64 + 16 + 8)];
  const int f = blockIdx.x, l = threadIdx.x, C = g.cells[0];
  if (l < C) {
    lds[l] = g.phi[f][0][l];
    lds[C + l] = g.f[f][0][l];
  }
  __syncthreads();
  wave_cycle<ND>(lds, g.lg[0], 0, g, f, g.bc, pre, post, par_lam(g, f));
  __syncthreads();
  if (l < C) g.phi[f][0][l] = lds[l];
}

// Every level from `top` (more than 64 cells) down in one workgroup's LDS, from
// the zero guess where finer levels exist (zero != 0: phi of `top` is not read).
// One CU works through a chain of dependent phases, bound by the instructions
// of each phase and its barrier, so the phases are few and short: pairs of
// cells with precomputed indices, the half-sweep from zero folded into the
// restriction, colour 0 not prolonged, and the levels of at most 64 cells one
// product with the coarse matrix.  Two fields, Neumann: from 64^2 27.1 -> 15.3 us,
// from 16^3 27.9 -> 17.1 us (one thread per cell and phase before).
template <int ND, bool MAT>
__global__ void __launch_bounds__(tail_threads<ND>()) k_mg_tail(MgDev g, int top, int pre, int post, int zero) {
  constexpr int NT = tail_threads<ND>(), TK = TAIL_CELLS / 2 / NT;  // pairs of the top level per thread
  extern __shared__ double lds[];
  __shared__ double s_ih2[MG_MAXL], s_idg[MG_MAXL];
  const int f = blockIdx.x, tid = threadIdx.x, bc = g.bc;
  const int lg0 = g.lg[top], H0 = g.cells[top] >> 1;
  constexpr int LGM = ND == 2 ? 3 : 2;  // the matrix level: 8^2 or 4^3
  const int nl = lg0 - LGM;             // levels above it: 1..3 (2D), 1..2 (3D)
  const double2* fg = reinterpret_cast<const double2*>(g.f[f][top]);
  double2* pg = reinterpret_cast<double2*>(g.phi[f][top]);
  double2 fv[TK], pv[TK];
  constexpr int CG = NT / 64, CQ = 64 / CG;  // the matrix product: column groups, columns each
  double cm[CQ];
#pragma unroll
  for (int k = 0; k < TK; k++) {
    const int p = tid + k * NT;
    fv[k] = p < H0 ? fg[p] : double2{0.0, 0.0};
    pv[k] = !zero && p < H0 ? pg[p] : double2{0.0, 0.0};
  }
  if (tid < MG_MAXL) {
    s_ih2[tid] = par_ih2(g, tid);
    s_idg[tid] = par_idiag(g, f, tid);
  }
  const double lam = par_lam(g, f), idg_top = par_idiag(g, f, top);
  // this thread's part of the matrix product: cell tid % 64, columns CQ (tid / 64) .. + CQ - 1
#pragma unroll
  for (int q = 0; q < CQ; q++) cm[q] = MAT ? g.cmat[f][(CQ * (tid >> 6) + q) * 64 + (tid & 63)] : 0.0;
  // level i (0: top): phi, then f
  auto P = [&](int i) {
    double* b = lds;
    for (int q = 0; q < i; q++) b += 4 * (H0 >> (ND * q));
    return b;
  };
  auto F = [&](int i) { return P(i) + 2 * (H0 >> (ND * i)); };
  auto colour_x = [&](int p) {  // colour of the pair's left cell
    const int r = p >> (lg0 - 1);
    return ND == 3 ? ((r & ((1 << lg0) - 1)) + (r >> lg0)) & 1 : r & 1;
  };
#pragma unroll
  for (int k = 0; k < TK; k++) {
    const int p = tid + k * NT;
    if (p < H0) {
      const bool s = colour_x(p);
      const double f0 = s ? fv[k].y : fv[k].x, f1 = s ? fv[k].x : fv[k].y;
      F(0)[p] = f0;
      F(0)[H0 + p] = f1;
      P(0)[p] = zero ? (0.0 - f0) * idg_top : (s ? pv[k].y : pv[k].x);
      P(0)[H0 + p] = s ? pv[k].x : pv[k].y;
    }
  }
  __syncthreads();
  // the coarse right-hand side of level i into level i + 1 (the matrix level:
  // natural order, right-hand side only, after phi where one wave cycles on it)
  auto restrict_to = [&](int i) {
    const int cc = (2 * H0) >> (ND * (i + 1)), lg = lg0 - i;
    if (i + 1 == nl) {
      if (tid < 64) tail_restrict<ND, false>(P(i), F(i), nullptr, P(i + 1) + (MAT ? 0 : 64), tid, lg, bc, s_ih2[top + i], lam, 0.0);
    } else {
      for (int t = tid; t < cc; t += NT)
        tail_restrict<ND, true>(P(i), F(i), P(i + 1), F(i + 1), t, lg, bc, s_ih2[top + i], lam, s_idg[top + i + 1]);
    }
    __syncthreads();
  };
  {
    const TailPairs<ND, TK> T = tail_pairs<ND, TK>(F(0), lg0, bc, tid);
    tail_sweeps<ND, TK>(T, P(0), H0, pre, zero, s_ih2[top], s_idg[top]);
    restrict_to(0);
  }
  for (int i = 1; i < nl; i++) {
    const TailPairs<ND, 1> T = tail_pairs<ND, 1>(F(i), lg0 - i, bc, tid);
    tail_sweeps<ND, 1>(T, P(i), H0 >> (ND * i), pre, true, s_ih2[top + i], s_idg[top + i]);
    restrict_to(i);
  }
  // the matrix level: right-hand side at P(nl), partial sums of the
  // column groups after it, the answer over the right-hand side
  if constexpr (!MAT) {
    double* c = P(nl);
    if (tid < 64) {
      c[tid] = 0.0;
      wave_cycle<ND>(c, LGM, top + nl, g, f, bc, pre, post, lam);
    }
    __syncthreads();
  } else {
    double* c = P(nl);
    double a = cm[0] * c[CQ * (tid >> 6)];
#pragma unroll
    for (int q = 1; q < CQ; q++) a = a + cm[q] * c[CQ * (tid >> 6) + q];
    c[64 + tid] = a;
    __syncthreads();
    if (tid < 64) {
      double v = c[64 + tid];
#pragma unroll
      for (int q = 1; q < CG; q++) v = v + c[64 + 64 * q + tid];
      c[tid] = v;
    }
    __syncthreads();
  }
  for (int i = nl - 1; i > 0; i--) {
    const int lg = lg0 - i;
    if (i + 1 == nl)
      tail_prolong<ND, 1, false>(P(i), P(i + 1), tid, lg, bc);
    else
      tail_prolong<ND, 1, true>(P(i), P(i + 1), tid, lg, bc);
    __syncthreads();
    const TailPairs<ND, 1> T = tail_pairs<ND, 1>(F(i), lg, bc, tid);
    tail_sweeps<ND, 1>(T, P(i), H0 >> (ND * i), post, false, s_ih2[top + i], s_idg[top + i]);
  }
  {
    if (nl == 1)
      tail_prolong<ND, TK, false>(P(0), P(1), tid, lg0, bc);
    else
      tail_prolong<ND, TK, true>(P(0), P(1), tid, lg0, bc);
    __syncthreads();
    const TailPairs<ND, TK> T = tail_pairs<ND, TK>(F(0), lg0, bc, tid);
    tail_sweeps<ND, TK>(T, P(0), H0, post, false, s_ih2[top], s_idg[top]);
  }
#pragma unroll
  for (int k = 0; k < TK; k++) {
    const int p = tid + k * NT;
    if (p < H0) {
      const bool s = colour_x(p);
      const double a = P(0)[p], b = P(0)[H0 + p];
      pg[p] = s ? double2{b, a} : double2{a, b};
    }
  }
}

// the same with a cell coefficient, every level on the whole workgroup
template <int ND>
__global__ void __launch_bounds__(TAIL_THREADS) k_mg_tail_var(MgDev g, int top, int pre, int post) {
  extern __shared__ double lds[];
  __shared__ double s_ih2[MG_MAXL];
  const int f = blockIdx.x;
  if (threadIdx.x < MG_MAXL) s_ih2[threadIdx.x] = par_ih2(g, threadIdx.x);
  const double lam = par_lam(g, f);
  auto P = [&](int l) { return lds + g.loffv[l]; };
  auto F = [&](int l) { return P(l) + g.cells[l]; };
  auto E = [&](int l) { return P(l) + 2 * g.cells[l]; };
  const int last = g.nlev - 1;
  for (int i = threadIdx.x; i < g.cells[top]; i += blockDim.x) {
    P(top)[i] = g.phi[f][top][i];
    F(top)[i] = g.f[f][top][i];
  }
  for (int l = top; l <= last; l++)
    for (int i = threadIdx.x; i < g.cells[l]; i += blockDim.x) E(l)[i] = g.eps[l][i];
  __syncthreads();
  for (int l = top; l < last; l++) {
    tail_sweeps_var<ND>(g, P(l), F(l), E(l), l, pre, s_ih2[l], lam);
    const double ih2 = s_ih2[l];
    for (int t = threadIdx.x; t < g.cells[l + 1]; t += blockDim.x) {
      int x, y, z;
      decode<ND>(t, g.n[l + 1], g.lg[l + 1], x, y, z);
      F(l + 1)[t] = restrict_cell_var<ND>(P(l), F(l), E(l), x, y, z, g.n[l], g.bc, ih2, lam);
      P(l + 1)[t] = 0.0;
    }
    __syncthreads();
  }
  coarse_exact_var<ND>(g, P(last), F(last), E(last), s_ih2[last], lam);
  for (int l = last - 1; l >= top; l--) {
    for (int t = threadIdx.x; t < g.cells[l]; t += blockDim.x) {
      int x, y, z;
      decode<ND>(t, g.n[l], g.lg[l], x, y, z);
      P(l)[t] += prolong_cell<ND>(P(l + 1), x, y, z, g.n[l + 1], g.bc);
    }
    __syncthreads();
    tail_sweeps_var<ND>(g, P(l), F(l), E(l), l, post, s_ih2[l], lam);
  }
  for (int i = threadIdx.x; i < g.cells[top]; i += blockDim.x) g.phi[f][top][i] = P(top)[i];
}

// ---- 3D levels above the tail (constant coefficient): phi and f with the two
// colours in two halves (split_idx), so that a colour sweep reads one half of phi
// and one of f and writes one; in the natural order every line was moved for
// half its values (128^3, two fields: 20.9 -> 10.4 us a colour sweep, 4.8 TB/s) ---------------------

// workgroup i of n to a contiguous range per XCD (workgroups are dealt to the 8
// XCDs round robin), so that neighbouring rows and planes share an L2
__device__ __forceinline__ int xcd_chunk(int i, int n) {
  const int q = n >> 3, r = n & 7, x = i & 7;
  return x * q + (x < r ? x : r) + (i >> 3);
}

// a colour sweep, two pairs (16-byte loads) per thread
__global__ void __launch_bounds__(256) k_mg3_smooth(MgDev g, int l, int c) {
  const int f = blockIdx.y, n = g.n[l], lg = g.lg[l], nh = n >> 1, half = 1 << (3 * lg - 1);
  const int p = 2 * (xcd_chunk(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
  if (p >= half) return;
  const bool per = g.bc == AMRV_MG_PERIODIC;
  const int xh = p & (nh - 1), r = p >> (lg - 1), y = r & (n - 1), z = r >> lg;
  double* own = g.phi[f][l] + (c ? half : 0);
  const double* oth = g.phi[f][l] + (c ? 0 : half);
  auto two = [](const double* a) { return *reinterpret_cast<const double2*>(a); };
  // a neighbour row: the other colour, or (a Neumann wall) the cells themselves
  auto at = [&](bool edge, int in, int wrap) { return two(!edge ? oth + p + in : (per ? oth + p + wrap : own + p)); };
  const int zs = 1 << (2 * lg - 1);
  const double2 fv = two(g.f[f][l] + (c ? half : 0) + p);
  const double2 in = two(oth + p);
  const double2 ym = at(y == 0, -nh, (n - 1) * nh), yp = at(y == n - 1, nh, -(n - 1) * nh);
  const double2 zm = at(z == 0, -zs, half - zs), zp = at(z == n - 1, zs, zs - half);
  // the outer x neighbours: of a pair's right cells p + 1, p + 2, of its left
  // cells p - 1, p
  const bool right = (y + z + c) & 1;
  const double* q = right ? (xh + 2 == nh ? (per ? oth + p + 2 - nh : own + p + 1) : oth + p + 2)
                          : (xh == 0 ? (per ? oth + p + nh - 1 : own + p) : oth + p - 1);
  const double o = *q;
  const double o0 = right ? in.y : o, o1 = right ? o : in.x;
  const double ih2 = par_ih2(g, l), idg = par_idiag(g, f, l);
  double2 v;
  v.x = ((((in.x + o0) + (ym.x + yp.x)) + (zm.x + zp.x)) * ih2 - fv.x) * idg;
  v.y = ((((in.y + o1) + (ym.y + yp.y)) + (zm.y + zp.y)) * ih2 - fv.y) * idg;
  *reinterpret_cast<double2*>(own + p) = v;
}

// coarse right-hand side, and (a level above the tail) its values after the
// first half-sweep from zero (tail_restrict)
__global__ void __launch_bounds__(256) k_mg3_restrict(MgDev g, int l, int split) {
  const int f = blockIdx.y;
  const int t = xcd_chunk(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (t >= g.cells[l + 1]) return;
  const double ih2 = par_ih2(g, l), lam = par_lam(g, f);
  if (split)
    tail_restrict<3, true>(g.phi[f][l], g.f[f][l], g.phi[f][l + 1], g.f[f][l + 1], t, g.lg[l], g.bc, ih2, lam,
                           par_idiag(g, f, l + 1));
  else
    tail_restrict<3, false>(g.phi[f][l], g.f[f][l], nullptr, g.f[f][l + 1], t, g.lg[l], g.bc, ih2, lam, 0.0);
}

// the correction on colour 1 (and colour 0 at a Neumann wall: tail_prolong), one
// coarse cell per thread: its 8 children from the 27 coarse values around it,
// interpolated along x, y, z in turn as prolong_cell does (per pair of cells 12
// loads for two: 26.5 -> 20.3 us at 128^3, two fields)
template <bool SPLIT>
__global__ void __launch_bounds__(256) k_mg3_prolong(MgDev g, int l) {
  const int f = blockIdx.y, n = g.n[l], lg = g.lg[l], nc = n >> 1, lgc = lg - 1, bc = g.bc;
  const int t = xcd_chunk(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (t >= g.cells[l + 1]) return;
  int xc, yc, zc;
  decode<3>(t, nc, lgc, xc, yc, zc);
  const double* e = g.phi[f][l + 1];
  double* P = g.phi[f][l];
  const int half = 1 << (3 * lg - 1), pz = 1 << (2 * lg - 1);
  const int p0 = (((2 * zc << lg) + 2 * yc) << lgc) + xc;
  double w[2][2];  // the children of colour 1, loaded with the coarse values
#pragma unroll
  for (int dz = 0; dz < 2; dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++) w[dz][dy] = P[half + p0 + dy * nc + dz * pz];
  const int xs[3] = {im(xc, nc, bc), xc, ip(xc, nc, bc)}, ys[3] = {im(yc, nc, bc), yc, ip(yc, nc, bc)},
            zs[3] = {im(zc, nc, bc), zc, ip(zc, nc, bc)};
  double a[3][3][2];  // along x: the left and right child's value per coarse row
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int j = 0; j < 3; j++) {
      const int base = ((zs[k] << lgc) + ys[j]) << lgc, s = (ys[j] + zs[k]) & 1;
      auto at = [&](int x) { return SPLIT ? e[((base + x) >> 1) + (((x + s) & 1) << (3 * lgc - 1))] : e[base + x]; };
      const double c = 0.75 * at(xs[1]);
      a[k][j][0] = c + 0.25 * at(xs[0]);
      a[k][j][1] = c + 0.25 * at(xs[2]);
    }
  auto child = [&](int dx, int dy, int dz) {
    const int jn = dy ? 2 : 0, kn = dz ? 2 : 0;
    const double q0 = 0.75 * a[1][1][dx] + 0.25 * a[1][jn][dx], q1 = 0.75 * a[kn][1][dx] + 0.25 * a[kn][jn][dx];
    return 0.75 * q0 + 0.25 * q1;
  };
#pragma unroll
  for (int dz = 0; dz < 2; dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++) P[half + p0 + dy * nc + dz * pz] = w[dz][dy] + child((dy + dz + 1) & 1, dy, dz);
  if (bc == AMRV_MG_PERIODIC || !(xc == 0 || xc == nc - 1 || yc == 0 || yc == nc - 1 || zc == 0 || zc == nc - 1)) return;
#pragma unroll
  for (int dz = 0; dz < 2; dz++)
#pragma unroll
    for (int dy = 0; dy < 2; dy++) {
      const int dx = (dy + dz) & 1, x = 2 * xc + dx, y = 2 * yc + dy, z = 2 * zc + dz;
      if (x == 0 || x == n - 1 || y == 0 || y == n - 1 || z == 0 || z == n - 1)
        P[p0 + dy * nc + dz * pz] += child(dx, dy, dz);
    }
}

// the cells of pair p by colour: value and Laplacian (lap_at's sums and order)
__device__ __forceinline__ void pair_lap3(const double* P, int p, int n, int lg, int bc, double ih2, double* w,
                                          double* lap) {
  const int nh = n >> 1, half = 1 << (3 * lg - 1), zs = 1 << (2 * lg - 1);
  const bool per = bc == AMRV_MG_PERIODIC;
  const int xh = p & (nh - 1), r = p >> (lg - 1), y = r & (n - 1), z = r >> lg;
  const bool odd = (y + z) & 1;  // the cell of colour 0 is the pair's right one
  w[0] = P[p];
  w[1] = P[half + p];
#pragma unroll
  for (int c = 0; c < 2; c++) {
    const double* own = P + (c ? half : 0);
    const double* oth = P + (c ? 0 : half);
    auto at = [&](bool edge, int in, int wrap) { return !edge ? oth[p + in] : (per ? oth[p + wrap] : own[p]); };
    const bool right = c ? !odd : odd;
    const double o = right ? at(xh == nh - 1, 1, 1 - nh) : at(xh == 0, -1, nh - 1);
    const double ym = at(y == 0, -nh, (n - 1) * nh), yp = at(y == n - 1, nh, -(n - 1) * nh);
    const double zm = at(z == 0, -zs, half - zs), zp = at(z == n - 1, zs, zs - half);
    double a = ((o + w[1 - c]) - 2.0 * w[c]) * ih2;
    a = a + ((ym + yp) - 2.0 * w[c]) * ih2;
    lap[c] = a + ((zm + zp) - 2.0 * w[c]) * ih2;
  }
}

__global__ void __launch_bounds__(256) k_mg3_resnorm(MgDev g, int with_f) {
  const int f = blockIdx.y, n = g.n[0], lg = g.lg[0], half = g.cells[0] >> 1;
  const double ih2 = par_ih2(g, 0), lam = par_lam(g, f);
  unsigned long long br = 0, bf = 0;
  for (int p = xcd_chunk(blockIdx.x, gridDim.x) * 256 + threadIdx.x; p < half; p += gridDim.x * 256) {
    double w[2], lap[2];
    pair_lap3(g.phi[f][0], p, n, lg, g.bc, ih2, w, lap);
#pragma unroll
    for (int c = 0; c < 2; c++) {
      const double fv = g.f[f][0][(c ? half : 0) + p];
      const double r = fv - (lap[c] - lam * w[c]);
      const unsigned long long a = (unsigned long long)__double_as_longlong(fabs(r));
      const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(fv));
      br = a > br ? a : br;
      bf = b > bf ? b : bf;
    }
  }
  fold_norms(g, f, br, bf, with_f);
}

// a pair of cells of a caller's field, which need only be aligned as doubles are
// (one 16-byte access all the same: global memory takes those at any 4 bytes)
__device__ __forceinline__ double2 load_pair(const double* p) {
  double2 v;
  __builtin_memcpy(&v, p, sizeof v);
  return v;
}
__device__ __forceinline__ void store_pair(double* p, double2 v) { __builtin_memcpy(p, &v, sizeof v); }

// a natural-order field to and from a split array, one pair per thread
__global__ void __launch_bounds__(256) k_mg3_reorder(int lg, const double* src, double* dst, int to_split) {
  const int p = blockIdx.x * 256 + threadIdx.x, half = 1 << (3 * lg - 1);
  if (p >= half) return;
  const int n = 1 << lg, r = p >> (lg - 1);
  const bool odd = ((r & (n - 1)) + (r >> lg)) & 1;  // the left cell's colour
  if (to_split) {
    const double2 v = load_pair(src + 2 * (size_t)p);
    dst[p] = odd ? v.y : v.x;
    dst[half + p] = odd ? v.x : v.y;
  } else {
    const double a = src[p], b = src[half + p];
    store_pair(dst + 2 * (size_t)p, odd ? double2{b, a} : double2{a, b});
  }
}

// ---- divergence control of the MHD runs (Sec. 2.4): lap(phi) = div B*,
// B = B* - grad phi, central differences (w(+1) - w(-1)) * (n / 2L) ---------

template <int ND>
__device__ __forceinline__ double cdiff(const double* w, int x, int y, int z, int n, int bc, int d, double c) {
  if (d == 0) return (w[(z * n + y) * n + ip(x, n, bc)] - w[(z * n + y) * n + im(x, n, bc)]) * c;
  if (d == 1) return (w[(z * n + ip(y, n, bc)) * n + x] - w[(z * n + im(y, n, bc)) * n + x]) * c;
  return (w[(ip(z, n, bc) * n + y) * n + x] - w[(im(z, n, bc) * n + y) * n + x]) * c;
}

template <int ND>
__device__ __forceinline__ double cdiv(const double* b0, const double* b1, const double* b2, int x, int y, int z,
                                       int n, int bc, double c) {
  double d = cdiff<ND>(b0, x, y, z, n, bc, 0, c);
  d = d + cdiff<ND>(b1, x, y, z, n, bc, 1, c);
  if constexpr (ND == 3) d = d + cdiff<ND>(b2, x, y, z, n, bc, 2, c);
  return d;
}

// index in a level-0 array of phi or f of the cell of natural index t
template <int ND>
__device__ __forceinline__ int idx0(const MgDev& g, int t, int x, int y, int z) {
  if constexpr (ND == 3)
    if (g.split0) return split_idx<3>(x, y, z, g.lg[0]);
  return t;
}

// right-hand side div B*, initial guess 0
template <int ND>
__global__ void __launch_bounds__(256) k_mg_divb(MgDev g, const double* b0, const double* b1, const double* b2,
                                                 double c) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const int o = idx0<ND>(g, t, x, y, z);
  g.f[0][0][o] = cdiv<ND>(b0, b1, b2, x, y, z, g.n[0], g.bc, c);
  g.phi[0][0][o] = 0.0;
}

template <int ND>
__global__ void __launch_bounds__(256) k_mg_gradsub(MgDev g, double* b0, double* b1, double* b2, double c) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const double* phi = g.phi[0][0];
  const int n = g.n[0], bc = g.bc;
  auto at = [&](int xx, int yy, int zz) { return phi[idx0<ND>(g, (zz * n + yy) * n + xx, xx, yy, zz)]; };
  b0[t] = b0[t] - (at(ip(x, n, bc), y, z) - at(im(x, n, bc), y, z)) * c;
  b1[t] = b1[t] - (at(x, ip(y, n, bc), z) - at(x, im(y, n, bc), z)) * c;
  if constexpr (ND == 3) b2[t] = b2[t] - (at(x, y, ip(z, n, bc)) - at(x, y, im(z, n, bc))) * c;
}

// max |div B| into the host slots of row 0
template <int ND>
__global__ void __launch_bounds__(256) k_mg_divnorm(MgDev g, const double* b0, const double* b1, const double* b2,
                                                    double c) {
  unsigned long long m = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < g.cells[0]; t += gridDim.x * blockDim.x) {
    int x, y, z;
    decode<ND>(t, g.n[0], g.lg[0], x, y, z);
    const unsigned long long a =
        (unsigned long long)__double_as_longlong(fabs(cdiv<ND>(b0, b1, b2, x, y, z, g.n[0], g.bc, c)));
    m = a > m ? a : m;
  }
  fold_norms(g, 0, m, 0ull, 0);
}

// ---- reaction-diffusion (Sec. 2.5) ---------------------------------------

__device__ __forceinline__ void react(const RdK& p, double u, double v, double& ru, double& rv) {
  if (p.model == AMRV_RD_SCHNAKENBERG) {
    const double uuv = (u * u) * v;
    ru = p.p1 * ((p.p2 - u) + uuv);
    rv = p.p1 * (p.p3 - uuv);
  } else {
    const double uvv = u * (v * v);
    ru = p.p1 * (1.0 - u) - uvv;
    rv = uvv - (p.p1 + p.p2) * v;
  }
}

// out = base + c F(src), F = F0 + D lap (explicit Euler and midpoint stages)
template <int ND>
__global__ void __launch_bounds__(256) k_rd_explicit(MgDev g, RdK p, const double* bu, const double* bv,
                                                     const double* su, const double* sv, double* ou, double* ov,
                                                     double c) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const double ih2 = par_ih2(g, 0);
  double ru, rv;
  react(p, su[t], sv[t], ru, rv);
  const double fu = ru + p.Du * lap_at<ND>(su, x, y, z, g.n[0], g.bc, ih2);
  const double fv = rv + p.Dv * lap_at<ND>(sv, x, y, z, g.n[0], g.bc, ih2);
  ou[t] = bu[t] + c * fu;
  ov[t] = bv[t] + c * fv;
}

// split scheme: f = -lambda (w + dt F0(w)), initial guess w
template <int ND>
__global__ void __launch_bounds__(256) k_rd_split_rhs(MgDev g, RdK p, const double* u, const double* v, double dt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  double ru, rv;
  react(p, u[t], v[t], ru, rv);
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const int o = idx0<ND>(g, t, x, y, z);
  g.f[0][0][o] = -par_lam(g, 0) * (u[t] + dt * ru);
  g.f[1][0][o] = -par_lam(g, 1) * (v[t] + dt * rv);
  g.phi[0][0][o] = u[t];
  g.phi[1][0][o] = v[t];
}

// IMEX first stage: f = -lambda ((w + dt F0(w)) + (dt/2) D lap(w)), initial
// guess the explicit Euler predictor w + dt F(w); F(w) kept for the second
// stage
template <int ND>
__global__ void __launch_bounds__(256) k_rd_imex_rhs(MgDev g, RdK p, const double* u, const double* v, double* Eu,
                                                     double* Ev, double dt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const double ih2 = par_ih2(g, 0);
  double ru, rv;
  react(p, u[t], v[t], ru, rv);
  const double du = p.Du * lap_at<ND>(u, x, y, z, g.n[0], g.bc, ih2);
  const double dv = p.Dv * lap_at<ND>(v, x, y, z, g.n[0], g.bc, ih2);
  Eu[t] = ru + du;
  Ev[t] = rv + dv;
  const double hdt = 0.5 * dt;
  const int o = idx0<ND>(g, t, x, y, z);
  g.f[0][0][o] = -par_lam(g, 0) * ((u[t] + dt * ru) + hdt * du);
  g.f[1][0][o] = -par_lam(g, 1) * ((v[t] + dt * rv) + hdt * dv);
  g.phi[0][0][o] = u[t] + dt * (ru + du);
  g.phi[1][0][o] = v[t] + dt * (rv + dv);
}

// IMEX second stage: w1 = w + (dt/2) (F(w) + F(w*)), w* = the solve's phi
template <int ND>
__global__ void __launch_bounds__(256) k_rd_imex_final(MgDev g, RdK p, double* u, double* v, const double* Eu,
                                                       const double* Ev, double dt) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= g.cells[0]) return;
  int x, y, z;
  decode<ND>(t, g.n[0], g.lg[0], x, y, z);
  const double ih2 = par_ih2(g, 0);
  const double* su = g.phi[0][0];
  const double* sv = g.phi[1][0];
  double ru, rv;
  react(p, su[t], sv[t], ru, rv);
  const double fu = ru + p.Du * lap_at<ND>(su, x, y, z, g.n[0], g.bc, ih2);
  const double fv = rv + p.Dv * lap_at<ND>(sv, x, y, z, g.n[0], g.bc, ih2);
  const double hdt = 0.5 * dt;
  u[t] = u[t] + hdt * (Eu[t] + fu);
  v[t] = v[t] + hdt * (Ev[t] + fv);
}

// the same in 3D on split phi, one pair of cells per thread
__global__ void __launch_bounds__(256) k_rd3_imex_final(MgDev g, RdK p, double* u, double* v, const double* Eu,
                                                        const double* Ev, double dt) {
  const int q = xcd_chunk(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  if (q >= (g.cells[0] >> 1)) return;
  const int n = g.n[0], lg = g.lg[0], r = q >> (lg - 1);
  const bool odd = ((r & (n - 1)) + (r >> lg)) & 1;  // the left cell's colour
  const double ih2 = par_ih2(g, 0), hdt = 0.5 * dt;
  double su[2], sv[2], lu[2], lv[2], fu[2], fv[2];
  pair_lap3(g.phi[0][0], q, n, lg, g.bc, ih2, su, lu);
  pair_lap3(g.phi[1][0], q, n, lg, g.bc, ih2, sv, lv);
#pragma unroll
  for (int c = 0; c < 2; c++) {
    double ru, rv;
    react(p, su[c], sv[c], ru, rv);
    fu[c] = ru + p.Du * lu[c];
    fv[c] = rv + p.Dv * lv[c];
  }
  double* u2 = u + 2 * (size_t)q;
  double* v2 = v + 2 * (size_t)q;
  const double2 eu = reinterpret_cast<const double2*>(Eu)[q], ev = reinterpret_cast<const double2*>(Ev)[q];
  double2 a = load_pair(u2), b = load_pair(v2);
  a.x = a.x + hdt * (eu.x + (odd ? fu[1] : fu[0]));
  a.y = a.y + hdt * (eu.y + (odd ? fu[0] : fu[1]));
  b.x = b.x + hdt * (ev.x + (odd ? fv[1] : fv[0]));
  b.y = b.y + hdt * (ev.y + (odd ? fv[0] : fv[1]));
  store_pair(u2, a);
  store_pair(v2, b);
}

int blocks_of(int n) { return (n + 255) / 256; }

}  // namespace

struct amrv_mg {
  amrv_mg_config cfg{};
  MgDev g{};
  hipStream_t st = nullptr;
  double* par = nullptr;
  unsigned long long* hpart = nullptr;  // pinned slots of per-block maxima
  int nb_cycle = 0, nb_init = 0;        // blocks folding norms: a V-cycle's last launch, the initial norms
  double* tmp[4] = {nullptr, nullptr, nullptr, nullptr};
  int tail = 0;
  size_t tail_lds = 0;
  hipGraphExec_t gexec = nullptr;
  bool profile = false;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  double prof_ms = 0.0;
  int64_t prof_cycles = 0;
  int last_cycles = 0;  // V-cycles of the last reaction-diffusion solve
  bool var = false;     // a cell coefficient is set (div(eps grad phi) - lambda phi)
  size_t tail_lds_var = 0;
  int par_nf = 0;         // fields of the last parameter block set (0: none yet)
  double par_lam0 = 0.0;  // its field-0 lambda
  double* eps[MG_MAXL] = {};
};

namespace {

using amrv::set_error;

int hip_err(hipError_t e, const char* where) {
  return set_error(AMRV_EDEVICE, (std::string(where) + ": " + hipGetErrorString(e)).c_str());
}

#define MGCHK(expr)                                \
  do {                                             \
    hipError_t e_ = (expr);                        \
    if (e_ != hipSuccess) return hip_err(e_, #expr); \
  } while (0)

constexpr size_t ALIGN = 256;
size_t up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

int validate(const amrv_mg_config* c) {
  if (!c) return set_error(AMRV_EINVAL, "null config");
  if (c->ndim != 2 && c->ndim != 3) return set_error(AMRV_EINVAL, "ndim must be 2 or 3");
  const int nmax = c->ndim == 2 ? 8192 : 512;
  if (!is_pow2(c->n) || c->n < 4 || c->n > nmax)
    return set_error(AMRV_EINVAL, "n must be a power of two in 4..8192 (2D) or 4..512 (3D)");
  if (c->bc != AMRV_MG_PERIODIC && c->bc != AMRV_MG_NEUMANN) return set_error(AMRV_EINVAL, "unknown boundary");
  if (c->nfields < 1 || c->nfields > NFMAX) return set_error(AMRV_EINVAL, "nfields must be 1 or 2");
  if (c->pre_sweeps < 1 || c->pre_sweeps > 8 || c->post_sweeps < 1 || c->post_sweeps > 8)
    return set_error(AMRV_EINVAL, "pre and post sweeps must be in 1..8");
  if (c->smoother != AMRV_MG_TILED && c->smoother != AMRV_MG_PER_COLOUR) return set_error(AMRV_EINVAL, "unknown smoother");
  if (!(c->length > 0.0) || !std::isfinite(c->length)) return set_error(AMRV_EINVAL, "length must be positive");
  return 0;
}

struct MgLayout {
  int nlev = 0;
  size_t off_phi[NFMAX][MG_MAXL]{}, off_f[NFMAX][MG_MAXL]{}, off_phi2[NFMAX][MG_MAXL]{}, off_eps[MG_MAXL]{},
      off_tmp[4]{}, off_par = 0, total = 0;
};

MgLayout layout(const amrv_mg_config* c) {
  MgLayout L;
  int lv = 0;
  for (int n = c->n; n >= 2; n >>= 1) lv++;
  L.nlev = lv;
  size_t o = 0;
  for (int f = 0; f < c->nfields; f++)
    for (int l = 0; l < lv; l++) {
      size_t cells = 1;
      for (int d = 0; d < c->ndim; d++) cells *= (size_t)(c->n >> l);
      L.off_phi[f][l] = o;
      o += up(cells * 8);
      L.off_f[f][l] = o;
      o += up(cells * 8);
      if (c->ndim == 2 && cells > (size_t)TAIL_CELLS) {
        L.off_phi2[f][l] = o;
        o += up(cells * 8);
      }
    }
  for (int l = 0; l < lv; l++) {
    size_t cells = 1;
    for (int d = 0; d < c->ndim; d++) cells *= (size_t)(c->n >> l);
    L.off_eps[l] = o;
    o += up(cells * 8);
  }
  size_t c0 = 1;
  for (int d = 0; d < c->ndim; d++) c0 *= (size_t)c->n;
  for (int i = 0; i < 4; i++) {
    L.off_tmp[i] = o;
    o += up(c0 * 8);
  }
  L.off_par = o;
  o += up(PAR_COUNT * 8);
  L.total = o;
  return L;
}

bool tiled(const amrv_mg* m) {
  return !m->var && m->g.nd == 2 && m->cfg.smoother == AMRV_MG_TILED && m->tail > 0 &&
         2 * std::max(m->cfg.pre_sweeps, m->cfg.post_sweeps) + 1 <= HMAX;
}

// residual norms of level 0 (with_f: also max |f|), published to the pinned
// host copy by the launch's last block
template <int ND>
void enqueue_norms_nd(amrv_mg* m, int with_f) {
  const MgDev& g = m->g;
  if (ND == 3 && g.split0) {
    hipLaunchKernelGGL(k_mg3_resnorm, dim3(m->nb_init, g.nf), dim3(256), 0, m->st, g, with_f);
    return;
  }
  if (m->var)
    hipLaunchKernelGGL((k_mg_resnorm<ND, true>), dim3(m->nb_init, g.nf), dim3(256), 0, m->st, g, with_f);
  else
    hipLaunchKernelGGL((k_mg_resnorm<ND, false>), dim3(m->nb_init, g.nf), dim3(256), 0, m->st, g, with_f);
}

// one V-cycle, ending (norms) with the residual norms of its result
template <int ND>
void enqueue_vcycle_nd(amrv_mg* m, bool norms) {
  const MgDev& g = m->g;
  const int nf = g.nf;
  const int pre = m->cfg.pre_sweeps, post = m->cfg.post_sweeps;
  if (tiled(m)) {
    for (int l = 0; l < m->tail; l++)
      hipLaunchKernelGGL(k_mg_down2d, dim3((g.n[l] / TS) * (g.n[l] / TS), nf), dim3(TT), 0, m->st, g, l, pre);
  } else if (ND == 3 && g.split0) {
    for (int l = 0; l < m->tail; l++) {
      for (int h = l ? 1 : 0; h < 2 * pre; h++)  // below level 0 the restriction made the first half-sweep
        hipLaunchKernelGGL(k_mg3_smooth, dim3(blocks_of(g.cells[l] >> 2), nf), dim3(256), 0, m->st, g, l, h & 1);
      hipLaunchKernelGGL(k_mg3_restrict, dim3(blocks_of(g.cells[l + 1]), nf), dim3(256), 0, m->st, g, l,
                         l + 1 < m->tail ? 1 : 0);
    }
  } else {
    for (int l = 0; l < m->tail; l++) {
      for (int s = 0; s < pre; s++)
        for (int c = 0; c < 2; c++)
          if (m->var)
            hipLaunchKernelGGL((k_mg_smooth<ND, true>), dim3(blocks_of(g.cells[l] >> 1), nf), dim3(256), 0, m->st, g,
                               l, c);
          else if constexpr (ND == 2)
            hipLaunchKernelGGL((k_mg_smooth<ND, false>), dim3(blocks_of(g.cells[l] >> 1), nf), dim3(256), 0, m->st,
                               g, l, c);
      if (m->var)
        hipLaunchKernelGGL((k_mg_restrict<ND, true>), dim3(blocks_of(g.cells[l + 1]), nf), dim3(256), 0, m->st, g, l);
      else if constexpr (ND == 2)
        hipLaunchKernelGGL((k_mg_restrict<ND, false>), dim3(blocks_of(g.cells[l + 1]), nf), dim3(256), 0, m->st, g,
                           l);
    }
  }
  if (m->var)
    hipLaunchKernelGGL((k_mg_tail_var<ND>), dim3(nf), dim3(TAIL_THREADS), m->tail_lds_var, m->st, g, m->tail, pre,
                       post);
  else if (g.cells[0] <= COARSE_CELLS)
    hipLaunchKernelGGL((k_mg_small<ND>), dim3(nf), dim3(64), 0, m->st, g, pre, post);
  else if (g.cmat[0])
    hipLaunchKernelGGL((k_mg_tail<ND, true>), dim3(nf), dim3(tail_threads<ND>()), m->tail_lds, m->st, g, m->tail, pre,
                       post, m->tail > 0 ? 1 : 0);
  else
    hipLaunchKernelGGL((k_mg_tail<ND, false>), dim3(nf), dim3(tail_threads<ND>()), m->tail_lds, m->st, g, m->tail, pre,
                       post, m->tail > 0 ? 1 : 0);
  if (tiled(m)) {
    for (int l = m->tail - 1; l >= 0; l--)
      hipLaunchKernelGGL(k_mg_up2d, dim3((g.n[l] / TS) * (g.n[l] / TS), nf), dim3(TT), 0, m->st, g, l, post,
                         l == 0 && norms ? 1 : 0);
    return;  // the finest level's up launch folded the norms
  }
  if (ND == 3 && g.split0) {
    for (int l = m->tail - 1; l >= 0; l--) {
      if (l + 1 < m->tail)
        hipLaunchKernelGGL(k_mg3_prolong<true>, dim3(blocks_of(g.cells[l + 1]), nf), dim3(256), 0, m->st, g, l);
      else
        hipLaunchKernelGGL(k_mg3_prolong<false>, dim3(blocks_of(g.cells[l + 1]), nf), dim3(256), 0, m->st, g, l);
      for (int h = 0; h < 2 * post; h++)
        hipLaunchKernelGGL(k_mg3_smooth, dim3(blocks_of(g.cells[l] >> 2), nf), dim3(256), 0, m->st, g, l, h & 1);
    }
    if (norms) enqueue_norms_nd<ND>(m, 0);
    return;
  }
  for (int l = m->tail - 1; l >= 0; l--) {
    hipLaunchKernelGGL(k_mg_prolong<ND>, dim3(blocks_of(g.cells[l]), nf), dim3(256), 0, m->st, g, l);
    for (int s = 0; s < post; s++)
      for (int c = 0; c < 2; c++)
        if (m->var)
          hipLaunchKernelGGL((k_mg_smooth<ND, true>), dim3(blocks_of(g.cells[l] >> 1), nf), dim3(256), 0, m->st, g,
                             l, c);
        else if constexpr (ND == 2)
          hipLaunchKernelGGL((k_mg_smooth<ND, false>), dim3(blocks_of(g.cells[l] >> 1), nf), dim3(256), 0, m->st, g,
                             l, c);
  }
  if (norms) enqueue_norms_nd<ND>(m, 0);
}

void enqueue_vcycle(amrv_mg* m, bool norms = true) {
  if (m->g.nd == 2)
    enqueue_vcycle_nd<2>(m, norms);
  else
    enqueue_vcycle_nd<3>(m, norms);
}

// matrix: a V-cycle follows (else the explicit steps, which use its memory)
int set_params(amrv_mg* m, const double* lam, bool matrix = true) {
  MgPar P{};
  const double L = m->cfg.length;
  for (int l = 0; l < m->g.nlev; l++) {
    const double r = m->g.n[l] / L;
    P.v[PAR_IH2 + l] = r * r;
  }
  for (int f = 0; f < m->g.nf; f++) {
    P.v[PAR_LAM + f] = lam[f];
    for (int l = 0; l < m->g.nlev; l++)
      P.v[PAR_IDIAG + f * MG_MAXL + l] = 1.0 / (2.0 * m->g.nd * P.v[PAR_IH2 + l] + lam[f]);
  }
  hipLaunchKernelGGL(k_mg_set, dim3(1), dim3(64), 0, m->st, m->par, P);
  if (matrix && m->g.cmat[0] && !m->var) {
    int lev = 0;
    while (m->g.cells[lev] > COARSE_CELLS) lev++;
    hipLaunchKernelGGL(m->g.nd == 2 ? k_mg_coarse_matrix<2> : k_mg_coarse_matrix<3>, dim3(COARSE_CELLS, m->g.nf),
                       dim3(64), 0, m->st, m->g, lev, m->cfg.pre_sweeps, m->cfg.post_sweeps);
  }
  MGCHK(hipGetLastError());
  m->par_nf = matrix && !m->var ? m->g.nf : 0;
  m->par_lam0 = lam[0];
  return 0;
}

double bits_to_double(unsigned long long b) {
  double d;
  std::memcpy(&d, &b, 8);
  return d;
}

int launch_cycle(amrv_mg* m) {
  if (m->cfg.use_graph) {
    if (!m->gexec) {
      hipGraph_t gr;
      MGCHK(hipStreamBeginCapture(m->st, hipStreamCaptureModeThreadLocal));
      enqueue_vcycle(m);
      MGCHK(hipStreamEndCapture(m->st, &gr));
      hipError_t e = hipGraphInstantiate(&m->gexec, gr, nullptr, nullptr, 0);
      (void)hipGraphDestroy(gr);
      MGCHK(e);
    }
    MGCHK(hipGraphLaunch(m->gexec, m->st));
  } else {
    enqueue_vcycle(m);
    MGCHK(hipGetLastError());
  }
  return 0;
}

// the V-cycle loop on level-0 buffers already filled: `unchecked` cycles
// are enqueued behind the initial norms before the host first waits (each
// host check is a synchronisation), then the residual is checked after every
// cycle.  Returns 0, or AMRV_ENOTCONVERGED / AMRV_ENONPHYSICAL.
int run_cycles(amrv_mg* m, double tol, int max_cycles, int unchecked, int* cycles, double* res_out,
               double* f_out) {
  const int nf = m->g.nf;
  if (m->profile) unchecked = 0;  // profiling times each cycle on its own
  unchecked = std::max(0, std::min(unchecked, max_cycles));
  // the norms of the initial guess (max |f| is taken from these)
  if (m->g.nd == 2)
    enqueue_norms_nd<2>(m, 1);
  else
    enqueue_norms_nd<3>(m, 1);
  MGCHK(hipGetLastError());
  for (int i = 0; i < unchecked; i++)
    if (int rc = launch_cycle(m)) return rc;
  MGCHK(hipStreamSynchronize(m->st));
  double fmax[NFMAX] = {0, 0}, res[NFMAX] = {0, 0};
  auto fold = [&](int row, int nb) {
    unsigned long long v = 0;
    const unsigned long long* p = m->hpart + (size_t)row * m->g.maxb;
    for (int b = 0; b < nb; b++) v = p[b] > v ? p[b] : v;
    return bits_to_double(v);
  };
  for (int f = 0; f < nf; f++) fmax[f] = fold(NFMAX + f, m->nb_init);
  int nb = unchecked ? m->nb_cycle : m->nb_init;
  auto done = [&]() {
    bool ok = true;
    for (int f = 0; f < nf; f++) {
      res[f] = fold(f, nb);
      ok = ok && (res[f] <= tol * fmax[f]);
    }
    return ok;
  };
  int c = unchecked;
  bool ok = done();
  for (int f = 0; f < nf; f++)
    if (std::isnan(res[f]) || std::isnan(fmax[f])) {
      if (cycles) *cycles = c;
      return set_error(AMRV_ENONPHYSICAL, "NaN in the multigrid right-hand side, initial guess or residual");
    }
  while (!ok && c < max_cycles) {
    if (m->profile) MGCHK(hipEventRecord(m->e0, m->st));
    if (int rc = launch_cycle(m)) return rc;
    if (m->profile) MGCHK(hipEventRecord(m->e1, m->st));
    MGCHK(hipStreamSynchronize(m->st));
    if (m->profile) {
      float ms = 0.0f;
      MGCHK(hipEventElapsedTime(&ms, m->e0, m->e1));
      m->prof_ms += ms;
      m->prof_cycles++;
    }
    c++;
    nb = m->nb_cycle;
    ok = done();
    for (int f = 0; f < nf; f++)
      if (std::isnan(res[f])) {
        if (cycles) *cycles = c;
        return set_error(AMRV_ENONPHYSICAL, "NaN in the multigrid residual");
      }
  }
  if (cycles) *cycles = c;
  for (int f = 0; f < nf; f++) {
    if (res_out) res_out[f] = res[f];
    if (f_out) f_out[f] = fmax[f];
  }
  if (!ok) return set_error(AMRV_ENOTCONVERGED, "multigrid residual above tol after max_cycles V-cycles");
  return 0;
}

}  // namespace

namespace amrv {

int mg_correction_grids(amrv_mg* m, double** f, double** e, bool* split) {
  if (!m || !f || !e || !split) return set_error(AMRV_EINVAL, "null argument");
  *split = m->g.split0 != 0;
  *f = m->g.f[0][0];
  *e = m->g.phi[0][0];
  return 0;
}

int mg_enqueue_correction(amrv_mg* m, const double* f, double* out, double lambda, int cycles, bool e_zeroed) {
  if (!m || !f || !out) return set_error(AMRV_EINVAL, "null argument");
  if (m->g.nf != 1 || m->var) return set_error(AMRV_EINVAL, "a correction solve needs one field and the constant coefficient");
  if (!(lambda >= 0.0) || !std::isfinite(lambda)) return set_error(AMRV_EINVAL, "lambda must be non-negative and finite");
  if (m->g.split0 && (f != m->g.f[0][0] || out != m->g.phi[0][0]))
    return set_error(AMRV_EINVAL, "a correction on split arrays works in the solver's own");
  if (m->par_nf != 1 || m->par_lam0 != lambda)
    if (int rc = set_params(m, &lambda)) return rc;
  const size_t bytes = (size_t)m->g.cells[0] * sizeof(double);
  if (f != m->g.f[0][0]) MGCHK(hipMemcpyAsync(m->g.f[0][0], f, bytes, hipMemcpyDeviceToDevice, m->st));
  if (!e_zeroed) MGCHK(hipMemsetAsync(m->g.phi[0][0], 0, bytes, m->st));
  for (int c = 0; c < cycles; c++) enqueue_vcycle(m, false);  // no host check: no residual norms
  MGCHK(hipGetLastError());
  if (out != m->g.phi[0][0]) MGCHK(hipMemcpyAsync(out, m->g.phi[0][0], bytes, hipMemcpyDeviceToDevice, m->st));
  return 0;
}

}  // namespace amrv

extern "C" {

size_t amrv_mg_workspace_bytes(const amrv_mg_config* cfg) {
  if (validate(cfg)) return 0;
  return layout(cfg).total;
}

int amrv_mg_create(const amrv_mg_config* cfg, void* workspace, size_t bytes, void* stream, amrv_mg** out) {
  if (!out) return set_error(AMRV_EINVAL, "null argument");
  *out = nullptr;
  if (int rc = validate(cfg)) return rc;
  if (!workspace) return set_error(AMRV_EINVAL, "null workspace");
  if (reinterpret_cast<uintptr_t>(workspace) % ALIGN) return set_error(AMRV_EINVAL, "workspace must be 256-byte aligned");
  const MgLayout L = layout(cfg);
  if (bytes < L.total) return set_error(AMRV_ENOMEM, ("workspace too small: need " + std::to_string(L.total)).c_str());
  if (cfg->use_graph && !stream) return set_error(AMRV_EINVAL, "graph replay needs a stream other than the null stream");
  amrv_mg* m = new amrv_mg;
  m->cfg = *cfg;
  m->st = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(workspace);
  MgDev& g = m->g;
  g.nd = cfg->ndim;
  g.bc = cfg->bc;
  g.nlev = L.nlev;
  g.nf = cfg->nfields;
  for (int l = 0; l < L.nlev; l++) {
    g.n[l] = cfg->n >> l;
    long long c = 1;
    for (int d = 0; d < cfg->ndim; d++) c *= g.n[l];
    g.cells[l] = (int)c;
    g.lg[l] = 0;
    while ((1 << g.lg[l]) < g.n[l]) g.lg[l]++;
    for (int f = 0; f < cfg->nfields; f++) {
      g.phi[f][l] = reinterpret_cast<double*>(base + L.off_phi[f][l]);
      g.f[f][l] = reinterpret_cast<double*>(base + L.off_f[f][l]);
      g.phi2[f][l] = L.off_phi2[f][l] ? reinterpret_cast<double*>(base + L.off_phi2[f][l]) : nullptr;
    }
  }
  for (int i = 0; i < 4; i++) m->tmp[i] = reinterpret_cast<double*>(base + L.off_tmp[i]);
  for (int l = 0; l < L.nlev; l++) {
    m->eps[l] = reinterpret_cast<double*>(base + L.off_eps[l]);
    g.eps[l] = m->eps[l];
  }
  m->par = reinterpret_cast<double*>(base + L.off_par);
  g.par = m->par;
  for (int f = 0; f < NFMAX; f++) g.cmat[f] = g.cells[0] >= COARSE_CELLS * COARSE_CELLS ? m->tmp[2 + f] : nullptr;
  // the tail: the first level of at most TAIL_CELLS cells, and every level below
  int tail = 0;
  while (g.cells[tail] > TAIL_CELLS) tail++;
  m->tail = tail;
  g.split0 = g.nd == 3 && tail > 0;
  int off = 0;
  for (int l = tail; l < L.nlev; l++) {
    if (g.cells[l] > COARSE_CELLS) off += 2 * g.cells[l];
  }
  off += COARSE_CELLS + TAIL_THREADS;  // the matrix level's right-hand side and partial sums
  m->tail_lds = (size_t)off * sizeof(double);
  int offv = 0;
  for (int l = tail; l < L.nlev; l++) {
    g.loffv[l] = offv;
    offv += 3 * g.cells[l];
  }
  m->tail_lds_var = (size_t)offv * sizeof(double);
  auto lds_limit = [](const void* k, size_t bytes) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  };
  const bool d2 = cfg->ndim == 2, mat = g.cmat[0] != nullptr;
  hipError_t e = lds_limit(d2 ? (mat ? reinterpret_cast<const void*>(k_mg_tail<2, true>)
                                     : reinterpret_cast<const void*>(k_mg_tail<2, false>))
                              : (mat ? reinterpret_cast<const void*>(k_mg_tail<3, true>)
                                     : reinterpret_cast<const void*>(k_mg_tail<3, false>)),
                           m->tail_lds);
  if (e == hipSuccess)
    e = lds_limit(d2 ? reinterpret_cast<const void*>(k_mg_tail_var<2>) : reinterpret_cast<const void*>(k_mg_tail_var<3>),
                  m->tail_lds_var);
  m->nb_init = std::min(blocks_of(g.cells[0]), g.nd == 3 ? 1024 : 256);
  m->nb_cycle = tiled(m) ? (g.n[0] / TS) * (g.n[0] / TS) : m->nb_init;
  g.maxb = std::max(m->nb_init, m->nb_cycle);
  const size_t hbytes = (size_t)2 * NFMAX * g.maxb * sizeof(unsigned long long);
  if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&m->hpart), hbytes);
  if (e == hipSuccess) {
    std::memset(m->hpart, 0, hbytes);
    g.hpart = m->hpart;
  }
  if (e == hipSuccess) e = hipEventCreate(&m->e0);
  if (e == hipSuccess) e = hipEventCreate(&m->e1);
  if (e != hipSuccess) {
    int rc = hip_err(e, "amrv_mg_create");
    amrv_mg_destroy(m);
    return rc;
  }
  *out = m;
  return 0;
}

int amrv_mg_destroy(amrv_mg* m) {
  if (!m) return 0;
  if (m->st) (void)hipStreamSynchronize(m->st);
  if (m->gexec) (void)hipGraphExecDestroy(m->gexec);
  if (m->hpart) (void)hipHostFree(m->hpart);
  if (m->e0) (void)hipEventDestroy(m->e0);
  if (m->e1) (void)hipEventDestroy(m->e1);
  delete m;
  return 0;
}

int amrv_mg_solve(amrv_mg* m, const double* f, double* phi, const double* lambda, double tol, int32_t max_cycles,
                  int32_t* cycles, double* res_max, double* f_max) {
  if (!m || !f || !phi || !lambda) return set_error(AMRV_EINVAL, "null argument");
  if (!(tol > 0.0)) return set_error(AMRV_EINVAL, "tol must be positive");
  if (max_cycles < 0) return set_error(AMRV_EINVAL, "max_cycles must be >= 0");
  for (int i = 0; i < m->g.nf; i++)
    if (!(lambda[i] >= 0.0) || !std::isfinite(lambda[i]))
      return set_error(AMRV_EINVAL, "lambda must be non-negative and finite");
  for (int i = 0; i < m->g.nf; i++)
    if (m->var && !(lambda[i] > 0.0)) return set_error(AMRV_EINVAL, "a solve with a coefficient needs lambda > 0");
  if (int rc = set_params(m, lambda)) return rc;
  const size_t bytes = (size_t)m->g.cells[0] * sizeof(double);
  // a caller's field to or from level 0
  auto copy = [&](const double* src, double* dst, int to_level) -> int {
    if (m->g.split0) {
      hipLaunchKernelGGL(k_mg3_reorder, dim3(blocks_of(m->g.cells[0] >> 1)), dim3(256), 0, m->st, m->g.lg[0], src, dst,
                         to_level);
      MGCHK(hipGetLastError());
    } else {
      MGCHK(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, m->st));
    }
    return 0;
  };
  for (int i = 0; i < m->g.nf; i++) {
    if (int rc = copy(f + (size_t)i * m->g.cells[0], m->g.f[i][0], 1)) return rc;
    if (int rc = copy(phi + (size_t)i * m->g.cells[0], m->g.phi[i][0], 1)) return rc;
  }
  int c = 0;
  const int rc = run_cycles(m, tol, max_cycles, 0, &c, res_max, f_max);
  if (cycles) *cycles = c;
  for (int i = 0; i < m->g.nf; i++)
    if (int rc2 = copy(m->g.phi[i][0], phi + (size_t)i * m->g.cells[0], 0)) return rc2;
  MGCHK(hipStreamSynchronize(m->st));
  return rc;
}

int amrv_mg_divb_project(amrv_mg* m, double* bx, double* by, double* bz, double tol, int32_t max_cycles,
                         int32_t* cycles, double* div_before, double* div_after) {
  if (!m || !bx || !by || (m->g.nd == 3 && !bz)) return set_error(AMRV_EINVAL, "null argument");
  if (m->g.nf != 1) return set_error(AMRV_EINVAL, "the projection needs a solver created with nfields = 1");
  if (m->var) return set_error(AMRV_EINVAL, "the projection needs the constant coefficient");
  if (m->g.bc != AMRV_MG_PERIODIC) return set_error(AMRV_EINVAL, "the projection needs periodic faces");
  if (!(tol > 0.0) || max_cycles < 0) return set_error(AMRV_EINVAL, "bad tol or max_cycles");
  const double lam0 = 0.0;
  if (int rc = set_params(m, &lam0)) return rc;
  const MgDev& g = m->g;
  const double c = 0.5 * g.n[0] / m->cfg.length;
  const bool d2 = g.nd == 2;
  const int nb = blocks_of(g.cells[0]);
  double* b2 = d2 ? bx : bz;  // not read in 2D
  auto divmax = [&](double* out) -> int {
    hipLaunchKernelGGL(d2 ? k_mg_divnorm<2> : k_mg_divnorm<3>, dim3(m->nb_init), dim3(256), 0, m->st, g, bx, by, b2,
                       c);
    MGCHK(hipGetLastError());
    MGCHK(hipStreamSynchronize(m->st));
    unsigned long long v = 0;
    for (int b = 0; b < m->nb_init; b++) v = m->hpart[b] > v ? m->hpart[b] : v;
    if (out) *out = bits_to_double(v);
    return 0;
  };
  if (int rc = divmax(div_before)) return rc;
  hipLaunchKernelGGL(d2 ? k_mg_divb<2> : k_mg_divb<3>, dim3(nb), dim3(256), 0, m->st, g, bx, by, b2, c);
  MGCHK(hipGetLastError());
  int cyc = 0;
  const int rc = run_cycles(m, tol, max_cycles, 0, &cyc, nullptr, nullptr);
  if (cycles) *cycles = cyc;
  if (rc) return rc;
  hipLaunchKernelGGL(d2 ? k_mg_gradsub<2> : k_mg_gradsub<3>, dim3(nb), dim3(256), 0, m->st, g, bx, by, b2, c);
  MGCHK(hipGetLastError());
  return divmax(div_after);
}

int amrv_rd_step(amrv_mg* m, const amrv_rd_params* p, int32_t scheme, double dt, int32_t nsteps, double* u, double* v,
                 double tol, int32_t max_cycles, int32_t* cycles_total, double* res_max) {
  if (!m || !p || !u || !v) return set_error(AMRV_EINVAL, "null argument");
  if (p->model != AMRV_RD_SCHNAKENBERG && p->model != AMRV_RD_GRAY_SCOTT) return set_error(AMRV_EINVAL, "unknown model");
  if (!(p->Du > 0.0) || !(p->Dv > 0.0)) return set_error(AMRV_EINVAL, "diffusion coefficients must be positive");
  if (!(dt > 0.0) || !std::isfinite(dt)) return set_error(AMRV_EINVAL, "dt must be positive and finite");
  if (nsteps < 0) return set_error(AMRV_EINVAL, "nsteps must be >= 0");
  if (scheme < AMRV_RD_EULER || scheme > AMRV_RD_IMEX) return set_error(AMRV_EINVAL, "unknown scheme");
  if (m->var) return set_error(AMRV_EINVAL, "reaction-diffusion steps need the constant coefficient");
  const bool implicit = scheme == AMRV_RD_SPLIT || scheme == AMRV_RD_IMEX;
  if (implicit && m->g.nf != 2) return set_error(AMRV_EINVAL, "split and IMEX steps need a solver with nfields = 2");
  if (implicit && (!(tol > 0.0) || max_cycles < 0)) return set_error(AMRV_EINVAL, "bad tol or max_cycles");
  RdK k{p->model, p->Du, p->Dv, p->p1, p->p2, p->p3};
  const MgDev& g = m->g;
  const int nb = blocks_of(g.cells[0]);
  const size_t bytes = (size_t)g.cells[0] * sizeof(double);
  double lam[2] = {1.0, 1.0};
  if (scheme == AMRV_RD_SPLIT) {
    lam[0] = 1.0 / (dt * p->Du);
    lam[1] = 1.0 / (dt * p->Dv);
  } else if (scheme == AMRV_RD_IMEX) {
    lam[0] = 2.0 / (dt * p->Du);
    lam[1] = 2.0 / (dt * p->Dv);
  }
  if (int rc = set_params(m, lam, implicit)) return rc;
  int total = 0;
  const bool d2 = g.nd == 2;
  double *cu = u, *cv = v, *au = m->tmp[0], *av = m->tmp[1];  // explicit schemes: current and other buffer
  for (int s = 0; s < nsteps; s++) {
    if (scheme == AMRV_RD_EULER || scheme == AMRV_RD_MIDPOINT) {
      // the new state goes to the other buffer of the pair (the caller's
      // arrays and tmp[0..1] alternate); one copy at the end if needed
      if (scheme == AMRV_RD_EULER) {
        hipLaunchKernelGGL(d2 ? k_rd_explicit<2> : k_rd_explicit<3>, dim3(nb), dim3(256), 0, m->st, g, k, cu, cv, cu,
                           cv, au, av, dt);
      } else {
        double *hu = m->tmp[2], *hv = m->tmp[3];
        hipLaunchKernelGGL(d2 ? k_rd_explicit<2> : k_rd_explicit<3>, dim3(nb), dim3(256), 0, m->st, g, k, cu, cv, cu,
                           cv, hu, hv, 0.5 * dt);
        hipLaunchKernelGGL(d2 ? k_rd_explicit<2> : k_rd_explicit<3>, dim3(nb), dim3(256), 0, m->st, g, k, cu, cv, hu,
                           hv, au, av, dt);
      }
      MGCHK(hipGetLastError());
      std::swap(cu, au);
      std::swap(cv, av);
      if (s + 1 == nsteps && cu != u) {
        MGCHK(hipMemcpyAsync(u, cu, bytes, hipMemcpyDeviceToDevice, m->st));
        MGCHK(hipMemcpyAsync(v, cv, bytes, hipMemcpyDeviceToDevice, m->st));
      }
      continue;
    }
    if (scheme == AMRV_RD_SPLIT)
      hipLaunchKernelGGL(d2 ? k_rd_split_rhs<2> : k_rd_split_rhs<3>, dim3(nb), dim3(256), 0, m->st, g, k, u, v, dt);
    else
      hipLaunchKernelGGL(d2 ? k_rd_imex_rhs<2> : k_rd_imex_rhs<3>, dim3(nb), dim3(256), 0, m->st, g, k, u, v,
                         m->tmp[0], m->tmp[1], dt);
    MGCHK(hipGetLastError());
    int c = 0;
    // the previous solve's cycle count, less one, runs before the first check
    const int rc = run_cycles(m, tol, max_cycles, m->last_cycles - 1, &c, res_max, nullptr);
    m->last_cycles = c;
    total += c;
    if (rc) {
      if (cycles_total) *cycles_total = total;
      return rc;
    }
    if (scheme == AMRV_RD_SPLIT && g.split0) {
      hipLaunchKernelGGL(k_mg3_reorder, dim3(blocks_of(g.cells[0] >> 1)), dim3(256), 0, m->st, g.lg[0], g.phi[0][0], u,
                         0);
      hipLaunchKernelGGL(k_mg3_reorder, dim3(blocks_of(g.cells[0] >> 1)), dim3(256), 0, m->st, g.lg[0], g.phi[1][0], v,
                         0);
      MGCHK(hipGetLastError());
    } else if (scheme == AMRV_RD_SPLIT) {
      MGCHK(hipMemcpyAsync(u, g.phi[0][0], bytes, hipMemcpyDeviceToDevice, m->st));
      MGCHK(hipMemcpyAsync(v, g.phi[1][0], bytes, hipMemcpyDeviceToDevice, m->st));
    } else if (g.split0) {
      hipLaunchKernelGGL(k_rd3_imex_final, dim3(blocks_of(g.cells[0] >> 1)), dim3(256), 0, m->st, g, k, u, v,
                         m->tmp[0], m->tmp[1], dt);
      MGCHK(hipGetLastError());
    } else {
      hipLaunchKernelGGL(d2 ? k_rd_imex_final<2> : k_rd_imex_final<3>, dim3(nb), dim3(256), 0, m->st, g, k, u, v,
                         m->tmp[0], m->tmp[1], dt);
      MGCHK(hipGetLastError());
    }
  }
  if (cycles_total) *cycles_total = total;
  MGCHK(hipStreamSynchronize(m->st));
  return 0;
}

int amrv_mg_set_coefficient(amrv_mg* m, const double* eps) {
  if (!m) return set_error(AMRV_EINVAL, "null argument");
  if (m->gexec) {  // the captured cycle belongs to the other operator
    MGCHK(hipGraphExecDestroy(m->gexec));
    m->gexec = nullptr;
  }
  if (!eps) {
    m->var = false;
    m->g.split0 = m->g.nd == 3 && m->tail > 0;
    m->g.eps[0] = m->eps[0];
    return 0;
  }
  const MgDev& g = m->g;
  MGCHK(hipMemcpyAsync(m->eps[0], eps, (size_t)g.cells[0] * sizeof(double), hipMemcpyDeviceToDevice, m->st));
  for (int l = 0; l + 1 < g.nlev; l++) {
    if (g.nd == 2)
      hipLaunchKernelGGL(k_mg_eps_restrict<2>, dim3(blocks_of(g.cells[l + 1])), dim3(256), 0, m->st, g, l,
                         m->eps[l + 1]);
    else
      hipLaunchKernelGGL(k_mg_eps_restrict<3>, dim3(blocks_of(g.cells[l + 1])), dim3(256), 0, m->st, g, l,
                         m->eps[l + 1]);
    MGCHK(hipGetLastError());
  }
  MGCHK(hipStreamSynchronize(m->st));
  m->var = true;
  m->g.split0 = 0;  // the variable-coefficient kernels keep the natural order
  return 0;
}

int amrv_mg_profile(amrv_mg* m, int32_t enable) {
  if (!m) return set_error(AMRV_EINVAL, "null argument");
  m->profile = enable != 0;
  return 0;
}

int amrv_mg_profile_read(amrv_mg* m, double* ms_total, int64_t* cycles) {
  if (!m || !ms_total || !cycles) return set_error(AMRV_EINVAL, "null argument");
  *ms_total = m->prof_ms;
  *cycles = m->prof_cycles;
  m->prof_ms = 0.0;
  m->prof_cycles = 0;
  return 0;
}

}  // extern "C"

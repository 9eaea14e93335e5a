// mlp.hip -- learned refinement flagger on gfx950.
//
// The paper refines blocks where the Loehner estimator exceeds a tolerance
// (arXiv 2004.03275, Sec. 1.3).  This file adds a small multilayer perceptron
// (128-64-64-2) that predicts those decisions from pooled block features, so
// most blocks can be flagged without the estimator's ghost fill and
// second-derivative pass:
//   k_mlp_features  per leaf: means of rho and p over 64 sub-blocks (4^3 cells
//                   in 3D, 2^2 in 2D), normalised by the leaf mean, to bfloat16
//   k_mlp_infer     refine and coarsen logits of all leaves: bfloat16 MFMA
//                   products (v_mfma_f32_16x16x32_bf16), binary32 accumulation,
//                   and each leaf's three-way flag from its two logits
//   k_mlp_grad      a batch's forward pass, class-weighted binary cross-entropy
//                   and backward pass (weight gradients again as bfloat16 MFMA
//                   products with binary32 accumulation), partial gradients
//   k_mlp_step      their sum in a fixed order, Adam
// Reductions run in a fixed order, so results are deterministic.
#include <type_traits>

#include <mutex>

#include "bf16.hpp"
#include "internal.hpp"
#include "mlp.hpp"
#include "physics.hpp"

namespace amrv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// 8 consecutive bfloat16 values (16 bytes, 16-byte aligned) as an MFMA operand
__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
  bf16x8 r;
  __builtin_memcpy(&r, p, 16);
  return r;
}

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 r;
  const uint4 z = make_uint4(0, 0, 0, 0);
  __builtin_memcpy(&r, &z, 16);
  return r;
}

// Operand layout of v_mfma_f32_16x16x32_bf16 (64 lanes): lane l holds
// A[m = l % 16][k = 8 (l / 16) .. +7], B[k = 8 (l / 16) .. +7][n = l % 16], and
// receives D[m = 4 (l / 16) + i][n = l % 16], i = 0..3.
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// features
// ---------------------------------------------------------------------------

template <int ND, int PH>
__global__ void __launch_bounds__(128) k_mlp_features(Geo g, const double* __restrict__ U,
                                                      const double* __restrict__ pp, uint16_t* __restrict__ X) {
  using S = Sys<ND, PH>;
  constexpr int NV = S::NV;
  __shared__ double means[2][64];
  __shared__ double mtot[2];
  const int leaf = blockIdx.x;
  const int t = threadIdx.x;
  const int var = t >> 6, sb = t & 63;  // var 0: rho, 1: p
  PhysParams P;
  P.gamma = pp[PP_GAMMA];
  P.gm1 = pp[PP_GM1];
  P.igm1 = pp[PP_IGM1];
  P.ch = 0.0;
  P.cad = pp[PP_CAD];
  P.gcad = pp[PP_GCAD];
  const size_t vs = (size_t)g.n * g.ncell;
  const double* base = U + (size_t)leaf * g.ncell;
  double s = 0.0;
  if constexpr (ND == 3) {
    const int bx = sb & 3, by = (sb >> 2) & 3, bz = sb >> 4;
    for (int k = 0; k < 4; k++)
      for (int j = 0; j < 4; j++)
        for (int i = 0; i < 4; i++) {
          const int cell = (4 * bx + i) + 16 * ((4 * by + j) + 16 * (4 * bz + k));
          double q;
          if (var == 0) {
            q = base[cell];
          } else {
            double u[NV], v[NV];
#pragma unroll
            for (int c = 0; c < NV; c++) u[c] = base[c * vs + cell];
            cons2prim<ND, PH>(u, v, P);
            q = pressure<ND, PH>(v, P);
          }
          s = s + q;
        }
    means[var][sb] = s / 64.0;
  } else {
    const int bx = sb & 7, by = sb >> 3;
    for (int j = 0; j < 2; j++)
      for (int i = 0; i < 2; i++) {
        const int cell = (2 * bx + i) + 16 * (2 * by + j);
        double q;
        if (var == 0) {
          q = base[cell];
        } else {
          double u[NV], v[NV];
#pragma unroll
          for (int c = 0; c < NV; c++) u[c] = base[c * vs + cell];
          cons2prim<ND, PH>(u, v, P);
          q = pressure<ND, PH>(v, P);
        }
        s = s + q;
      }
    means[var][sb] = s / 4.0;
  }
  __syncthreads();
  if (sb == 0) {
    double m = 0.0;
    for (int i = 0; i < 64; i++) m = m + means[var][i];
    mtot[var] = m / 64.0;
  }
  __syncthreads();
  const float f = (float)(means[var][sb] / mtot[var] - 1.0);
  X[(size_t)leaf * MLP_NIN + 64 * var + sb] = to_bf16(f);
}

// ---------------------------------------------------------------------------
// parameters: binary32 master vector -> bfloat16 operand copies
// ---------------------------------------------------------------------------

// W1b [64][128], W2b [64][64], W2bT [64][64] (transposed), W3b [2][64]
__global__ void k_mlp_prep(const float* __restrict__ w, uint16_t* __restrict__ wb) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < MLP_NH * MLP_NIN; i += gridDim.x * blockDim.x)
    wb[MLP_WB_W1 + i] = to_bf16(w[MLP_W1 + i]);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < MLP_NH * MLP_NH; i += gridDim.x * blockDim.x) {
    const uint16_t b = to_bf16(w[MLP_W2 + i]);
    wb[MLP_WB_W2 + i] = b;
    const int n2 = i / MLP_NH, n1 = i % MLP_NH;  // W2[n2][n1]
    wb[MLP_WB_W2T + n1 * MLP_NH + n2] = b;
  }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < MLP_NOUT * MLP_NH; i += gridDim.x * blockDim.x)
    wb[MLP_WB_W3 + i] = to_bf16(w[MLP_W3 + i]);
}

// ---------------------------------------------------------------------------
// forward pass of one 16-row tile by one wave
// ---------------------------------------------------------------------------

// rows of X: xrow(r) -> pointer to 128 bfloat16 features, or nullptr (zeros)
// h1t, h2t: the wave's LDS tiles [16][64] bfloat16.  Returns, in lane l < 16,
// the refine logit of row l and, in lane 16 + l, the coarsen logit of row l
// (other lanes: undefined).
template <class XRow>
__device__ __forceinline__ float tile_forward(XRow xrow, const uint16_t* __restrict__ wb, const float* __restrict__ w,
                                              uint16_t* h1t, uint16_t* h2t) {
  const int l = threadIdx.x & 63;
  const int lm = l & 15, lk = 8 * (l >> 4);
  const uint16_t* xr = xrow(lm);
  bf16x8 xa[4];
#pragma unroll
  for (int kt = 0; kt < 4; kt++) xa[kt] = xr ? load8(xr + kt * 32 + lk) : zero8();
#pragma unroll
  for (int nt = 0; nt < 4; nt++) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
      acc = mfma(xa[kt], load8(wb + MLP_WB_W1 + (nt * 16 + lm) * MLP_NIN + kt * 32 + lk), acc);
    const int n = nt * 16 + lm;
    const float bias = w[MLP_B1 + n];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float a = acc[i] + bias;
      h1t[(4 * (l >> 4) + i) * MLP_NH + n] = to_bf16(a > 0.f ? a : 0.f);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int nt = 0; nt < 4; nt++) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
      acc = mfma(load8(h1t + lm * MLP_NH + kt * 32 + lk), load8(wb + MLP_WB_W2 + (nt * 16 + lm) * MLP_NH + kt * 32 + lk),
                 acc);
    const int n = nt * 16 + lm;
    const float bias = w[MLP_B2 + n];
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const float a = acc[i] + bias;
      h2t[(4 * (l >> 4) + i) * MLP_NH + n] = to_bf16(a > 0.f ? a : 0.f);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  float z = 0.f;
  if (l < 32) {
    const int o = l >> 4, r = l & 15;
    for (int k = 0; k < MLP_NH; k++)
      z = z + from_bf16(h2t[r * MLP_NH + k]) * from_bf16(wb[MLP_WB_W3 + o * MLP_NH + k]);
    z = z + w[MLP_B3 + o];
  }
  return z;
}

// logits of n rows of X [n][128] into z [n][2], and each leaf's flag from
// its logits (z_r, z_c): +1 where z_r > 0 below the finest level, -1 where
// z_r <= 0 and z_c > 0 above level 1, else 0; `uncertain` (optional) marks
// leaves with |z_r| < margin or |z_c| < margin (fallback mode), `zout`
// (optional) receives z_r.  256 threads = 4 waves x 16 rows.
__global__ void __launch_bounds__(256) k_mlp_infer(const uint16_t* __restrict__ X, int n, const uint16_t* __restrict__ wb,
                                                   const float* __restrict__ w, float* __restrict__ z,
                                                   const int32_t* __restrict__ lvl, int max_level, float margin,
                                                   int8_t* __restrict__ flags, int8_t* __restrict__ uncertain,
                                                   double* __restrict__ zout) {
  __shared__ __attribute__((aligned(16))) uint16_t h1[4][16 * MLP_NH];
  __shared__ __attribute__((aligned(16))) uint16_t h2[4][16 * MLP_NH];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int r0 = blockIdx.x * 64 + wave * 16;
  auto xrow = [&](int m) -> const uint16_t* { return r0 + m < n ? X + (size_t)(r0 + m) * MLP_NIN : nullptr; };
  const float zz = tile_forward(xrow, wb, w, h1[wave], h2[wave]);
  const int r = l & 15, o = l >> 4;
  const float zc = __shfl(zz, r + 16, 64);  // lane r (< 16) gets the coarsen logit of its row
  if (l < 32 && r0 + r < n) z[(size_t)(r0 + r) * MLP_NOUT + o] = zz;
  if (l < 16 && r0 + r < n) {
    const int i = r0 + r;
    const float zr = zz;
    const int lv = lvl[i];
    flags[i] = (zr > 0.f && lv < max_level) ? 1 : ((!(zr > 0.f) && zc > 0.f && lv > 1) ? -1 : 0);
    if (uncertain) uncertain[i] = (fabsf(zr) < margin || fabsf(zc) < margin) ? 1 : 0;
    if (zout) zout[i] = (double)zr;
  }
}

// ---------------------------------------------------------------------------
// training step: the batch's rows over many workgroups, then one update launch
// ---------------------------------------------------------------------------

// A step is two launches.  k_mlp_grad: each workgroup takes `rows` rows of the
// batch through the forward and backward pass with every activation in LDS
// and writes its own partial gradient (part[workgroup][NPARAM + 1], the last
// value its loss sum); k_mlp_step adds the partials in workgroup order and
// applies Adam, so the sums have a fixed order and the result is
// deterministic.  Bound by latency (0.03 GFLOP a batch of 1,024).  One
// workgroup per batch, its activations in global scratch, left 255 CUs idle:
// 1,060 us a batch of 1,024; 32 rows per workgroup (one K step of the
// 16x16x32 products, 32 workgroups) 13.2 us + 4.0 us.
constexpr int TR = 32;           // rows of a K step
constexpr int TS = TR + 8;       // LDS row stride of the [feature][row] arrays (16-byte multiples, spread over banks)
constexpr int HS = MLP_NH + 8;   // and of the [row][unit] arrays

// rows per workgroup: 32, or 64 where 32 would give more than 64 partials (the
// scratch then stays below that of a whole batch's activations)
constexpr int mlp_train_rows(int B) { return B <= 64 * TR ? TR : 2 * TR; }

__global__ void __launch_bounds__(256) k_mlp_grad(const uint16_t* __restrict__ X, const float* __restrict__ Y,
                                                  const int32_t* __restrict__ order, int n, int B, int batch, int rows,
                                                  const float* __restrict__ w, const uint16_t* __restrict__ wb,
                                                  TrainHyper hp, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint16_t xT[MLP_NIN * TS];
  __shared__ __attribute__((aligned(16))) uint16_t h1[TR * HS], h1T[MLP_NH * TS], h2[TR * HS];
  __shared__ __attribute__((aligned(16))) uint16_t dh2[TR * HS], dh2T[MLP_NH * TS], dh1T[MLP_NH * TS];
  __shared__ float dh1[TR * (MLP_NH + 1)];
  __shared__ float zs[TR][MLP_NOUT], dz[TR][MLP_NOUT], ls[TR];
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int lm = l & 15, lk = 8 * (l >> 4), lq = 4 * (l >> 4);
  const int b0 = batch * B;
  int nvalid = n - b0;
  if (nvalid > B) nvalid = B;
  const float Bv = (float)nvalid;
  const int rt = wave & 1, np = wave >> 1;  // forward: a 16-row tile and half of the output units per wave

  f32x4 g1[8], g2[4];  // dW1, dW2 tiles of this wave
#pragma unroll
  for (int i = 0; i < 8; i++) g1[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; i++) g2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gs = 0.f, gb1 = 0.f;  // W3 (threads 0..127), b3 (128, 129), loss (130), b2 (192..255); b1 (192..255)

  const int rend = min(B, (int)(blockIdx.x + 1) * rows);
  for (int r0 = blockIdx.x * rows; r0 < rend; r0 += TR) {
    // layer 1; the rows (zeros past the batch's last sample) also to xT
    {
      const int r = r0 + rt * 16 + lm;
      const uint16_t* xr = r < nvalid ? X + (size_t)order[b0 + r] * MLP_NIN : nullptr;
      bf16x8 xa[4];
#pragma unroll
      for (int kt = 0; kt < 4; kt++) xa[kt] = xr ? load8(xr + kt * 32 + lk) : zero8();
#pragma unroll
      for (int k2 = 0; k2 < 2; k2++) {
        uint16_t t[8];
        const bf16x8 v = np ? xa[2 + k2] : xa[k2];
        __builtin_memcpy(t, &v, 16);
#pragma unroll
        for (int j = 0; j < 8; j++) xT[((2 * np + k2) * 32 + lk + j) * TS + rt * 16 + lm] = t[j];
      }
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const int u = (2 * np + q) * 16 + lm;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; kt++) acc = mfma(xa[kt], load8(wb + MLP_WB_W1 + u * MLP_NIN + kt * 32 + lk), acc);
        const float bias = w[MLP_B1 + u];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const float a = acc[i] + bias;
          const uint16_t hb = to_bf16(a > 0.f ? a : 0.f);
          h1[(rt * 16 + lq + i) * HS + u] = hb;
          h1T[u * TS + rt * 16 + lq + i] = hb;
        }
      }
    }
    __syncthreads();
    // layer 2
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int u = (2 * np + q) * 16 + lm;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < 2; kt++)
        acc = mfma(load8(h1 + (rt * 16 + lm) * HS + kt * 32 + lk), load8(wb + MLP_WB_W2 + u * MLP_NH + kt * 32 + lk), acc);
      const float bias = w[MLP_B2 + u];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const float a = acc[i] + bias;
        h2[(rt * 16 + lq + i) * HS + u] = to_bf16(a > 0.f ? a : 0.f);
      }
    }
    __syncthreads();
    // logits, in unit order
    if (tid < TR * MLP_NOUT) {
      const int o = tid >> 5, r = tid & 31;
      float z = 0.f;
      for (int k = 0; k < MLP_NH; k++) z = z + from_bf16(h2[r * HS + k]) * from_bf16(wb[MLP_WB_W3 + o * MLP_NH + k]);
      zs[r][o] = z + w[MLP_B3 + o];
    }
    __syncthreads();
    // logit gradients and loss per row.  The label is Loehner's class (+1
    // refine, -1 coarsen, 0 keep): target 1 of the refine output for +1, of
    // the coarsen output for -1; each output's class-weighted binary
    // cross-entropy, summed
    if (tid < TR) {
      float d[MLP_NOUT] = {0.f, 0.f}, lr = 0.f;
      if (r0 + tid < nvalid) {
        const float lab = Y[order[b0 + r0 + tid]];
#pragma unroll
        for (int o = 0; o < MLP_NOUT; o++) {
          const float z = zs[tid][o];
          const float y = o == 0 ? (lab > 0.5f ? 1.f : 0.f) : (lab < -0.5f ? 1.f : 0.f);
          const float pw = o == 0 ? hp.pos_weight : hp.pos_weight_c;
          const float sg = 1.f / (1.f + expf(-z));
          d[o] = ((1.f - y) * sg - pw * y * (1.f - sg)) / Bv;
          // -(pw y log s + (1-y) log(1-s)) with log s = -softplus(-z)
          const float sp_neg = fmaxf(-z, 0.f) + log1pf(expf(-fabsf(z)));
          const float sp_pos = fmaxf(z, 0.f) + log1pf(expf(-fabsf(z)));
          lr = lr + (pw * y * sp_neg + (1.f - y) * sp_pos);
        }
      }
      dz[tid][0] = d[0];
      dz[tid][1] = d[1];
      ls[tid] = lr;
    }
    __syncthreads();
    // dh2 = (dz_r w3_r + dz_c w3_c) * [h2 > 0] (binary32, then bfloat16); the
    // W3, b3, b2 gradients and the loss
    auto dh2_of = [&](int r, int c, float wr, float wc) -> float {
      return from_bf16(h2[r * HS + c]) > 0.f ? dz[r][0] * wr + dz[r][1] * wc : 0.f;
    };
    {
      const int c = tid & 63, ra = 8 * wave;
      const float wr = from_bf16(wb[MLP_WB_W3 + c]), wc = from_bf16(wb[MLP_WB_W3 + MLP_NH + c]);
      uint16_t t[8];
#pragma unroll
      for (int j = 0; j < 8; j++) {
        t[j] = to_bf16(dh2_of(ra + j, c, wr, wc));
        dh2[(ra + j) * HS + c] = t[j];
      }
      __builtin_memcpy(&dh2T[c * TS + ra], t, 16);
      if (wave == 3) {
#pragma unroll 8
        for (int r = 0; r < TR; r++) gs = gs + dh2_of(r, c, wr, wc);
      }
    }
    if (tid < MLP_NOUT * MLP_NH) {
      const int o = tid / MLP_NH, c = tid % MLP_NH;
#pragma unroll 8
      for (int r = 0; r < TR; r++) gs = gs + dz[r][o] * from_bf16(h2[r * HS + c]);
    } else if (tid < MLP_NOUT * MLP_NH + MLP_NOUT) {
      for (int r = 0; r < TR; r++) gs = gs + dz[r][tid - MLP_NOUT * MLP_NH];
    } else if (tid == MLP_NOUT * MLP_NH + MLP_NOUT) {
      for (int r = 0; r < TR; r++) gs = gs + ls[r];
    }
    __syncthreads();
    // dh1 = dh2 W2 * [h1 > 0]: 8 tiles, two per wave
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int u = wave * 16 + lm;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < 2; kt++)
        acc = mfma(load8(dh2 + (j * 16 + lm) * HS + kt * 32 + lk), load8(wb + MLP_WB_W2T + u * MLP_NH + kt * 32 + lk), acc);
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = j * 16 + lq + i;
        const float d = from_bf16(h1[r * HS + u]) > 0.f ? acc[i] : 0.f;
        dh1[r * (MLP_NH + 1) + u] = d;
        dh1T[u * TS + r] = to_bf16(d);
      }
    }
    __syncthreads();
    // dW2 += dh2^T h1 (16 tiles), dW1 += dh1^T X (32 tiles), K = 32 rows; b1
#pragma unroll
    for (int j = 0; j < 4; j++)
      g2[j] = mfma(load8(dh2T + (j * 16 + lm) * TS + lk), load8(h1T + (wave * 16 + lm) * TS + lk), g2[j]);
#pragma unroll
    for (int j = 0; j < 8; j++)
      g1[j] = mfma(load8(dh1T + ((j >> 1) * 16 + lm) * TS + lk), load8(xT + ((2 * wave + (j & 1)) * 16 + lm) * TS + lk), g1[j]);
    if (wave == 3) {
#pragma unroll 8
      for (int r = 0; r < TR; r++) gb1 = gb1 + dh1[r * (MLP_NH + 1) + l];
    }
    __syncthreads();
  }
  float* p = part + (size_t)blockIdx.x * MLP_PART;
#pragma unroll
  for (int j = 0; j < 4; j++)
#pragma unroll
    for (int i = 0; i < 4; i++) p[MLP_W2 + (j * 16 + lq + i) * MLP_NH + wave * 16 + lm] = g2[j][i];
#pragma unroll
  for (int j = 0; j < 8; j++)
#pragma unroll
    for (int i = 0; i < 4; i++)
      p[MLP_W1 + ((j >> 1) * 16 + lq + i) * MLP_NIN + (2 * wave + (j & 1)) * 16 + lm] = g1[j][i];
  if (tid < MLP_NOUT * MLP_NH + MLP_NOUT + 1) p[MLP_W3 + tid] = gs;  // W3, b3, then the loss sum at NPARAM
  if (wave == 3) {
    p[MLP_B2 + l] = gs;
    p[MLP_B1 + l] = gb1;
  }
}

// one parameter per thread: the partial gradients added in workgroup order,
// Adam on the binary32 master weight, and its bfloat16 operand copies; the
// thread past the last parameter writes the batch's mean loss
__global__ void __launch_bounds__(256) k_mlp_step(const float* __restrict__ part, int nparts, int nvalid,
                                                  float* __restrict__ w, float* __restrict__ am, float* __restrict__ av,
                                                  uint16_t* __restrict__ wb, TrainHyper hp, float c1, float c2,
                                                  float* __restrict__ loss_out, float* __restrict__ grad_out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i > MLP_NPARAM) return;
  float gr = 0.f;
  int k = 0;
  for (; k + 8 <= nparts; k += 8) {
    float t[8];
#pragma unroll
    for (int j = 0; j < 8; j++) t[j] = part[(size_t)(k + j) * MLP_PART + i];
#pragma unroll
    for (int j = 0; j < 8; j++) gr = gr + t[j];
  }
  for (; k < nparts; k++) gr = gr + part[(size_t)k * MLP_PART + i];
  if (i == MLP_NPARAM) {
    if (loss_out) *loss_out = gr / (float)nvalid;
    return;
  }
  if (grad_out) grad_out[i] = gr;
  const float m = hp.beta1 * am[i] + (1.f - hp.beta1) * gr;
  const float v = hp.beta2 * av[i] + (1.f - hp.beta2) * gr * gr;
  am[i] = m;
  av[i] = v;
  const float wn = w[i] - hp.lr * (m / c1) / (sqrtf(v / c2) + hp.eps);
  w[i] = wn;
  const uint16_t b = to_bf16(wn);
  if (i < MLP_B1) {
    wb[MLP_WB_W1 + i] = b;
  } else if (i >= MLP_W2 && i < MLP_B2) {
    const int q = i - MLP_W2;
    wb[MLP_WB_W2 + q] = b;
    wb[MLP_WB_W2T + (q % MLP_NH) * MLP_NH + q / MLP_NH] = b;
  } else if (i >= MLP_W3 && i < MLP_B3) {
    wb[MLP_WB_W3 + i - MLP_W3] = b;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_mlp_features(const Geo& g, const LaunchCfg& c, const double* U, const double* physp, uint16_t* X,
                               hipStream_t st) {
  auto go = [&](auto nd) {
    constexpr int ND = decltype(nd)::value;
    if (c.phys == PH_MHD)
      hipLaunchKernelGGL((k_mlp_features<ND, PH_MHD>), dim3(g.n), dim3(128), 0, st, g, U, physp, X);
    else if (c.phys == PH_POLY)
      hipLaunchKernelGGL((k_mlp_features<ND, PH_POLY>), dim3(g.n), dim3(128), 0, st, g, U, physp, X);
    else
      hipLaunchKernelGGL((k_mlp_features<ND, PH_EULER>), dim3(g.n), dim3(128), 0, st, g, U, physp, X);
  };
  if (c.ndim == 2) {
    go(std::integral_constant<int, 2>{});
  } else if (c.ndim == 3) {
    go(std::integral_constant<int, 3>{});
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mlp_prep(const float* w, uint16_t* wb, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_prep, dim3(16), dim3(256), 0, st, w, wb);
  return hipGetLastError();
}

hipError_t launch_mlp_infer(const uint16_t* X, int n, const uint16_t* wb, const float* w, float* z, const int32_t* lvl,
                            int max_level, float margin, int8_t* flags, int8_t* uncertain, double* zout,
                            hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_infer, dim3((n + 63) / 64), dim3(256), 0, st, X, n, wb, w, z, lvl, max_level, margin, flags,
                     uncertain, zout);
  return hipGetLastError();
}

size_t mlp_train_scratch_bytes(int B) { return mlp_train_scratch_bytes_c(B); }

hipError_t launch_mlp_train(const uint16_t* X, const float* Y, const int32_t* order, int n, int B, int first_batch,
                            int nbatch, float* w, float* am, float* av, const TrainHyper& hp, int t0, void* ws,
                            float* loss_out, float* grad_out, hipStream_t st) {
  const int rows = mlp_train_rows(B), nparts = (B + rows - 1) / rows;
  uint16_t* wb = (uint16_t*)ws;
  float* part = (float*)((char*)ws + mlp_align256(2 * (size_t)MLP_WB_COUNT));
  hipLaunchKernelGGL(k_mlp_prep, dim3(16), dim3(256), 0, st, w, wb);
  for (int b = first_batch; b < first_batch + nbatch; b++) {
    const int t = t0 + (b - first_batch) + 1;
    const float c1 = (float)(1.0 - pow((double)hp.beta1, (double)t));
    const float c2 = (float)(1.0 - pow((double)hp.beta2, (double)t));
    const int nvalid = n - b * B < B ? n - b * B : B;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nparts), dim3(256), 0, st, X, Y, order, n, B, b, rows, w, wb, hp, part);
    hipLaunchKernelGGL(k_mlp_step, dim3(MLP_NPARAM / 256 + 1), dim3(256), 0, st, part, nparts, nvalid, w, am, av, wb, hp,
                       c1, c2, loss_out ? loss_out + b : nullptr, b + 1 == first_batch + nbatch ? grad_out : nullptr);
  }
  return hipGetLastError();
}

// Training scratch held by the library for callers that cannot allocate
// (amrv_mlp_train_noalloc): room for the largest batch, one copy per device
// for the life of the process.  Host code never passes the array's name to a
// kernel: it resolves each device's address with hipGetSymbolAddress once,
// with that device current, and uses that address only.
static __device__ __align__(256) char scratch[MLP_STATIC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[MLP_MAX_DEVICES] = {};
}  // namespace

hipError_t mlp_static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MLP_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace amrv

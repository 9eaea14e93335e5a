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
//   k_mlp_rows      a batch's forward pass, class-weighted binary cross-entropy
//                   and backward pass
//   k_mlp_update    its gradients (weight gradients again as bfloat16 MFMA
//                   products with binary32 accumulation) and Adam
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

// 8 consecutive bfloat16 values as an MFMA operand (copied: a caller's rows need only a bfloat16's alignment)
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

// A step is two launches.  k_mlp_rows: each workgroup takes 32 rows of the
// batch (one K step of the 16x16x32 products) through the forward and backward
// pass with every activation in LDS and writes what the gradients are made of;
// k_mlp_update: a wave per 16x16 tile of dW1 and dW2, and per 16 parameters of
// the rest, runs over all rows of the batch in row order and applies Adam to
// its own parameters.  Every gradient is one chain over the rows: a sum of the
// workgroups' partial sums is as exact, but bfloat16 roundings of the weights
// carry a last-place difference to 3% of a weight within an epoch of small
// batches.  Bound by latency (0.03 GFLOP a batch of 1,024).  One workgroup per
// batch took 1,060 us a batch of 1,024; now 9.5 + 11.2 us.
constexpr int TR = 32;           // rows of a K step
constexpr int TS = TR + 8;       // LDS row stride of the [feature][row] arrays (16-byte multiples, spread over banks)
constexpr int HS = MLP_NH + 8;   // and of the [row][unit] arrays

// what k_mlp_rows leaves for k_mlp_update (mlp_train_scratch_bytes_c)
struct TrainScratch {
  uint16_t *xT, *h1T, *dh2T, *dh1T;  // [feature or unit][B]
  uint16_t* h2;                      // [B][64]
  float *dh2, *dh1;                  // [B][64], before their rounding
  float *dz, *loss;                  // [B][2], [B]
};

__global__ void __launch_bounds__(256) k_mlp_rows(const uint16_t* __restrict__ X, const float* __restrict__ Y,
                                                  const int32_t* __restrict__ order, int n, int B, int batch,
                                                  const float* __restrict__ w, const uint16_t* __restrict__ wb,
                                                  TrainHyper hp, TrainScratch s) {
  __shared__ __attribute__((aligned(16))) uint16_t xT[MLP_NIN * TS];
  __shared__ __attribute__((aligned(16))) uint16_t h1[TR * HS], h1T[MLP_NH * TS], h2[TR * HS];
  __shared__ __attribute__((aligned(16))) uint16_t dh2[TR * HS], dh2T[MLP_NH * TS], dh1T[MLP_NH * TS];
  __shared__ float dh1[TR * (MLP_NH + 1)];
  __shared__ float zs[TR][MLP_NOUT], dz[TR][MLP_NOUT];
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int lm = l & 15, lk = 8 * (l >> 4), lq = 4 * (l >> 4);
  const int b0 = batch * B;
  int nvalid = n - b0;
  if (nvalid > B) nvalid = B;
  const float Bv = (float)nvalid;
  const int rt = wave & 1, np = wave >> 1;  // forward: a 16-row tile and half of the output units per wave

  const int r0 = blockIdx.x * TR;
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
    s.dz[(size_t)(r0 + tid) * MLP_NOUT] = d[0];
    s.dz[(size_t)(r0 + tid) * MLP_NOUT + 1] = d[1];
    s.loss[r0 + tid] = lr;
  }
  __syncthreads();
  // dh2 = (dz_r w3_r + dz_c w3_c) * [h2 > 0] (binary32, then bfloat16)
  auto dh2_of = [&](int r, int c, float wr, float wc) -> float {
    return from_bf16(h2[r * HS + c]) > 0.f ? dz[r][0] * wr + dz[r][1] * wc : 0.f;
  };
  {
    const int c = tid & 63, ra = 8 * wave;
    const float wr = from_bf16(wb[MLP_WB_W3 + c]), wc = from_bf16(wb[MLP_WB_W3 + MLP_NH + c]);
    uint16_t t[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
      const float d = dh2_of(ra + j, c, wr, wc);
      s.dh2[(size_t)(r0 + ra + j) * MLP_NH + c] = d;
      t[j] = to_bf16(d);
      dh2[(ra + j) * HS + c] = t[j];
    }
    __builtin_memcpy(&dh2T[c * TS + ra], t, 16);
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
  // the transposed operands and the rows' values to memory, 16 bytes a thread
  auto put = [&](uint16_t* to, const uint16_t* from) { __builtin_memcpy(to, from, 16); };
  for (int i = tid; i < MLP_NIN * TR / 8; i += 256)
    put(s.xT + (size_t)(i >> 2) * B + r0 + 8 * (i & 3), xT + (i >> 2) * TS + 8 * (i & 3));
  const int u = tid >> 2, q = 8 * (tid & 3);
  put(s.h1T + (size_t)u * B + r0 + q, h1T + u * TS + q);
  put(s.dh2T + (size_t)u * B + r0 + q, dh2T + u * TS + q);
  put(s.dh1T + (size_t)u * B + r0 + q, dh1T + u * TS + q);
  put(s.h2 + (size_t)(r0 + (tid >> 3)) * MLP_NH + 8 * (tid & 7), h2 + (tid >> 3) * HS + 8 * (tid & 7));
  for (int i = tid; i < TR * MLP_NH; i += 256)
    s.dh1[(size_t)r0 * MLP_NH + i] = dh1[(i >> 6) * (MLP_NH + 1) + (i & 63)];
}

// Workgroups 0..11: the 32 + 16 tiles of dW1 = dh1^T X and dW2 = dh2^T h1, one
// per wave; 12..15 b1, 16..19 b2, 20..27 W3, 28 b3 and the loss: 16 sums each,
// their terms staged in LDS (1,024 rows at a time), one lane a sum.  Then Adam
// on the binary32 master weights and their bfloat16 operand copies.
constexpr int UPD_WGS = 29, UPD_ROWS = 1024;

__global__ void __launch_bounds__(256) k_mlp_update(TrainScratch s, int B, int nvalid, float* __restrict__ w,
                                                    float* __restrict__ am, float* __restrict__ av,
                                                    uint16_t* __restrict__ wb, TrainHyper hp, float c1, float c2,
                                                    float* __restrict__ loss_out, float* __restrict__ grad_out) {
  __shared__ __attribute__((aligned(16))) float term[UPD_ROWS * 16];
  const int tid = threadIdx.x, l = tid & 63, lm = l & 15, lk = 8 * (l >> 4);
  const int b = blockIdx.x;
  auto adam = [&](int i, float gr) {
    if (grad_out) grad_out[i] = gr;
    const float m = hp.beta1 * am[i] + (1.f - hp.beta1) * gr;
    const float v = hp.beta2 * av[i] + (1.f - hp.beta2) * gr * gr;
    am[i] = m;
    av[i] = v;
    const float wn = w[i] - hp.lr * (m / c1) / (sqrtf(v / c2) + hp.eps);
    w[i] = wn;
    const uint16_t h = to_bf16(wn);
    if (i < MLP_B1) {
      wb[MLP_WB_W1 + i] = h;
    } else if (i >= MLP_W2 && i < MLP_B2) {
      const int q = i - MLP_W2;
      wb[MLP_WB_W2 + q] = h;
      wb[MLP_WB_W2T + (q % MLP_NH) * MLP_NH + q / MLP_NH] = h;
    } else if (i >= MLP_W3 && i < MLP_B3) {
      wb[MLP_WB_W3 + i - MLP_W3] = h;
    }
  };
  if (b < 12) {
    const int tile = 4 * b + (tid >> 6);
    const bool one = tile < 32;
    const int mt = one ? tile >> 3 : (tile - 32) >> 2, nt = one ? tile & 7 : tile & 3;
    const uint16_t* pa = (one ? s.dh1T : s.dh2T) + (size_t)(mt * 16 + lm) * B + lk;
    const uint16_t* pb = (one ? s.xT : s.h1T) + (size_t)(nt * 16 + lm) * B + lk;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 8 * TR <= B; k += 8 * TR) {
      bf16x8 ra[8], rb[8];
#pragma unroll
      for (int j = 0; j < 8; j++) {
        ra[j] = load8(pa + k + j * TR);
        rb[j] = load8(pb + k + j * TR);
      }
#pragma unroll
      for (int j = 0; j < 8; j++) acc = mfma(ra[j], rb[j], acc);
    }
    for (; k < B; k += TR) acc = mfma(load8(pa + k), load8(pb + k), acc);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int row = mt * 16 + 4 * (l >> 4) + i, col = nt * 16 + lm;
      adam(one ? MLP_W1 + row * MLP_NIN + col : MLP_W2 + row * MLP_NH + col, acc[i]);
    }
    return;
  }
  const int c0 = 16 * ((b - 12) & 3), o = b >= 24 ? 1 : 0;  // columns; W3's output
  float g = 0.f;
  for (int r0 = 0; r0 < B; r0 += UPD_ROWS) {
    const int rows = min(UPD_ROWS, B - r0);
    // eight loads a thread in flight
    if (b < 20) {
      const float* src = (b < 16 ? s.dh1 : s.dh2) + (size_t)r0 * MLP_NH + c0;
      for (int i0 = 0; i0 < rows * 4; i0 += 8 * 256) {
        float4 t[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int i = min(i0 + j * 256 + tid, rows * 4 - 1);
          t[j] = *reinterpret_cast<const float4*>(src + (size_t)(i >> 2) * MLP_NH + 4 * (i & 3));
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
          *reinterpret_cast<float4*>(term + 4 * min(i0 + j * 256 + tid, rows * 4 - 1)) = t[j];
      }
    } else if (b < 28) {
      const uint16_t* src = s.h2 + (size_t)r0 * MLP_NH + c0;
      for (int i0 = 0; i0 < rows * 2; i0 += 8 * 256) {
        uint16_t t[8][8];
        float d[8];
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int i = min(i0 + j * 256 + tid, rows * 2 - 1);
          __builtin_memcpy(t[j], src + (size_t)(i >> 1) * MLP_NH + 8 * (i & 1), 16);
          d[j] = s.dz[(size_t)(r0 + (i >> 1)) * MLP_NOUT + o];
        }
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int i = min(i0 + j * 256 + tid, rows * 2 - 1);
#pragma unroll
          for (int q = 0; q < 8; q++) term[8 * i + q] = d[j] * from_bf16(t[j][q]);
        }
      }
    } else {
      for (int r = tid; r < rows; r += 256) {
        term[16 * r] = s.dz[(size_t)(r0 + r) * MLP_NOUT];
        term[16 * r + 1] = s.dz[(size_t)(r0 + r) * MLP_NOUT + 1];
        term[16 * r + 2] = s.loss[r0 + r];
      }
    }
    __syncthreads();
    if (tid < 16) {  // rows is a multiple of 32
      for (int r = 0; r < rows; r += 32) {
        float t[32];
#pragma unroll
        for (int j = 0; j < 32; j++) t[j] = term[16 * (r + j) + tid];
#pragma unroll
        for (int j = 0; j < 32; j++) g = g + t[j];
      }
    }
    __syncthreads();
  }
  if (tid >= 16) return;
  if (b < 28) {
    adam((b < 16 ? MLP_B1 : b < 20 ? MLP_B2 : MLP_W3 + o * MLP_NH) + c0 + tid, g);
  } else if (tid < MLP_NOUT) {
    adam(MLP_B3 + tid, g);
  } else if (tid == MLP_NOUT && loss_out) {
    *loss_out = g / (float)nvalid;
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
  char* at = (char*)ws;
  auto take = [&](size_t bytes) {
    void* p = at;
    at += mlp_align256(bytes);
    return p;
  };
  uint16_t* wb = (uint16_t*)take(2 * (size_t)MLP_WB_COUNT);
  const size_t n2 = 2 * (size_t)MLP_NH * B, n4 = 4 * (size_t)MLP_NH * B;
  TrainScratch s;
  s.xT = (uint16_t*)take(2 * (size_t)MLP_NIN * B);
  s.h1T = (uint16_t*)take(n2);
  s.dh2T = (uint16_t*)take(n2);
  s.dh1T = (uint16_t*)take(n2);
  s.h2 = (uint16_t*)take(n2);
  s.dh2 = (float*)take(n4);
  s.dh1 = (float*)take(n4);
  s.dz = (float*)take(4 * (size_t)MLP_NOUT * B);
  s.loss = (float*)take(4 * (size_t)B);
  hipLaunchKernelGGL(k_mlp_prep, dim3(16), dim3(256), 0, st, w, wb);
  for (int b = first_batch; b < first_batch + nbatch; b++) {
    const int t = t0 + (b - first_batch) + 1;
    const float c1 = (float)(1.0 - pow((double)hp.beta1, (double)t));
    const float c2 = (float)(1.0 - pow((double)hp.beta2, (double)t));
    const int nvalid = n - b * B < B ? n - b * B : B;
    hipLaunchKernelGGL(k_mlp_rows, dim3(B / TR), dim3(256), 0, st, X, Y, order, n, B, b, w, wb, hp, s);
    hipLaunchKernelGGL(k_mlp_update, dim3(UPD_WGS), dim3(256), 0, st, s, B, nvalid, w, am, av, wb, hp, c1, c2,
                       loss_out ? loss_out + b : nullptr, b + 1 == first_batch + nbatch ? grad_out : nullptr);
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

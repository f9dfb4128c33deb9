// The proposal network of the stochastic steps: a width-64 tanh MLP in FP32 (forward, backward), the
// variance objective over groups of its logits, and Adam.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "lsx_block.h"
#include "lsx_internal.h"

namespace lsx {

// ---------------------------------------------------------------- proposal network
// Flat FP32 parameters: W1 [nin][64], b1 [64], W2 [64][64], b2 [64], w3 [64], b3.
// z = w3 . tanh(W2^T tanh(W1^T x + b1) + b2) + b3.
constexpr int MLP_H = 64;
constexpr int MLP_NIN_MAX = 8;

struct MlpOff {
  int W1, b1, W2, b2, w3, b3, n;
  __host__ __device__ explicit MlpOff(int nin) {
    W1 = 0;
    b1 = nin * MLP_H;
    W2 = b1 + MLP_H;
    b2 = W2 + MLP_H * MLP_H;
    w3 = b2 + MLP_H;
    b3 = w3 + MLP_H;
    n = b3 + 1;
  }
};

int mlp_nparams(int nin) { return MlpOff(nin).n; }

__device__ __forceinline__ void mlp_stage(const float* theta, int n, float* sp) {
  for (int k = threadIdx.x; k < n; k += blockDim.x) sp[k] = theta[k];
}

__device__ __forceinline__ void mlp_load_row(const float* X, int64_t M, int nin, int64_t m, float (&x)[MLP_NIN_MAX]) {
#pragma unroll
  for (int i = 0; i < MLP_NIN_MAX; ++i) x[i] = (m < M && i < nin) ? X[m * nin + i] : 0.f;
}

// The hidden-layer products are dense contractions over 64 units: H1 (rows x 64) W2, and in the
// backward pass D2 W2^T and H1^T D2.  Each wave takes chunks of 16 rows and forms them on the
// matrix cores with v_mfma_f32_16x16x4f32 (FP32 operands and accumulation, the network's own
// precision); the first layer (nin inputs), the tanh and the output layer stay on the VALU.
// The VALU bounds both passes (a third of it the tanh), with the matrix cores busy 28 % (forward) and
// 44 %: the input count is compiled in, the tanh has no branches (a build option of this file), and a
// chunk's inputs are loaded while the one before is worked on, so that a chunk is two or three blocks of
// straight code.  1.14e6 rows of 5 inputs: forward 262 to 221 us, backward 540 to 438.
// Operand layouts of the instruction: A (16 x 4): lane l holds A[l % 16][l / 16]; B (4 x 16):
// lane l holds B[l / 16][l % 16]; C (16 x 16): element r of lane l is C[4 (l / 16) + r][l % 16].
typedef float mlp_v4f __attribute__((ext_vector_type(4)));
constexpr int MLP_CH = 16;    // rows per wave chunk
constexpr int MLP_LDT = 68;   // LDS row stride of a chunk's 64-wide tiles (floats)
constexpr int MLP_WTILE = 2 * MLP_CH * MLP_LDT + MLP_CH * MLP_NIN_MAX;  // per-wave LDS (H1, D, X)
// LDS row stride of the backward pass's copy of W2, read both along its rows (lane 16 lk + li at row
// lk, column li) and across them (row li, column lk): 84 = 64 + 20 floats put the 64 lanes of the
// second pattern on 64 different banks and the first on at most two per bank, where a stride of 64
// gave 16 and 4 lanes per bank (backward pass over 1.14e6 rows: 680 to 545 us)
constexpr int MLP_LDW = 84;

// W2 in the B layout: w2[kk][ct] = W2[4 kk + lk][16 ct + li]
__device__ __forceinline__ void mlp_w2_frag(const float* sp, const MlpOff& o, int li, int lk, float (&w2)[16][4]) {
#pragma unroll
  for (int kk = 0; kk < 16; ++kk)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) w2[kk][ct] = sp[o.W2 + (4 * kk + lk) * MLP_H + 16 * ct + li];
}

// H1[li][4 kk + lk] for kk = 0..15 (the A layout of the layer-2 product), fed straight into it:
// acc[ct] = pre-activation of layer 2, rows 4 lk + r, units 16 ct + li.  H1 (may be null) gets
// the chunk's first-layer activations at [row][unit].  W2 operands from registers (w2, REG) or
// from the staged parameters in LDS.
template <bool REG>
__device__ __forceinline__ void mlp_hidden(const float* sp, const MlpOff& o, int nin, const float (&x)[MLP_NIN_MAX],
                                           int li, int lk, const float (*w2)[4], const float* W2, mlp_v4f (&acc)[4],
                                           float* H1) {
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = (mlp_v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) {
    const int j = 4 * kk + lk;
    float a = sp[o.b1 + j];
#pragma unroll
    for (int i = 0; i < MLP_NIN_MAX; ++i)
      if (i < nin) a += x[i] * sp[o.W1 + i * MLP_H + j];
    const float h = tanhf(a);
    if (H1) H1[li * MLP_LDT + j] = h;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const float b = REG ? w2[kk][ct] : W2[(4 * kk + lk) * MLP_LDW + 16 * ct + li];
      acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(h, b, acc[ct], 0, 0, 0);
    }
  }
}

template <int NIN>
__global__ LSX_MFMA_BOUNDS(256, true) void k_mlp_fwd(const float* theta, int nin_, const float* X, int64_t M, float* z) {
  extern __shared__ float sp[];
  const int nin = NIN > 0 ? NIN : nin_;
  const MlpOff o(nin);
  mlp_stage(theta, o.n, sp);
  __syncthreads();
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
  float w2[16][4], b2[4], w3[4];
  mlp_w2_frag(sp, o, li, lk, w2);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    b2[ct] = sp[o.b2 + 16 * ct + li];
    w3[ct] = sp[o.w3 + 16 * ct + li];
  }
  const float b3 = sp[o.b3];
  const int64_t nch = (M + MLP_CH - 1) / MLP_CH;
  float nx[MLP_NIN_MAX];  // the next chunk's inputs
  mlp_load_row(X, M, nin, ((int64_t)blockIdx.x * 4 + wave) * MLP_CH + li, nx);
  for (int64_t c = (int64_t)blockIdx.x * 4 + wave; c < nch; c += (int64_t)gridDim.x * 4) {
    float x[MLP_NIN_MAX];
#pragma unroll
    for (int i = 0; i < MLP_NIN_MAX; ++i) x[i] = nx[i];
    mlp_load_row(X, M, nin, (c + (int64_t)gridDim.x * 4) * MLP_CH + li, nx);
    mlp_v4f acc[4];
    mlp_hidden<true>(sp, o, nin, x, li, lk, w2, nullptr, acc, nullptr);
    float zr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      zr[r] = 0.f;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) zr[r] += tanhf(acc[ct][r] + b2[ct]) * w3[ct];
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) zr[r] += __shfl_xor(zr[r], off);
    }
    if (li == 0)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = c * MLP_CH + 4 * lk + r;
        if (m < M) z[m] = zr[r] + b3;
      }
  }
}

// Backward of sum_m g_m z_m, g_m = dz[m] * (*gscale when set):
//   d2 = g w3 (1 - h2^2),  d1 = (d2 W2^T)(1 - h1^2),
//   grad W2 = H1^T d2 (matrix cores, accumulated in registers over the wave's chunks),
//   grad W1 = X^T d1, b1, b2, w3, b3: sums over rows.
// Each wave stages its chunk's H1, d2 (then d1) and inputs in its own LDS tiles; the waves'
// sums are added in wave order at the end and the workgroup writes partial[blockIdx.x][:].
template <int NIN>
__global__ LSX_MFMA_BOUNDS(256, true) void k_mlp_bwd(const float* theta, int nin_, const float* X, int64_t M,
                                                 const float* dz, const double* gscale, float* partial) {
  extern __shared__ float sp[];
  const int nin = NIN > 0 ? NIN : nin_;
  const MlpOff o(nin);
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
  float* W2 = sp + ((o.n + 3) & ~3);
  float* H1 = W2 + MLP_H * MLP_LDW + wave * MLP_WTILE;
  float* D = H1 + MLP_CH * MLP_LDT;
  float* XS = D + MLP_CH * MLP_LDT;
  mlp_stage(theta, o.n, sp);
  for (int e = threadIdx.x; e < MLP_H * MLP_H; e += 256) W2[(e >> 6) * MLP_LDW + (e & 63)] = theta[o.W2 + e];
  __syncthreads();
  const float gs = gscale ? (float)*gscale : 1.f;
  float b2[4], w3[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    b2[ct] = sp[o.b2 + 16 * ct + li];
    w3[ct] = sp[o.w3 + 16 * ct + li];
  }
  mlp_v4f gW2[4][4];  // [jt][kt]: grad W2[16 jt + 4 lk + r][16 kt + li]
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) gW2[jt][kt] = (mlp_v4f){0.f, 0.f, 0.f, 0.f};
  float gb2[4] = {0.f, 0.f, 0.f, 0.f}, gw3[4] = {0.f, 0.f, 0.f, 0.f};  // units 16 ct + li, rows 4 lk + r
  float gW1[MLP_NIN_MAX], gb1 = 0.f, gb3 = 0.f;                          // unit = lane
#pragma unroll
  for (int i = 0; i < MLP_NIN_MAX; ++i) gW1[i] = 0.f;
  const int64_t nch = (M + MLP_CH - 1) / MLP_CH;
  // the next chunk's inputs and dz
  float nx[MLP_NIN_MAX], ng[4];
  auto load = [&](int64_t c) {
    mlp_load_row(X, M, nin, c * MLP_CH + li, nx);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = c * MLP_CH + 4 * lk + r;
      ng[r] = m < M ? dz[m] : 0.f;
    }
  };
  load((int64_t)blockIdx.x * 4 + wave);
  for (int64_t c = (int64_t)blockIdx.x * 4 + wave; c < nch; c += (int64_t)gridDim.x * 4) {
    float x[MLP_NIN_MAX], g[4];
#pragma unroll
    for (int i = 0; i < MLP_NIN_MAX; ++i) x[i] = nx[i];
#pragma unroll
    for (int r = 0; r < 4; ++r) g[r] = ng[r] * gs;
    load(c + (int64_t)gridDim.x * 4);
    if (lk == 0)
#pragma unroll
      for (int i = 0; i < MLP_NIN_MAX; ++i) XS[li * MLP_NIN_MAX + i] = x[i];
    mlp_v4f acc[4];
    mlp_hidden<false>(sp, o, nin, x, li, lk, nullptr, W2, acc, H1);
    if (li == 0) gb3 += (g[0] + g[1]) + (g[2] + g[3]);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float h2 = tanhf(acc[ct][r] + b2[ct]);
        const float d2 = g[r] * w3[ct] * (1.f - h2 * h2);
        D[(4 * lk + r) * MLP_LDT + 16 * ct + li] = d2;
        gb2[ct] += d2;
        gw3[ct] += g[r] * h2;
      }
    // the chunk's tiles are written by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // grad W2 += H1^T d2 (k-steps over the chunk's rows)
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const int row = 4 * s4 + lk;
      float a[4], b[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[t] = H1[row * MLP_LDT + 16 * t + li];
        b[t] = D[row * MLP_LDT + 16 * t + li];
      }
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
          gW2[jt][kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[jt], b[kt], gW2[jt][kt], 0, 0, 0);
    }
    // e = d2 W2^T: rows 4 lk + r, units 16 jt + li
    mlp_v4f e[4];
#pragma unroll
    for (int jt = 0; jt < 4; ++jt) e[jt] = (mlp_v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const float a = D[li * MLP_LDT + 4 * kk + lk];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
        e[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, W2[(16 * jt + li) * MLP_LDW + 4 * kk + lk], e[jt], 0, 0, 0);
    }
    // d1 = e (1 - h1^2), written over d2 (every lane has read its d2 operands above)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 4 * lk + r, j = 16 * jt + li;
        const float h = H1[row * MLP_LDT + j];
        D[row * MLP_LDT + j] = e[jt][r] * (1.f - h * h);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // grad W1, b1 for unit j = lane over the chunk's rows
#pragma unroll 4
    for (int row = 0; row < MLP_CH; ++row) {
      const float d1 = D[row * MLP_LDT + lane];
      gb1 += d1;
#pragma unroll
      for (int i = 0; i < MLP_NIN_MAX; ++i)
        if (i < nin) gW1[i] += XS[row * MLP_NIN_MAX + i] * d1;
    }
    // the tiles are rewritten by the next chunk
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // sums over the lane groups lk (rows) of the unit-per-lane-group terms
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    gb2[ct] += __shfl_xor(gb2[ct], 16);
    gb2[ct] += __shfl_xor(gb2[ct], 32);
    gw3[ct] += __shfl_xor(gw3[ct], 16);
    gw3[ct] += __shfl_xor(gw3[ct], 32);
  }
  gb3 += __shfl_xor(gb3, 16);
  gb3 += __shfl_xor(gb3, 32);
  // the waves' sums, added in wave order into sp (theta is no longer needed)
  __syncthreads();
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
      auto put = [&](int idx, float v) { sp[idx] = (w == 0) ? v : sp[idx] + v; };
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) put(o.W2 + (16 * jt + 4 * lk + r) * MLP_H + 16 * kt + li, gW2[jt][kt][r]);
      for (int i = 0; i < nin; ++i) put(o.W1 + i * MLP_H + lane, gW1[i]);
      put(o.b1 + lane, gb1);
      if (lk == 0)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          put(o.b2 + 16 * ct + li, gb2[ct]);
          put(o.w3 + 16 * ct + li, gw3[ct]);
        }
      if (lane == 0) put(o.b3, gb3);
    }
    __syncthreads();
  }
  float* out = partial + (int64_t)blockIdx.x * o.n;
  for (int k = threadIdx.x; k < o.n; k += blockDim.x) out[k] = sp[k];
}

// grad[e] = sum over workgroups of partial[b][e] (FP64, fixed order): 64 entries per workgroup, 16
// threads per entry each taking every 16th partial (one thread per entry walked up to 512 of them
// one after the other: 124 us for 4609 entries and 512 partials, 11 us now)
__global__ __launch_bounds__(1024) void k_mlp_reduce(int nparts, int n, const float* partial, float* grad) {
  __shared__ double red[16][64];
  const int te = threadIdx.x & 63, tp = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + te;
  double s = 0.0;
  if (e < n)
    for (int b = tp; b < nparts; b += 16) s += partial[(int64_t)b * n + e];
  red[tp][te] = s;
  __syncthreads();
  if (tp == 0 && e < n) {
    double t = 0.0;
    for (int k = 0; k < 16; ++k) t += red[k][te];
    grad[e] = (float)t;
  }
}

// Variance objective per group g (rows gptr[g]..gptr[g+1]), one workgroup per group:
// q = (1 - eps) softmax(z) + eps / n, l_g = sum b/q / (sum sqrt b)^2 and the unscaled
// gradient (1 - eps)/S sigma_f (sum_h r_h sigma_h - r_f), r = b / q^2; groups with
// sum b = 0 get l_g = 0, active = 0 and zero gradient.
__global__ __launch_bounds__(256) void k_loss_groups(const float* z, const double* b, const int64_t* gptr,
                                                     int64_t G, double eps, double* lg, int32_t* active,
                                                     float* dz) {
  __shared__ double red[256];
  for (int64_t g = blockIdx.x; g < G; g += gridDim.x) {
    const int64_t r0 = gptr[g], r1 = gptr[g + 1];
    const double n = (double)(r1 - r0);
    double mx = -INFINITY, sb = 0.0, ss = 0.0;
    for (int64_t k = r0 + threadIdx.x; k < r1; k += blockDim.x) {
      mx = fmax(mx, (double)z[k]);
      sb += b[k];
      ss += sqrt(b[k]);
    }
    mx = block_max(mx, red);
    sb = block_sum(sb, red);
    ss = block_sum(ss, red);
    if (!(sb > 0.0)) {
      for (int64_t k = r0 + threadIdx.x; k < r1; k += blockDim.x) dz[k] = 0.f;
      if (threadIdx.x == 0) {
        lg[g] = 0.0;
        active[g] = 0;
      }
      continue;
    }
    double se = 0.0;
    for (int64_t k = r0 + threadIdx.x; k < r1; k += blockDim.x) se += exp((double)z[k] - mx);
    se = block_sum(se, red);
    double sl = 0.0, srs = 0.0;
    for (int64_t k = r0 + threadIdx.x; k < r1; k += blockDim.x) {
      const double sig = exp((double)z[k] - mx) / se;
      const double qf = (1.0 - eps) * sig + eps / n;
      sl += b[k] / qf;
      srs += b[k] / (qf * qf) * sig;
    }
    sl = block_sum(sl, red);
    srs = block_sum(srs, red);
    const double S = ss * ss;
    for (int64_t k = r0 + threadIdx.x; k < r1; k += blockDim.x) {
      const double sig = exp((double)z[k] - mx) / se;
      const double qf = (1.0 - eps) * sig + eps / n;
      const double rf = b[k] / (qf * qf);
      dz[k] = (float)((1.0 - eps) / S * sig * (srs - rf));
    }
    if (threadIdx.x == 0) {
      lg[g] = sl / S;
      active[g] = 1;
    }
  }
}

// out[0] = mean of l_g over active groups, out[1] = 1 / (number of active groups) (0 if none)
__global__ __launch_bounds__(256) void k_loss_final(int64_t G, const double* lg, const int32_t* active,
                                                    double* out) {
  __shared__ double red[256];
  double s = 0.0, a = 0.0;
  for (int64_t g = threadIdx.x; g < G; g += blockDim.x) {
    s += lg[g];
    a += active[g];
  }
  s = block_sum(s, red);
  a = block_sum(a, red);
  if (threadIdx.x == 0) {
    out[0] = a > 0.0 ? s / a : 0.0;
    out[1] = a > 0.0 ? 1.0 / a : 0.0;
  }
}

__global__ __launch_bounds__(256) void k_scale_f32(int64_t n, const double* scale, float* x) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) x[e] = (float)((double)x[e] * *scale);
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// theta -= lr (m c1) / (sqrt(v c2) + eps) with c1 = 1/(1-b1^t), c2 = 1/(1-b2^t).
__global__ __launch_bounds__(256) void k_adam(int n, float* theta, float* m, float* v, const float* grad,
                                              double lr, double b1, double b2, double eps, double c1, double c2) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const double g = grad[e];
  const double mm = b1 * m[e] + (1.0 - b1) * g;
  const double vv = b2 * v[e] + (1.0 - b2) * g * g;
  m[e] = (float)mm;
  v[e] = (float)vv;
  theta[e] = (float)((double)theta[e] - lr * (mm * c1) / (sqrt(vv * c2) + eps));
}

// ================================================================ launchers
static size_t mlp_lds_fwd(int nin) { return (size_t)((MlpOff(nin).n + 3) & ~3) * sizeof(float); }
static size_t mlp_lds_bwd(int nin) {
  return (size_t)(((MlpOff(nin).n + 3) & ~3) + MLP_H * MLP_LDW + 4 * MLP_WTILE) * sizeof(float);
}

// workgroups of the backward pass (4 waves of 16-row chunks each): one partial gradient each
int mlp_bwd_blocks(int64_t M) {
  const int64_t nblk = (M + 4 * MLP_CH - 1) / (4 * MLP_CH);
  return (int)(nblk < 1 ? 1 : (nblk > 512 ? 512 : nblk));
}

hipError_t launch_mlp_fwd(hipStream_t s, const float* theta, int nin, const float* X, int64_t M, float* z) {
  if (M == 0) return hipSuccess;
  const int64_t nblk = (M + 4 * MLP_CH - 1) / (4 * MLP_CH);
  const unsigned grid = (unsigned)(nblk > 2048 ? 2048 : nblk);
  // d + 3 inputs of one- and two-dimensional systems compiled in, other networks at run time
  const auto k = nin == 4 ? k_mlp_fwd<4> : nin == 5 ? k_mlp_fwd<5> : k_mlp_fwd<0>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(256), mlp_lds_fwd(nin), s, theta, nin, X, M, z);
  return hipGetLastError();
}

hipError_t launch_mlp_bwd(hipStream_t s, const float* theta, int nin, const float* X, int64_t M, const float* dz,
                          const double* gscale, float* partial, float* grad) {
  const int nparts = mlp_bwd_blocks(M);
  const int n = MlpOff(nin).n;
  const auto k = nin == 4 ? k_mlp_bwd<4> : nin == 5 ? k_mlp_bwd<5> : k_mlp_bwd<0>;
  hipLaunchKernelGGL(k, dim3(nparts), dim3(256), mlp_lds_bwd(nin), s, theta, nin, X, M, dz, gscale, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_reduce, dim3((n + 63) / 64), dim3(1024), 0, s, nparts, n, partial, grad);
  return hipGetLastError();
}

hipError_t launch_loss(hipStream_t s, const float* z, const double* b, const int64_t* gptr, int64_t G, double eps,
                       double* lg, int32_t* active, float* dz, double* out) {
  if (G == 0) return hipSuccess;
  const unsigned grid = (unsigned)(G > 65536 ? 65536 : G);
  hipLaunchKernelGGL(k_loss_groups, dim3(grid), dim3(256), 0, s, z, b, gptr, G, eps, lg, active, dz);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, G, lg, active, out);
  return hipGetLastError();
}

hipError_t launch_scale_f32(hipStream_t s, int64_t n, const double* scale, float* x) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scale_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, scale, x);
  return hipGetLastError();
}

hipError_t launch_adam(hipStream_t s, int n, float* theta, float* m, float* v, const float* grad, double lr,
                       double b1, double b2, double eps, double c1, double c2) {
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, n, theta, m, v, grad, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

}  // namespace lsx

// Plan kernels of liblsx: fibre Hamiltonians, their eigendecomposition, the propagators and
// their bands.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lsx_pass.h"

namespace lsx {

template <int BS>
__device__ double block_sum(double v, double* sh) {
  // deterministic tree sum over a block of BS threads
  sh[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = BS / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------- assembly (eq. 3.6 on one fibre)
// A (ndim x ndim, row-major) <- H_j restricted to fibre f, or for complex H its real
// embedding [[Re H, -Im H], [Im H, Re H]]; padding rows/cols are zero.  Row i's lifted
// index is mn[i*stride ...]; layer j's own block starts at entry `own`; the kinetic share
// on the diagonal is kfac |K|^2 with kfac = (1 - kappa) / (2 nl) for nl layers.
// Workgroups (b, y) assemble fibre fid[b] into its own slot b.
__global__ void k_assemble(const int32_t* fid, const int32_t* ptr, const int32_t* rows, const int32_t* mn, int d,
                           int stride, int own, double kfac, const double* K2, int nv, const int32_t* vidx,
                           const double* vre, const double* vim, int embed, double* Aall, const int64_t* moff,
                           const int32_t* ndim) {
  const int b = blockIdx.x;
  const int f = fid[b];
  const int r0 = ptr[f], L = ptr[f + 1] - r0;
  const int n = ndim[b];
  double* A = Aall + moff[b];
  const int La = embed ? 2 * L : L;
  const int64_t nn = (int64_t)n * n;
  for (int64_t e = blockIdx.y * blockDim.x + threadIdx.x; e < nn; e += gridDim.y * blockDim.x) {
    const int a = (int)(e / n), b = (int)(e % n);
    double val = 0.0;
    if (a < La && b < La) {
      const int ar = a % L, br = b % L, qa = a / L, qb = b / L;
      const int ia = rows[r0 + ar], ib = rows[r0 + br];
      double hr = 0.0, hi = 0.0;
      for (int v = 0; v < nv; ++v) {
        bool match = true;
        for (int k = 0; k < d; ++k)
          match = match && (mn[(int64_t)ia * stride + own + k] - mn[(int64_t)ib * stride + own + k] == vidx[v * d + k]);
        if (match) {
          hr += vre[v];
          hi += vim[v];
        }
      }
      if (ar == br) hr += kfac * K2[ia];
      if (!embed) val = hr;
      else val = (qa == qb) ? hr : (qa == 0 ? -hi : hi);
    }
    A[e] = val;
  }
}

// ---------------------------------------------------------------- batched cyclic Jacobi
// One workgroup per fibre.  Round-robin (circle) ordering: in round r the pairs are
// (n-1, r) and ((r+i) mod (n-1), (r-i) mod (n-1)), i = 1..n/2-1, all disjoint, so a round
// is A <- J^T A J with J a product of n/2 independent plane rotations.  The update is
// done one 2x2 block at a time (block (i,j) depends only on rotations i and j), which
// needs no barrier between the row and the column transformation.  VT holds V^T, so
// H = V diag(lambda) V^T on exit, eigenvalues in the diagonal of A.
// Last step of both Jacobi solvers.  Each rotation is orthogonal only up to the rounding of
// (c, s): near-degenerate pairs (potential-only fibres) take 45-degree rotations with
// c = s = fl(1/sqrt 2), and 2 fl(1/sqrt 2)^2 = 1 + 2^-52, so both rows grow by the same factor and
// thousands of such rotations per row leave V scaled-orthogonal, V = Q diag(nu), and
// A = diag(nu) Q^T H Q diag(nu).  Normalising each eigenvector (row of V^T) and dividing its
// diagonal entry by nu^2 recovers Q and the eigenvalues.  One workgroup of BS threads.
template <int BS>
__device__ void jacobi_finish(const double* A, double* VT, int n, double* lamf) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  for (int k = wv; k < n; k += BS / 64) {
    double s = 0.0;
    for (int c = lane; c < n; c += 64) {
      const double x = VT[(int64_t)k * n + c];
      s += x * x;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    const double r = 1.0 / sqrt(s);
    for (int c = lane; c < n; c += 64) VT[(int64_t)k * n + c] *= r;
    if (lane == 0) lamf[k] = A[(int64_t)k * n + k] / s;
  }
}

// sel (nullable): workgroup i solves matrix sel[i] (else matrix i).
template <int BS>
__global__ __launch_bounds__(BS) void k_jacobi(double* Aall, double* VTall, const int64_t* moff,
                                               const int32_t* ndim, double* lam, const int64_t* loff,
                                               int32_t* info, int maxsweeps, const int32_t* sel) {
  const int f = sel ? sel[blockIdx.x] : blockIdx.x;
  const int n = ndim[f];
  double* A = Aall + moff[f];
  double* VT = VTall + moff[f];
  extern __shared__ double sh[];
  const int np = n / 2;
  double* rc = sh;
  double* rs = sh + np;
  int* rp = reinterpret_cast<int*>(sh + 2 * np);
  int* rq = rp + np;
  __shared__ double red[BS];
  __shared__ int rotated;
  const int tid = threadIdx.x;
  const int64_t nn = (int64_t)n * n;

  for (int64_t e = tid; e < nn; e += BS) VT[e] = ((e / n) == (e % n)) ? 1.0 : 0.0;
  double s2 = 0.0;
  for (int64_t e = tid; e < nn; e += BS) s2 += A[e] * A[e];
  const double normF = sqrt(block_sum<BS>(s2, red));
  // rotations are skipped below 1e-16 of the pair's diagonal scale plus 1e-16 ||H||_F:
  // the absolute term sits at rounding-noise level, so matrices with zero diagonal
  // (potential-only fibres) converge instead of rotating noise until the sweep limit
  const double tiny = 1e-16 * normF;

  int sweep = 0;
  bool done = (n < 2);
  for (; sweep < maxsweeps && !done; ++sweep) {
    if (tid == 0) rotated = 0;
    __syncthreads();
    const int m = n - 1;
    for (int r = 0; r < m; ++r) {
      for (int i = tid; i < np; i += BS) {
        const int p = (i == 0) ? m : (r + i) % m;
        const int q = (i == 0) ? r : (r - i + m) % m;
        const double app = A[(int64_t)p * n + p], aqq = A[(int64_t)q * n + q], apq = A[(int64_t)p * n + q];
        double c = 1.0, s = 0.0;
        if (fabs(apq) > 1e-16 * sqrt(fabs(app * aqq)) + tiny) {
          const double th = (aqq - app) / (2.0 * apq);
          const double t = (fabs(th) > 1e150) ? 0.5 / th
                                              : ((th >= 0.0) ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
          c = 1.0 / sqrt(t * t + 1.0);
          s = t * c;
          rotated = 1;
        }
        rc[i] = c;
        rs[i] = s;
        rp[i] = p;
        rq[i] = q;
      }
      __syncthreads();
      const int nb = np * np;
      for (int idx = tid; idx < nb; idx += BS) {
        const int i = idx / np, j = idx - (idx / np) * np;
        const double ci = rc[i], si = rs[i], cj = rc[j], sj = rs[j];
        if (si == 0.0 && sj == 0.0) continue;
        const int64_t p = rp[i], q = rq[i], p2 = rp[j], q2 = rq[j];
        const double a = A[p * n + p2], b = A[p * n + q2], cc = A[q * n + p2], dd = A[q * n + q2];
        const double a1 = ci * a - si * cc, b1 = ci * b - si * dd;
        const double c1 = si * a + ci * cc, d1 = si * b + ci * dd;
        double a2 = cj * a1 - sj * b1, b2 = sj * a1 + cj * b1;
        double c2 = cj * c1 - sj * d1, d2 = sj * c1 + cj * d1;
        if (i == j) {
          b2 = 0.0;
          c2 = 0.0;
        }
        A[p * n + p2] = a2;
        A[p * n + q2] = b2;
        A[q * n + p2] = c2;
        A[q * n + q2] = d2;
      }
      const int nv = np * n;
      for (int idx = tid; idx < nv; idx += BS) {
        const int i = idx / n, col = idx - (idx / n) * n;
        const double s = rs[i];
        if (s == 0.0) continue;
        const double c = rc[i];
        const int64_t p = rp[i], q = rq[i];
        const double x = VT[p * n + col], y = VT[q * n + col];
        VT[p * n + col] = c * x - s * y;
        VT[q * n + col] = s * x + c * y;
      }
      __syncthreads();
    }
    done = (rotated == 0);
    __syncthreads();
  }
  jacobi_finish<BS>(A, VT, n, lam + loff[f]);
  if (tid == 0) info[f] = done ? sweep : -1;
}

// ---------------------------------------------------------------- blocked two-sided Jacobi
// For long fibres.  A matrix of padded size n (a multiple of 32; padding rows and columns are
// zero and are never rotated) is cut into nb = n/16 blocks of 16 rows.  A round pairs the
// blocks with the same circle method the scalar solver uses for rows, into nb/2 disjoint pairs
// P = (I, J).  For every pair the 32x32 diagonal subproblem A[P, P] is rotated in LDS (its share
// of one cyclic Jacobi sweep), the rotations accumulating into Q_P; then every 32x32 tile of A and of V^T is
// replaced, A[P, P'] <- Q_P^T A[P, P'] Q_P' and V^T[P, R] <- Q_P^T V^T[P, R] (R: 32 columns).
// Each output tile depends only on its own input tile and two rotations, so a round is two
// launches with no other synchronisation, and the tile products run on the FP64 matrix cores.
// A sweep with no rotation in any subproblem leaves every off-diagonal entry below the same
// threshold as the scalar solver's; the same final normalisation applies.

// blocks (I, J) of pair i in round r of nb blocks (circle method, nb even)
__device__ __forceinline__ void bj_pair(int nb, int r, int i, int& I, int& J) {
  const int M = nb - 1;
  if (i == 0) {
    I = M;
    J = r;
  } else {
    I = (r + i) % M;
    J = (r - i + M) % M;
  }
}

__global__ __launch_bounds__(1024) void k_bj_init(BJArgs g, const int32_t* sel) {
  const int m = sel[blockIdx.x];
  const int n = g.ndim[m];
  const double* A = g.A + g.moff[m];
  double* VT = g.VT + g.moff[m];
  __shared__ double red[1024];
  const int64_t nn = (int64_t)n * n;
  double s2 = 0.0;
  for (int64_t e = threadIdx.x; e < nn; e += 1024) {
    VT[e] = ((e / n) == (e % n)) ? 1.0 : 0.0;
    s2 += A[e] * A[e];
  }
  const double normF = sqrt(block_sum<1024>(s2, red));
  if (threadIdx.x == 0) g.tiny[m] = 1e-16 * normF;
}

// 1 / sqrt(x) for x in [0.25, 8): the hardware estimate y0, with e = 1 - x y0^2 corrected by the binomial
// series of (1 - e)^(-1/2) to second order, 1 + e / 2 + 3 e^2 / 8, and then by one Newton step,
// 1 + e / 2.
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = fma(-x * y, y, 1.0);
  y = fma(y * e, fma(0.375, e, 0.5), y);
  e = fma(-x * y, y, 1.0);
  return fma(0.5 * y, e, y);
}

// Rotation (c, s) of the pair with entries app, aqq, apq; false: apq is below the threshold and stays.
// The scalar solver's angle, tan = sgn(d / apq) 2 |apq| / (|d| + h) with d = aqq - app and
// h = sqrt(d^2 + 4 apq^2), from two reciprocal roots: c^2 = (1 + |d| / h) / 2, |s| = |apq| / (h c).
// d and apq are scaled by a power of two first, so that no square leaves the range.
__device__ __forceinline__ bool bj_rotation(double app, double aqq, double apq, double tiny, double& c, double& s) {
  c = 1.0;
  s = 0.0;
  const double over = fabs(apq) - tiny;  // rotated when |apq| > tiny + 1e-16 sqrt|app aqq|
  if (!(over > 0.0 && over * over > 1e-32 * fabs(app * aqq))) return false;
  double d = aqq - app;
  const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(apq)));
  d = __builtin_amdgcn_ldexp(d, -e);
  const double a = __builtin_amdgcn_ldexp(apq, -e);
  const double r = rsqrt_f64(fma(d, d, 4.0 * a * a));
  const double x = fma(0.5 * fabs(d), r, 0.5);
  const double y = rsqrt_f64(x);
  c = x * y;
  s = (d >= 0.0 ? a : -a) * r * y;
  return true;
}

// Every index pair of the matrix meets once a sweep: the pairs across the two blocks of P in sixteen
// rounds here, the pairs inside a block in the fifteen before them in the sweep's first round of
// blocks.  A round takes one barrier: every wave works out all sixteen rotations and S alternates
// between two arrays.  Bound by the latency of that chain (LDS, two reciprocal roots, lane exchange,
// LDS), and by its fixed part (launch, loads) in the rounds that rotate nothing: 13.6 us a launch on
// average (twisted bilayer, N = 85261, 459 launches), 25.7 (432 launches) with every pair in every
// block round, three divisions and three roots a rotation and two barriers.
__global__ __launch_bounds__(256) void k_bj_pairs(BJArgs g) {
  __shared__ double S[2][32][33];
  __shared__ double Qs[32][33];
  const int a = blockIdx.x, i = blockIdx.y;
  const int m = g.mat[a];
  const int n = g.ndim[m];
  if (i >= n >> 5) return;
  int I, J;
  bj_pair(n >> 4, g.round, i, I, J);
  const double* A = g.A + g.moff[m];
  const int tid = threadIdx.x;
  for (int e = tid; e < 1024; e += 256) {
    const int x = e >> 5, y = e & 31;
    const int gx = (x < 16 ? I : J) * 16 + (x & 15), gy = (y < 16 ? I : J) * 16 + (y & 15);
    S[0][x][y] = A[(int64_t)gx * n + gy];
    Qs[x][y] = (x == y) ? 1.0 : 0.0;
  }
  const double tiny = g.tiny[m];
  const int bi = tid >> 4, bj = tid & 15;
  int cur = 0;
  bool any = false;
  // S <- J^T S J, rows (p, q), columns (p2, q2) by this thread; Q <- Q J, columns (p2, q2) of rows bi
  // and bi + 16
  auto round = [&](int p, int q, int p2, int q2) {
    const double(*X)[33] = S[cur];
    double(*Y)[33] = S[cur ^ 1];
    double cj, sj;
    const bool rj = bj_rotation(X[p2][p2], X[q2][q2], X[p2][q2], tiny, cj, sj);
    any |= rj;
    const double ci = __shfl(cj, bi), si = __shfl(sj, bi);  // lane bi of each wave has pair bi's
    const double a0 = X[p][p2], b0 = X[p][q2], c0 = X[q][p2], d0 = X[q][q2];
    const double a1 = ci * a0 - si * c0, b1 = ci * b0 - si * d0;
    const double c1 = si * a0 + ci * c0, d1 = si * b0 + ci * d0;
    const bool own = bi == bj && rj;  // the rotated pair's own entry
    Y[p][p2] = cj * a1 - sj * b1;
    Y[p][q2] = own ? 0.0 : sj * a1 + cj * b1;
    Y[q][p2] = own ? 0.0 : cj * c1 - sj * d1;
    Y[q][q2] = sj * c1 + cj * d1;
    if (rj) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double u = Qs[bi + 16 * h][p2], v = Qs[bi + 16 * h][q2];
        Qs[bi + 16 * h][p2] = cj * u - sj * v;
        Qs[bi + 16 * h][q2] = sj * u + cj * v;
      }
    }
    cur ^= 1;
    __syncthreads();
  };
  __syncthreads();
  if (g.round == 0) {
    // circle method inside each block: pair k < 8 in the first, k >= 8 in the second
#pragma unroll 1
    for (int r = 0; r < 15; ++r) {
      auto first = [&](int k) { return (k & 7) == 0 ? 15 : (r + (k & 7)) % 15; };
      auto second = [&](int k) { return (k & 7) == 0 ? r : (r - (k & 7) + 15) % 15; };
      const int oi = (bi & 8) * 2, oj = (bj & 8) * 2;
      round(oi + first(bi), oi + second(bi), oj + first(bj), oj + second(bj));
    }
  }
#pragma unroll 4
  for (int r = 0; r < 16; ++r) round(bi, 16 + ((bi + r) & 15), bj, 16 + ((bj + r) & 15));
  const int item = g.pfx_pairs[a] + i;
  double* Qo = g.Q + (int64_t)item * 1024;
  for (int e = tid; e < 1024; e += 256) Qo[e] = Qs[e >> 5][e & 31];
  const int rot = __syncthreads_or(any);
  if (tid == 0) {
    g.rotated[item] = rot;
    if (rot) g.flag[m] = 1;
  }
}

// One wave per 32x32 tile, four tiles per workgroup.  v_mfma_f64_16x16x4f64 takes A as lane l =
// A[l % 16][l / 16] and B as B[l / 16][l % 16] of a 16x4 / 4x16 step and leaves C[4 r + l / 16]
// [l % 16] in element r, so the accumulators of X = A_t Q_P' are, element for element, the B
// operands of the second product Q_P^T X.
__global__ LSX_MFMA_BOUNDS(256, true) void k_bj_tiles(BJArgs g) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int t = blockIdx.y * 4 + wv, a = blockIdx.x;
  const int m = g.mat[a];
  const int n = g.ndim[m], nb = n >> 4, np = nb >> 1;
  if (t >= 2 * np * np) return;
  const int li = lane & 15, lk = lane >> 4;
  const double* Qb = g.Q + (int64_t)g.pfx_pairs[a] * 1024;
  const v4d zero4 = {0.0, 0.0, 0.0, 0.0};
  v4d T[2][2] = {{zero4, zero4}, {zero4, zero4}};
  const int32_t* rotated = g.rotated + g.pfx_pairs[a];  // tiles between unrotated pairs stay as they are
  if (t < np * np) {
    const int P = t / np, P2 = t - (t / np) * np;
    if (!rotated[P] && !rotated[P2]) return;
    int I, J, I2, J2;
    bj_pair(nb, g.round, P, I, J);
    bj_pair(nb, g.round, P2, I2, J2);
    double* A = g.A + g.moff[m];
    const double* Q1 = Qb + (int64_t)P * 1024;
    const double* Q2 = Qb + (int64_t)P2 * 1024;
    v4d X[2][2] = {{zero4, zero4}, {zero4, zero4}};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * s + lk;
      const int gc = (k < 16 ? I2 : J2) * 16 + (k & 15);
      const double a0 = A[(int64_t)(I * 16 + li) * n + gc];
      const double a1 = A[(int64_t)(J * 16 + li) * n + gc];
      const double b0 = Q2[k * 32 + li], b1 = Q2[k * 32 + 16 + li];
      X[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, X[0][0], 0, 0, 0);
      X[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, X[0][1], 0, 0, 0);
      X[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, X[1][0], 0, 0, 0);
      X[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, X[1][1], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * s + lk;
      const double q0 = Q1[k * 32 + li], q1 = Q1[k * 32 + 16 + li];
      const double x0 = X[s >> 2][0][s & 3], x1 = X[s >> 2][1][s & 3];
      T[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(q0, x0, T[0][0], 0, 0, 0);
      T[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(q0, x1, T[0][1], 0, 0, 0);
      T[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(q1, x0, T[1][0], 0, 0, 0);
      T[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(q1, x1, T[1][1], 0, 0, 0);
    }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          A[(int64_t)((bi ? J : I) * 16 + 4 * r + lk) * n + (bj ? J2 : I2) * 16 + li] = T[bi][bj][r];
  } else {
    const int tv = t - np * np;
    const int P = tv / np, R = tv - (tv / np) * np;
    if (!rotated[P]) return;
    int I, J;
    bj_pair(nb, g.round, P, I, J);
    double* VT = g.VT + g.moff[m];
    const double* Q1 = Qb + (int64_t)P * 1024;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * s + lk;
      const int64_t gk = (int64_t)((k < 16 ? I : J) * 16 + (k & 15)) * n + R * 32;
      const double q0 = Q1[k * 32 + li], q1 = Q1[k * 32 + 16 + li];
      const double v0 = VT[gk + li], v1 = VT[gk + 16 + li];
      T[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(q0, v0, T[0][0], 0, 0, 0);
      T[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(q0, v1, T[0][1], 0, 0, 0);
      T[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(q1, v0, T[1][0], 0, 0, 0);
      T[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(q1, v1, T[1][1], 0, 0, 0);
    }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          VT[(int64_t)((bi ? J : I) * 16 + 4 * r + lk) * n + R * 32 + 16 * bj + li] = T[bi][bj][r];
  }
}

__global__ __launch_bounds__(1024) void k_bj_finish(BJArgs g, const int32_t* sel, double* lam, const int64_t* loff) {
  const int m = sel[blockIdx.x];
  const int n = g.ndim[m];
  jacobi_finish<1024>(g.A + g.moff[m], g.VT + g.moff[m], n, lam + loff[m]);
}

hipError_t launch_bj_init(hipStream_t s, int nsel, const int32_t* sel, const BJArgs& g) {
  if (nsel == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bj_init, dim3(nsel), dim3(1024), 0, s, g, sel);
  return hipGetLastError();
}

hipError_t launch_bj_round(hipStream_t s, int count, int maxn, const BJArgs& g) {
  if (count == 0) return hipSuccess;
  // Matrices in x: their number has no bound below x's, where y and z end at 65535.  The pairs of a
  // matrix of 8192 rows (the most precompute_layer takes) are 256, its workgroups of tiles 32768.
  const int np = maxn / 32;
  hipLaunchKernelGGL(k_bj_pairs, dim3(count, np), dim3(256), 0, s, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bj_tiles, dim3(count, (2 * np * np + 3) / 4), dim3(256), 0, s, g);
  return hipGetLastError();
}

hipError_t launch_bj_finish(hipStream_t s, int nsel, const int32_t* sel, const BJArgs& g, double* lam,
                            const int64_t* loff) {
  if (nsel == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bj_finish, dim3(nsel), dim3(1024), 0, s, g, sel, lam, loff);
  return hipGetLastError();
}

// f(lambda) = g + i h of one sub-step of length t for each eigenvalue:
//   flow 0 (exact flow)        exp(-i t lambda)
//   flow 1 (backward Euler)    1 / (1 + i t lambda)                     (Alg. 2)
//   flow 2 (Crank-Nicolson)    (1 - i t lambda / 2) / (1 + i t lambda / 2)  (eq. 4.6)
__global__ void k_eig_fn(int64_t nlam, const double* lam, double t, int flow, double2* gh) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nlam) {
    const double x = t * lam[i];
    double g, h;
    if (flow == 0) {
      double sn, cn;
      sincos(x, &sn, &cn);
      g = cn;
      h = -sn;
    } else if (flow == 1) {
      const double den = 1.0 + x * x;
      g = 1.0 / den;
      h = -x / den;
    } else {
      const double q = 0.25 * x * x, den = 1.0 + q;
      g = (1.0 - q) / den;
      h = -x / den;
    }
    gh[i] = make_double2(g, h);
  }
}

// ---------------------------------------------------------------- propagator formation
// P(t) = f(H) = sum_k V[.][k] f(lambda_k) V[.][k]^T with f = g + i h.  For an embedded
// complex H (real form M = [[Re H, -Im H], [Im H, Re H]]), g(M) and h(M) hold Re/Im of g(H)
// and h(H) in their left blocks (C_A, C_B and S_A, S_B), so P = (C_A - S_B) + i (C_B + S_A).
// Workgroups (b, y) form fibre fid[b] (slot b); the mixed formats' diagonal goes to positions ptr[f]+a.
//
// A contraction over the eigenvectors, on the FP64 matrix cores: a wave takes a 16-row block by 16
// NB columns, with the entries' columns as the matrix rows and the entries' rows as the matrix columns,
// so that C[4 r + l / 16][l % 16] of lane l is element l of chunk 4 cb + r of the stored order and both
// operands are rows of V^T as they lie.  Twisted bilayer, N = 85261: 187 us a propagator set, 1.9 ms
// with one entry a thread and no operand shared.
template <int FMT, bool EMB>
__device__ __forceinline__ void form_tile(const double* VT, const double2* gh, int n, int L, int rb, int cb0, char* P,
                                          double2* diag) {
  constexpr int NB = 2;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const v4d zero4 = {0.0, 0.0, 0.0, 0.0};
  v4d CA[NB], SA[NB], CB[NB], SB[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) CA[nb] = SA[nb] = CB[nb] = SB[nb] = zero4;
  const int arow = 16 * rb + li;
  const bool rok = arow < L;
  int col[NB];
  bool cok[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    col[nb] = 16 * (cb0 + nb) + li;
    cok[nb] = col[nb] < L;
  }
  constexpr int U = 4;
  struct Step {
    double u, u2, v[NB];
    double2 c;
  };
  // k-step ks: eigenvectors 4 ks + lk; entries outside the fibre are zero
  auto load = [&](Step& s, int ks) {
    const int k = 4 * ks + lk;
    const bool ok = k < n;
    const double* row = VT + (int64_t)(ok ? k : 0) * n;
    s.u = ok && rok ? row[arow] : 0.0;
    if (EMB) s.u2 = ok && rok ? row[L + arow] : 0.0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) s.v[nb] = ok && cok[nb] ? row[col[nb]] : 0.0;
    s.c = ok ? gh[k] : make_double2(0.0, 0.0);
  };
  const int nks = (n + 3) >> 2;
  Step A[U];
#pragma unroll
  for (int j = 0; j < U; ++j) load(A[j], j);
  for (int ks = 0; ks < nks; ks += U) {
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const Step s = A[j];
      load(A[j], ks + U + j);
      const double uc = s.u * s.c.x, us = s.u * s.c.y;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        CA[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.v[nb], uc, CA[nb], 0, 0, 0);
        SA[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.v[nb], us, SA[nb], 0, 0, 0);
        if (EMB) {
          CB[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.v[nb], s.u2 * s.c.x, CB[nb], 0, 0, 0);
          SB[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.v[nb], s.u2 * s.c.y, SB[nb], 0, 0, 0);
        }
      }
    }
  }
  if (!rok) return;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int bb = 16 * (cb0 + nb) + 4 * r + lk;
      if (bb >= L) continue;
      const double pr = EMB ? CA[nb][r] - SB[nb][r] : CA[nb][r], pi = EMB ? CB[nb][r] + SA[nb][r] : SA[nb][r];
      if (FMT != PF_F64 && arow == bb) {
        diag[arow] = make_double2(pr, pi);
      } else if (FMT == PF_BF16X3) {
        const int Lp = (L + 31) & ~31;
        const int64_t chunk = (int64_t)rb * (Lp >> 5) + (bb >> 5);
        const int el = bb & 7;
        unsigned short* Q = reinterpret_cast<unsigned short*>(P);
        unsigned short t[6];
        split3(pr, t[0], t[2], t[4]);
        split3(pi, t[1], t[3], t[5]);
#pragma unroll
        for (int pl = 0; pl < 6; ++pl) Q[((chunk * 6 + pl) * 64 + li + 16 * ((bb & 31) >> 3)) * 8 + el] = t[pl];
      } else {
        const int Lp = (L + 15) & ~15;
        const int64_t idx = ((int64_t)rb * (Lp >> 2) + (bb >> 2)) * 64 + lane;
        if (FMT == PF_F64) reinterpret_cast<double2*>(P)[idx] = make_double2(pr, pi);
        else reinterpret_cast<float2*>(P)[idx] = make_float2((float)pr, (float)pi);
      }
    }
}

template <int FMT>
__global__ LSX_MFMA_BOUNDS(256, true) void k_form(const int32_t* fid, const int32_t* ptr, const double* VTall,
                                                  const int64_t* moff, const int32_t* ndim, const int32_t* embed,
                                                  const double2* ghall, const int64_t* loff, void* Pall,
                                                  const int64_t* poff, double2* diag) {
  const int b = blockIdx.x;
  const int f = fid[b];
  const int r0 = ptr[f], L = ptr[f + 1] - r0;
  const double* VT = VTall + moff[b];
  const double2* gh = ghall + loff[b];
  char* P = reinterpret_cast<char*>(Pall) + poff[b];
  const int nrb = (L + 15) >> 4, ncb = (L + 31) >> 5;
  for (int u = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); u < nrb * ncb; u += 4 * gridDim.y) {
    const int rb = u / ncb, cb0 = 2 * (u - rb * ncb);
    if (embed[b]) form_tile<FMT, true>(VT, gh, ndim[b], L, rb, cb0, P, diag + (FMT == PF_F64 ? 0 : r0));
    else form_tile<FMT, false>(VT, gh, ndim[b], L, rb, cb0, P, diag + (FMT == PF_F64 ? 0 : r0));
  }
}

// ---------------------------------------------------------------- propagator bands
// Over one short step an entry P_ab of a fibre propagator is reached only through chains of
// potential couplings from a to b, each link carrying a factor of order t|v|, so the entries
// fall off quickly away from the diagonal and most column chunks of a row block hold nothing
// a product could feel.  For every 16-row block of every stored propagator this records the
// first and one past the last column chunk (4 columns; 32 for the BF16x3 format) that holds an
// entry with |Re| + |Im| >= tol (for BF16x3 the sum over the three terms' magnitudes bounds
// the entry); a block with no such entry keeps its diagonal chunk.  Workgroups (b, y) take stored
// propagator b, one row block a wave.
template <int FMT>
__global__ __launch_bounds__(256) void k_band(const int32_t* fid, const int32_t* ptr, const void* Pall,
                                              const int64_t* poff, const int64_t* boff, double tol,
                                              int32_t* band) {
  constexpr int CW = FMT == PF_BF16X3 ? 32 : 4;
  constexpr int G = FMT == PF_BF16X3 ? 1 : 8;  // chunks read together
  const int b = blockIdx.x;
  const int f = fid[b];
  const int L = ptr[f + 1] - ptr[f];
  const int Lp = FMT == PF_BF16X3 ? (L + 31) & ~31 : (L + 15) & ~15;
  const int nc = Lp / CW, nrb = (L + 15) >> 4;
  const int lane = threadIdx.x & 63;
  const char* P = reinterpret_cast<const char*>(Pall) + poff[b];
  for (int rb = 4 * blockIdx.y + (threadIdx.x >> 6); rb < nrb; rb += 4 * gridDim.y) {
    int lo = -1, hi = -1;
    for (int kc0 = 0; kc0 < nc; kc0 += G) {
      bool big[G];
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int64_t ch = (int64_t)rb * nc + min(kc0 + j, nc - 1);
        if (FMT == PF_F64) {
          const double2 v = reinterpret_cast<const double2*>(P)[ch * 64 + lane];
          big[j] = fabs(v.x) + fabs(v.y) >= tol;
        } else if (FMT == PF_F32) {
          const float2 v = reinterpret_cast<const float2*>(P)[ch * 64 + lane];
          big[j] = (double)fabsf(v.x) + (double)fabsf(v.y) >= tol;
        } else {
          const v8u16* Q = reinterpret_cast<const v8u16*>(P) + ch * 6 * 64 + lane;
          v8u16 pl[6];
#pragma unroll
          for (int k = 0; k < 6; ++k) pl[k] = Q[k * 64];
          big[j] = false;
#pragma unroll
          for (int el = 0; el < 8; ++el) {
            double m = 0.0;
#pragma unroll
            for (int k = 0; k < 6; ++k) m += fabs((double)bf2f(pl[k][el]));
            big[j] = big[j] || m >= tol;
          }
        }
      }
#pragma unroll
      for (int j = 0; j < G; ++j)
        if (__any(big[j]) && kc0 + j < nc) {
          if (lo < 0) lo = kc0 + j;
          hi = kc0 + j + 1;
        }
    }
    if (lo < 0) {
      lo = (16 * rb) / CW;
      hi = lo + 1;
    }
    if (lane == 0) {
      band[2 * (boff[b] + rb)] = lo;
      band[2 * (boff[b] + rb) + 1] = hi;
    }
  }
}

// ================================================================ launchers
hipError_t launch_assemble(hipStream_t s, int nb, int maxn, const int32_t* fid, const int32_t* ptr, const int32_t* rows,
                           const int32_t* mn, int d, int stride, int own, double kfac, const double* K2, int nv,
                           const int32_t* vidx, const double* vre, const double* vim, int embed, double* A,
                           const int64_t* moff, const int32_t* ndim) {
  const unsigned gy = (unsigned)std::max<int64_t>(1, std::min<int64_t>(((int64_t)maxn * maxn + 1023) / 1024, 256));
  hipLaunchKernelGGL(k_assemble, dim3(nb, gy), dim3(256), 0, s, fid, ptr, rows, mn, d, stride, own, kfac, K2, nv, vidx,
                     vre, vim, embed, A, moff, ndim);
  return hipGetLastError();
}

hipError_t launch_jacobi(hipStream_t s, int nf, int maxn, double* A, double* VT, const int64_t* moff,
                         const int32_t* ndim, double* lam, const int64_t* loff, int32_t* info, int maxsweeps,
                         const int32_t* sel) {
  if (nf == 0) return hipSuccess;
  const size_t shm = (size_t)(maxn / 2) * (2 * sizeof(double) + 2 * sizeof(int));
  if (maxn > 256)
    hipLaunchKernelGGL(k_jacobi<1024>, dim3(nf), dim3(1024), shm, s, A, VT, moff, ndim, lam, loff, info,
                       maxsweeps, sel);
  else
    hipLaunchKernelGGL(k_jacobi<256>, dim3(nf), dim3(256), shm, s, A, VT, moff, ndim, lam, loff, info,
                       maxsweeps, sel);
  return hipGetLastError();
}

hipError_t launch_eig_fn(hipStream_t s, int64_t nlam, const double* lam, double t, int flow, double2* gh) {
  if (nlam == 0) return hipSuccess;
  hipLaunchKernelGGL(k_eig_fn, dim3((unsigned)((nlam + 255) / 256)), dim3(256), 0, s, nlam, lam, t, flow, gh);
  return hipGetLastError();
}

hipError_t launch_band(hipStream_t s, int fmt, int nb, int maxL, const int32_t* fid, const int32_t* ptr, const void* P,
                       const int64_t* poff, const int64_t* boff, double tol, int32_t* band) {
  if (nb == 0) return hipSuccess;
  const dim3 g(nb, (unsigned)std::min(64, std::max(1, (maxL + 63) / 64)));
  if (fmt == PF_F64)
    hipLaunchKernelGGL(k_band<PF_F64>, g, dim3(256), 0, s, fid, ptr, P, poff, boff, tol, band);
  else if (fmt == PF_F32)
    hipLaunchKernelGGL(k_band<PF_F32>, g, dim3(256), 0, s, fid, ptr, P, poff, boff, tol, band);
  else
    hipLaunchKernelGGL(k_band<PF_BF16X3>, g, dim3(256), 0, s, fid, ptr, P, poff, boff, tol, band);
  return hipGetLastError();
}

hipError_t launch_form(hipStream_t s, int fmt, int nb, int maxL, const int32_t* fid, const int32_t* ptr,
                       const double* VT, const int64_t* moff, const int32_t* ndim, const int32_t* embed,
                       const double2* gh, const int64_t* loff, void* P, const int64_t* poff, double2* diag) {
  const int64_t units = (int64_t)((maxL + 15) / 16) * ((maxL + 31) / 32);
  const unsigned gy = (unsigned)std::max<int64_t>(1, std::min<int64_t>((units + 3) / 4, 4096));
  const dim3 g(nb, gy);
  if (fmt == PF_F64)
    hipLaunchKernelGGL(k_form<PF_F64>, g, dim3(256), 0, s, fid, ptr, VT, moff, ndim, embed, gh, loff, P, poff, diag);
  else if (fmt == PF_F32)
    hipLaunchKernelGGL(k_form<PF_F32>, g, dim3(256), 0, s, fid, ptr, VT, moff, ndim, embed, gh, loff, P, poff, diag);
  else
    hipLaunchKernelGGL(k_form<PF_BF16X3>, g, dim3(256), 0, s, fid, ptr, VT, moff, ndim, embed, gh, loff, P, poff,
                       diag);
  return hipGetLastError();
}

}  // namespace lsx

// Fibre-pass kernels of liblsx for MI355X (gfx950, CDNA4, wave64).
//
// Exact-flow layer splitting on the lifted plane-wave coefficients
// (Wang, Chen, Zhou & Zhou, arXiv 2103.14897, Secs. 3-4, App. A): X_f <- P_f X_f for all fibres
// of a layer (Alg. 2 steps 1/2) as grouped complex GEMMs on MFMA (FP64, FP32, BF16x3), or
// matrix-vector products for a single state.  The row-split passes are in lsx_rowsplit.hip, the
// propagators' set-up in lsx_plan.hip, phase and reductions in lsx_reduce.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <map>
#include <mutex>
#include <type_traits>

#include "lsx_pass.h"

namespace lsx {

// ---------------------------------------------------------------- MFMA fibre passes
// Tile = (fibre, 16 output rows rb, 16*NB columns wb).  The KS waves of a workgroup
// take interleaved groups of U k-steps; all loads of a group (propagator chunk and
// state operands) are issued before its MFMAs, so a group pays the memory latency
// once.  When the input array is laid out fibre-contiguously (in_pos null) the state
// operands need no index load at all.

// Operand loads of one group of U k-steps (4 fibre positions each) for the FP64/FP32
// kernels: propagator chunk per k-step (A operand) and NB state values (B operand).
template <typename PT, int NB, int U>
struct Group4 {
  PT p[U];
  double2 x[U][NB];
};

// All operand loads are unconditional: an out-of-range operand (k-step past the tile's
// band end kend, column past W) is read from a zeroed buffer instead, so the address is
// selected, not the value, and no loaded value is consumed before the MFMAs that need
// it -- the loads of the next group stay in flight during the current group.
template <bool GATHER, typename PT, int NB, int U>
__device__ __forceinline__ void load_group4(Group4<PT, NB, U>& G, const PassArgs& a, const PT* P, int g, int kend,
                                            int r0, int L, int lk, const int (&wc)[NB], const bool (&wok)[NB]) {
  const PT* zp = reinterpret_cast<const PT*>(a.zero);
  const double2* zx = reinterpret_cast<const double2*>(a.zero);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int ks = g + u, k = 4 * ks + lk;
    G.p[u] = *((ks < kend) ? P + (int64_t)ks * 64 : zp);
    const bool ok = ks < kend && k < L;
    const int64_t row = xrow<GATHER>(a, r0 + (ok ? k : 0));
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) G.x[u][nb] = *((ok && wok[nb]) ? a.X + row * a.W + wc[nb] : zx);
  }
}

// Complex products with three real MFMAs (the 3M / Gauss form): for P = a + ib and
// x = c + id,  k1 = (a + b) c,  k2 = a (d - c),  k3 = b (c + d);  Re = k1 - k3, Im = k1 + k2.
// The sums a + b, d - c, c + d are formed on the VALU in the operand precision.
template <int NB, int U>
__device__ __forceinline__ void mma_group_f64(v4d (&k1)[NB], v4d (&k2)[NB], v4d (&k3)[NB],
                                              const Group4<double2, NB, U>& G) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const double ps = G.p[u].x + G.p[u].y;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const double xr = G.x[u][nb].x, xi = G.x[u][nb].y;
      k1[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ps, xr, k1[nb], 0, 0, 0);
      k2[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(G.p[u].x, xi - xr, k2[nb], 0, 0, 0);
      k3[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(G.p[u].y, xr + xi, k3[nb], 0, 0, 0);
    }
  }
}

template <int NB, int U>
__device__ __forceinline__ void mma_group_f32(v4f (&k1)[NB], v4f (&k2)[NB], v4f (&k3)[NB],
                                              const Group4<float2, NB, U>& G) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const float ps = G.p[u].x + G.p[u].y;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float xr = (float)G.x[u][nb].x, xi = (float)G.x[u][nb].y;
      k1[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ps, xr, k1[nb], 0, 0, 0);
      k2[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(G.p[u].x, xi - xr, k2[nb], 0, 0, 0);
      k3[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(G.p[u].y, xr + xi, k3[nb], 0, 0, 0);
    }
  }
}

// ---------------------------------------------------------------- persistent batched launches
// The grid holds what the chip keeps resident (a multiple of 8 workgroups).  The tile list is
// XCD interleaved (tile i belongs to XCD i mod 8) and workgroup b runs on XCD b mod 8.
//  persist = 1: workgroup b takes the tiles i = 8 k + (b mod 8), k = 0, 1, ..., of its XCD's
//    queue through a device atomic counter, so uneven tiles balance dynamically within each
//    XCD; the claim of the next tile is issued before the current tile runs, so its latency
//    overlaps the tile's loads.  queue[0..7] are the per-XCD counters and queue[8] counts
//    finished workgroups; the last workgroup to finish clears all nine, so every launch starts
//    from zeros without a memset node (graph replays).
//  persist = 2: workgroup b takes the tiles b, b + G, b + 2G, ... (G = grid size), no atomics.
// No workgroup waits on another.
template <typename Tile>
__device__ __forceinline__ void persistent_tiles(const PassArgs& a0, Tile&& tile) {
  if (a0.persist == 2) {
    for (int ti = blockIdx.x; ti < a0.ntiles; ti += gridDim.x) {
      tile(ti);
      __syncthreads();  // the tile's LDS is free again
    }
    return;
  }
  __shared__ int next;
  const int x = blockIdx.x & 7;
  if (threadIdx.x == 0) next = 8 * atomicAdd(a0.queue + x, 1) + x;
  __syncthreads();
  int ti = next;
  while (ti < a0.ntiles) {
    int ahead = 0;
    if (threadIdx.x == 0) ahead = 8 * atomicAdd(a0.queue + x, 1) + x;
    tile(ti);
    __syncthreads();  // the tile's LDS and `next` are free again
    if (threadIdx.x == 0) next = ahead;
    __syncthreads();
    ti = next;
  }
  if (threadIdx.x == 0 && atomicAdd(a0.queue + 8, 1) == (int)gridDim.x - 1)
    for (int i = 0; i < 9; ++i) atomicExch(a0.queue + i, 0);
}

// FP64: complex128 P, X on v_mfma_f64_16x16x4f64.  Three independent accumulator chains
// per column block (the 3M products above); groups of U k-steps are double buffered in
// registers, so the loads of group g+1 are in flight during the MFMAs of g.
template <int NB, int KS, int U, bool GATHER, bool BATCH>
__device__ __forceinline__ void k_pass_f64_tile(const PassArgs& a0, int ti, double* red) {
  const TileDesc t = a0.tiles[ti];
  if (t.f < 0) return;
  // batched launches: this tile's system arguments (uniform scalar loads)
  const PassArgs a = BATCH ? a0.batch[t.f] : a0;
  const int r0 = t.r0, L = t.L;
  const int nks = ((L + 15) & ~15) >> 2;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const double2* P = reinterpret_cast<const double2*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                     (int64_t)t.rb * nks * 64 + lane;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  v4d k1[NB], k2[NB], k3[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (v4d){0.0, 0.0, 0.0, 0.0};
  // two register buffers in ping-pong: B is loaded while A is consumed and vice versa
  Group4<double2, NB, U> A, B;
  const int stride = KS * U;
  int klo, khi;
  tile_band(t, 4 * nks, 4, klo, khi);
  int g = klo + kw * U;
  load_group4<GATHER>(A, a, P, g, khi, r0, L, lk, wc, wok);
  for (; g < khi; g += 2 * stride) {
    load_group4<GATHER>(B, a, P, g + stride, khi, r0, L, lk, wc, wok);  // past the band: zeros
    __builtin_amdgcn_sched_barrier(0);
    mma_group_f64(k1, k2, k3, A);
    if (g + stride >= khi) break;
    load_group4<GATHER>(A, a, P, g + 2 * stride, khi, r0, L, lk, wc, wok);
    __builtin_amdgcn_sched_barrier(0);
    mma_group_f64(k1, k2, k3, B);
  }
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = k1[nb][r] - k3[nb][r];
      acc[nb][1][r] = k1[nb][r] + k2[nb][r];
    }
  pass_epilogue<NB, KS, false, true>(a, t, acc, red, wc, wok);
}

template <int NB, int KS, int U, bool GATHER, bool BATCH>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB < 4) void k_pass_f64(PassArgs a0) {
  extern __shared__ double red[];
  k_pass_f64_tile<NB, KS, U, GATHER, BATCH>(a0, blockIdx.x, red);
}

template <int NB, int KS, int U, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB < 4) void k_pass_f64_persist(PassArgs a0) {
  extern __shared__ double red[];
  persistent_tiles(a0, [&](int ti) { k_pass_f64_tile<NB, KS, U, GATHER, true>(a0, ti, red); });
}

// Mixed FP32: y = d .* x (FP64) + E x~ with E complex64, x~ = fp32(x), FP32 MFMA
// accumulation (v_mfma_f32_16x16x4f32, 3M products), same pipelining as the FP64 kernel.
template <int NB, int KS, int U, bool GATHER, bool BATCH>
__device__ __forceinline__ void k_pass_f32_tile(const PassArgs& a0, int ti, double* red) {
  const TileDesc t = a0.tiles[ti];
  if (t.f < 0) return;
  // batched launches: this tile's system arguments (uniform scalar loads)
  const PassArgs a = BATCH ? a0.batch[t.f] : a0;
  const int r0 = t.r0, L = t.L;
  const int nks = ((L + 15) & ~15) >> 2;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const float2* P = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                    (int64_t)t.rb * nks * 64 + lane;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  v4f k1[NB], k2[NB], k3[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  Group4<float2, NB, U> A, B;
  const int stride = KS * U;
  int klo, khi;
  tile_band(t, 4 * nks, 4, klo, khi);
  int g = klo + kw * U;
  load_group4<GATHER>(A, a, P, g, khi, r0, L, lk, wc, wok);
  for (; g < khi; g += 2 * stride) {
    load_group4<GATHER>(B, a, P, g + stride, khi, r0, L, lk, wc, wok);  // past the band: zeros
    __builtin_amdgcn_sched_barrier(0);
    mma_group_f32(k1, k2, k3, A);
    if (g + stride >= khi) break;
    load_group4<GATHER>(A, a, P, g + 2 * stride, khi, r0, L, lk, wc, wok);
    __builtin_amdgcn_sched_barrier(0);
    mma_group_f32(k1, k2, k3, B);
  }
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = (double)k1[nb][r] - (double)k3[nb][r];
      acc[nb][1][r] = (double)k1[nb][r] + (double)k2[nb][r];
    }
  pass_epilogue<NB, KS, true, false>(a, t, acc, red, wc, wok);
}

template <int NB, int KS, int U, bool GATHER, bool BATCH>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB * U < 16) void k_pass_f32(PassArgs a0) {
  extern __shared__ double red[];
  k_pass_f32_tile<NB, KS, U, GATHER, BATCH>(a0, blockIdx.x, red);
}

template <int NB, int KS, int U, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB * U < 16) void k_pass_f32_persist(PassArgs a0) {
  extern __shared__ double red[];
  persistent_tiles(a0, [&](int ti) { k_pass_f32_tile<NB, KS, U, GATHER, true>(a0, ti, red); });
}

// Mixed BF16x3: E = E0+E1+E2 and x~ = x0+x1+x2 (bf16 terms); the six products E0x0,
// E0x1, E1x0, E0x2, E1x1, E2x0 on v_mfma_f32_16x16x32_bf16 with FP32 accumulation, plus
// the FP64 diagonal term.  A k-step here is a chunk of 32 fibre positions.  Four
// accumulator chains (Er Xr, Ei Xi, Er Xi, Ei Xr); chunk loads are double buffered.
template <int NB>
struct ChunkBF {
  v8u16 e[6];
  double2 x[NB][8];
};

template <bool GATHER, int NB>
__device__ __forceinline__ void load_chunk_bf(ChunkBF<NB>& C, const PassArgs& a, const v8u16* P, int kc, int kend,
                                              int r0, int L, int lk, const int (&wc)[NB], const bool (&wok)[NB]) {
  const bool kin = kc < kend;
  const v8u16* zp = reinterpret_cast<const v8u16*>(a.zero);
  const double2* zx = reinterpret_cast<const double2*>(a.zero);
#pragma unroll
  for (int pl = 0; pl < 6; ++pl) C.e[pl] = *(kin ? P + ((int64_t)kc * 6 + pl) * 64 : zp);
#pragma unroll
  for (int el = 0; el < 8; ++el) {
    const int k = 32 * kc + 8 * lk + el;
    const bool ok = kin && k < L;
    const int64_t row = xrow<GATHER>(a, r0 + (ok ? k : 0));
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) C.x[nb][el] = *((ok && wok[nb]) ? a.X + row * a.W + wc[nb] : zx);
  }
}

template <int NB>
__device__ __forceinline__ void mma_chunk_bf(v4f (&rr)[NB], v4f (&ii)[NB], v4f (&ri)[NB], v4f (&ir)[NB],
                                             const ChunkBF<NB>& C) {
  const v8bf er0 = as_bf(C.e[0]), ei0 = as_bf(C.e[1]), er1 = as_bf(C.e[2]);
  const v8bf ei1 = as_bf(C.e[3]), er2 = as_bf(C.e[4]), ei2 = as_bf(C.e[5]);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    v8u16 xr0, xr1, xr2, xi0, xi1, xi2;
#pragma unroll
    for (int el = 0; el < 8; ++el) {
      unsigned short a0, a1, a2, b0, b1, b2;
      split3f((float)C.x[nb][el].x, a0, a1, a2);
      split3f((float)C.x[nb][el].y, b0, b1, b2);
      xr0[el] = a0; xr1[el] = a1; xr2[el] = a2;
      xi0[el] = b0; xi1[el] = b1; xi2[el] = b2;
    }
    const v8bf Xr0 = as_bf(xr0), Xr1 = as_bf(xr1), Xr2 = as_bf(xr2);
    const v8bf Xi0 = as_bf(xi0), Xi1 = as_bf(xi1), Xi2 = as_bf(xi2);
    rr[nb] = mma3(rr[nb], er0, er1, er2, Xr0, Xr1, Xr2);
    ii[nb] = mma3(ii[nb], ei0, ei1, ei2, Xi0, Xi1, Xi2);
    ri[nb] = mma3(ri[nb], er0, er1, er2, Xi0, Xi1, Xi2);
    ir[nb] = mma3(ir[nb], ei0, ei1, ei2, Xr0, Xr1, Xr2);
  }
}

template <int NB, int KS, int U, bool GATHER, bool BATCH>
__device__ __forceinline__ void k_pass_bf16x3_tile(const PassArgs& a0, int ti, double* red) {
  const TileDesc t = a0.tiles[ti];
  if (t.f < 0) return;
  // batched launches: this tile's system arguments (uniform scalar loads)
  const PassArgs a = BATCH ? a0.batch[t.f] : a0;
  const int r0 = t.r0, L = t.L;
  const int nkc = ((L + 31) & ~31) >> 5;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const v8u16* P = reinterpret_cast<const v8u16*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                   (int64_t)t.rb * nkc * 6 * 64 + lane;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  v4f rr[NB], ii[NB], ri[NB], ir[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) rr[nb] = ii[nb] = ri[nb] = ir[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  ChunkBF<NB> A, B;
  int klo, khi;
  tile_band(t, 32 * nkc, 32, klo, khi);
  int kc = klo + kw;
  load_chunk_bf<GATHER>(A, a, P, kc, khi, r0, L, lk, wc, wok);
  for (; kc < khi; kc += 2 * KS) {
    load_chunk_bf<GATHER>(B, a, P, kc + KS, khi, r0, L, lk, wc, wok);  // past the band: zeros
    __builtin_amdgcn_sched_barrier(0);
    mma_chunk_bf(rr, ii, ri, ir, A);
    if (kc + KS >= khi) break;
    load_chunk_bf<GATHER>(A, a, P, kc + 2 * KS, khi, r0, L, lk, wc, wok);
    __builtin_amdgcn_sched_barrier(0);
    mma_chunk_bf(rr, ii, ri, ir, B);
  }
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = (double)rr[nb][r] - (double)ii[nb][r];
      acc[nb][1][r] = (double)ri[nb][r] + (double)ir[nb][r];
    }
  pass_epilogue<NB, KS, true, false>(a, t, acc, red, wc, wok);
}

template <int NB, int KS, int U, bool GATHER, bool BATCH>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB == 1) void k_pass_bf16x3(PassArgs a0) {
  extern __shared__ double red[];
  k_pass_bf16x3_tile<NB, KS, U, GATHER, BATCH>(a0, blockIdx.x, red);
}

template <int NB, int KS, int U, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * KS, NB == 1) void k_pass_bf16x3_persist(PassArgs a0) {
  extern __shared__ double red[];
  persistent_tiles(a0, [&](int ti) { k_pass_bf16x3_tile<NB, KS, U, GATHER, true>(a0, ti, red); });
}

// ---------------------------------------------------------------- sampled passes (W > 1)
// Weighted fibre increments x + g (P_f x - x) of the drawn (fibre, wavepacket) pairs, from the
// compacted columns of every class of fibres with one propagator (SlotArgs), written straight into
// the state.  A workgroup takes one 16-row block of a class's propagator and all of the class's
// slots, 32 at a time; its KS waves split the fibre length in groups of U k-steps as in the passes
// above.  The weights, tens at a time, multiply the rounding of the mixed formats' FP32 sums, so which
// k-steps a sum covers shows in the result (1e-8 of the state): KS and U are those of a K-split pass of
// the state's size.
// Bound by reading the propagators (253 MB twice at most, at 16 draws for each of 128 wavepackets of
// the twisted bilayer, kappa = 1, N = 398821): 123 us a pass and 32 for the compaction.  Tiles of
// single fibres read a shared propagator once per drawn fibre (889 fibres share 58 of them) for 2.3
// drawn columns of 16 on average, on a grid sized for every fibre and column, and wrote a second
// array that was copied back: 650 to 790 us and 330.
template <int FMT, int KS, int U>
__global__ LSX_MFMA_BOUNDS(64 * KS, FMT != PF_BF16X3) void k_pass_slots(SlotArgs a) {
  constexpr int NB = 2;
  extern __shared__ double red[];
  const SlotUnit t = a.units[blockIdx.x];
  const int n = a.n[t.cls], L = t.L;
  const int64_t xb = a.xbase[t.cls];
  const Slot* slots = a.slot + a.sbase[t.cls];
  PassArgs pa;
  pa.X = a.Xc + xb;
  pa.zero = a.zero;
  pa.W = n;
  TileDesc td;
  td.k0 = t.k0;
  td.k1 = t.k1;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const char* Pb = reinterpret_cast<const char*>(a.P) + t.poff;
  for (int s0 = 16 * NB * blockIdx.y; s0 < n; s0 += 16 * NB * gridDim.y) {
    int wc[NB];
    bool wok[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      wc[nb] = s0 + 16 * nb + li;
      wok[nb] = wc[nb] < n;
    }
    double acc[NB][2][4];
    if constexpr (FMT == PF_BF16X3) {
      const int nkc = ((L + 31) & ~31) >> 5;
      const v8u16* P = reinterpret_cast<const v8u16*>(Pb) + (int64_t)t.rb * nkc * 6 * 64 + lane;
      v4f rr[NB], ii[NB], ri[NB], ir[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) rr[nb] = ii[nb] = ri[nb] = ir[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
      int klo, khi;
      tile_band(td, 32 * nkc, 32, klo, khi);
      for (int kc = klo + kw; kc < khi; kc += KS) {
        ChunkBF<NB> C;
        load_chunk_bf<false>(C, pa, P, kc, khi, 0, L, lk, wc, wok);
        mma_chunk_bf(rr, ii, ri, ir, C);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[nb][0][r] = (double)rr[nb][r] - (double)ii[nb][r];
          acc[nb][1][r] = (double)ri[nb][r] + (double)ir[nb][r];
        }
    } else {
      using PT = typename std::conditional<FMT == PF_F64, double2, float2>::type;
      using V = typename std::conditional<FMT == PF_F64, v4d, v4f>::type;
      const int nks = ((L + 15) & ~15) >> 2;
      const PT* P = reinterpret_cast<const PT*>(Pb) + (int64_t)t.rb * nks * 64 + lane;
      V k1[NB], k2[NB], k3[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (V){0, 0, 0, 0};
      int klo, khi;
      tile_band(td, 4 * nks, 4, klo, khi);
      Group4<PT, NB, U> A, B;
      const int stride = KS * U;
      auto mma = [&](const Group4<PT, NB, U>& G) {
        if constexpr (FMT == PF_F64) mma_group_f64(k1, k2, k3, G);
        else mma_group_f32(k1, k2, k3, G);
      };
      int g = klo + kw * U;
      load_group4<false>(A, pa, P, g, khi, 0, L, lk, wc, wok);
      for (; g < khi; g += 2 * stride) {
        load_group4<false>(B, pa, P, g + stride, khi, 0, L, lk, wc, wok);
        __builtin_amdgcn_sched_barrier(0);
        mma(A);
        if (g + stride >= khi) break;
        load_group4<false>(A, pa, P, g + 2 * stride, khi, 0, L, lk, wc, wok);
        __builtin_amdgcn_sched_barrier(0);
        mma(B);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc[nb][0][r] = (double)k1[nb][r] - (double)k3[nb][r];
          acc[nb][1][r] = (double)k1[nb][r] + (double)k2[nb][r];
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(((kw * NB + nb) * 2 + c) * 4 + r) * 64 + lane] = acc[nb][c][r];
    __syncthreads();
    for (int r = kw; r < 4; r += KS) {
      const int arow = 16 * t.rb + (FMT == PF_F64 ? 4 * r + lk : 4 * lk + r);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if (arow >= L || !wok[nb]) continue;
        double yr = 0.0, yi = 0.0;
        for (int j = 0; j < KS; ++j) {
          yr += red[(((j * NB + nb) * 2 + 0) * 4 + r) * 64 + lane];
          yi += red[(((j * NB + nb) * 2 + 1) * 4 + r) * 64 + lane];
        }
        const double2 x = pa.X[(int64_t)arow * n + wc[nb]];
        if (FMT != PF_F64) {
          const double2 dg = a.diag[t.d0 + arow];
          yr += dg.x * x.x - dg.y * x.y;
          yi += dg.x * x.y + dg.y * x.x;
        }
        const Slot sl = slots[wc[nb]];
        yr = x.x + sl.g * (yr - x.x);
        yi = x.y + sl.g * (yi - x.y);
        const int64_t row = a.pos ? a.pos[sl.r0 + arow] : sl.r0 + arow;
        if (a.pend) {  // the stored value: the true one with the pending phase taken off
          const double2 h = a.pend[row];
          const double zr = h.x * yr + h.y * yi;
          yi = h.x * yi - h.y * yr;
          yr = zr;
        }
        a.Y[row * a.W + sl.w] = make_double2(yr, yi);
      }
    }
    __syncthreads();  // the LDS is free again
  }
}

// ---------------------------------------------------------------- single-state fibre pass (W = 1)
// y += p x and (sr, si) <- h (sr, si) for complex operands as explicit fused multiply-adds in
// a fixed order, so the per-fibre and the orbit single-state kernels round alike
__device__ __forceinline__ void cmac(double& yr, double& yi, double pr, double pi, double2 x) {
  yr = __builtin_fma(pr, x.x, yr);
  yr = __builtin_fma(-pi, x.y, yr);
  yi = __builtin_fma(pr, x.y, yi);
  yi = __builtin_fma(pi, x.x, yi);
}
__device__ __forceinline__ void cscale(double& sr, double& si, double2 h) {
  const double zr = __builtin_fma(h.x, sr, -(h.y * si));
  si = __builtin_fma(h.x, si, h.y * sr);
  sr = zr;
}
// Single-state GEMV, one 16-row block per tile: each propagator entry is read once per pass.
// Lane (li, lk) of chunk (rb, k) multiplies entry (16rb+li, col) by x[col]; the four k-lanes
// and the KS waves are summed in fixed order.  Mixed formats: E entries (rounded to their
// storage precision) times the FP64 state, FP64 accumulation, plus the FP64 diagonal term.
template <int KS, int FMT, bool BATCH>
__device__ __forceinline__ void k_gemv_tile(const PassArgs& a0, int ti, double* red) {
  const TileDesc t = a0.tiles[ti];
  if (t.f < 0) return;
  const PassArgs a = BATCH ? a0.batch[t.f] : a0;
  const int r0 = t.r0, L = t.L;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const char* Pb = reinterpret_cast<const char*>(a.P) + t.poff;
  double yr = 0.0, yi = 0.0;
  if constexpr (FMT == PF_BF16X3) {
    const int nkc = ((L + 31) & ~31) >> 5;
    const v8u16* P = reinterpret_cast<const v8u16*>(Pb) + (int64_t)t.rb * nkc * 6 * 64 + lane;
    int klo, khi;
    tile_band(t, 32 * nkc, 32, klo, khi);
    for (int kc = klo + kw; kc < khi; kc += KS) {
      const v8u16* Pc = P + (int64_t)kc * 6 * 64;
      const v8u16 r0v = Pc[0], i0v = Pc[64], r1v = Pc[128], i1v = Pc[192], r2v = Pc[256], i2v = Pc[320];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 32 * kc + 8 * lk + e;
        if (k < L) {
          const double2 x = a.X[in_row(a, r0 + k)];
          const double er = (double)(bf2f(r0v[e]) + bf2f(r1v[e]) + bf2f(r2v[e]));
          const double ei = (double)(bf2f(i0v[e]) + bf2f(i1v[e]) + bf2f(i2v[e]));
          cmac(yr, yi, er, ei, x);
        }
      }
    }
  } else {
    // Groups of G k-steps: all loads of a group are issued before its products, with the
    // state operand of positions past the fibre read from the zero buffer (their propagator
    // entries are zero padding), so the loads stay branch-free; the products are summed in
    // k-step order as one at a time.
    using PT = typename std::conditional<FMT == PF_F64, double2, float2>::type;
    constexpr int G = 8;
    const int nks = ((L + 15) & ~15) >> 2;
    const double2* zx = reinterpret_cast<const double2*>(a.zero);
    const PT* P = reinterpret_cast<const PT*>(Pb) + (int64_t)t.rb * nks * 64 + lane;
    int klo, khi;
    tile_band(t, 4 * nks, 4, klo, khi);
    int ks = klo + kw;
    for (; ks + (G - 1) * KS < khi; ks += G * KS) {
      PT p[G];
      double2 x[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int kk = ks + g * KS, k = 4 * kk + lk;
        const bool ok = k < L;
        p[g] = P[(int64_t)kk * 64];
        x[g] = *(ok ? a.X + in_row(a, r0 + (ok ? k : 0)) : zx);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) cmac(yr, yi, p[g].x, p[g].y, x[g]);
    }
    for (; ks < khi; ks += KS) {
      const int k = 4 * ks + lk;
      const bool ok = k < L;
      const double2 x = *(ok ? a.X + in_row(a, r0 + (ok ? k : 0)) : zx);
      const PT pe = P[(int64_t)ks * 64];
      cmac(yr, yi, pe.x, pe.y, x);
    }
  }
  // sum the four k-lanes of each row (lanes li, li+16, li+32, li+48)
  yr += __shfl_xor(yr, 16);
  yi += __shfl_xor(yi, 16);
  yr += __shfl_xor(yr, 32);
  yi += __shfl_xor(yi, 32);
  if (lk == 0) {
    red[(kw * 2 + 0) * 16 + li] = yr;
    red[(kw * 2 + 1) * 16 + li] = yi;
  }
  __syncthreads();
  if (threadIdx.x < 16) {
    const int lr = threadIdx.x;
    const int arow = 16 * t.rb + lr;
    if (arow < L) {
      double sr = 0.0, si = 0.0;
      for (int w = 0; w < KS; ++w) {
        sr += red[(w * 2 + 0) * 16 + lr];
        si += red[(w * 2 + 1) * 16 + lr];
      }
      const int p = r0 + arow;
      if (FMT != PF_F64 || a.wt) {
        const double2 x = a.X[in_row(a, p)];
        if (FMT != PF_F64) {
          const double2 dg = a.diag[t.d0 + arow];
          cmac(sr, si, dg.x, dg.y, x);
        }
        if (a.wt) {
          const double g = a.wt[t.f];
          sr = x.x + g * (sr - x.x);
          si = x.y + g * (si - x.y);
        }
      }
      if (a.ph) cscale(sr, si, a.ph[a.ph_idx ? a.ph_idx[p] : p]);
      a.Y[a.out_pos ? a.out_pos[p] : p] = make_double2(sr, si);
    }
  }
}

template <int KS, int FMT, bool BATCH>
__global__ __launch_bounds__(64 * KS) void k_gemv(PassArgs a0) {
  __shared__ double red[2 * KS * 16];
  if (a0.tcount && (int)blockIdx.x >= *a0.tcount) return;
  k_gemv_tile<KS, FMT, BATCH>(a0, blockIdx.x, red);
}

template <int KS, int FMT>
__global__ __launch_bounds__(64 * KS) void k_gemv_persist(PassArgs a0) {
  __shared__ double red[2 * KS * 16];
  persistent_tiles(a0, [&](int ti) { k_gemv_tile<KS, FMT, true>(a0, ti, red); });
}

// ---------------------------------------------------------------- single-state orbit pass (W = 1)
// Fibres with one stored propagator (point-symmetry orbits, kappa = 1 translation classes)
// are multiplied together: a tile covers a 16-row block of the shared propagator for the
// states of up to M fibres of a group (PassArgs::orbit), so every propagator chunk is loaded
// once for the whole group instead of once per fibre.  Each fibre's products are summed in
// the order k_gemv_tile sums them for the same KS (k-steps in order per lane, then the four
// k-lanes, then the waves), so the two kernels give identical results.
template <int KS, int FMT, int M>
__global__ __launch_bounds__(64 * KS) void k_gemv_orbit(PassArgs a) {
  __shared__ double red[KS * M * 2 * 16];
  const TileDesc t = a.tiles[blockIdx.x];
  if (t.f < 0) return;
  const int32_t* og = a.orbit + (int64_t)t.f * kOrbitStride;
  const int nm = og[0];
  int r0[M];
#pragma unroll
  for (int m = 0; m < M; ++m) r0[m] = og[1 + m];
  const int L = t.L;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const char* Pb = reinterpret_cast<const char*>(a.P) + t.poff;
  double yr[M], yi[M];
#pragma unroll
  for (int m = 0; m < M; ++m) yr[m] = yi[m] = 0.0;
  if constexpr (FMT == PF_BF16X3) {
    const int nkc = ((L + 31) & ~31) >> 5;
    const v8u16* P = reinterpret_cast<const v8u16*>(Pb) + (int64_t)t.rb * nkc * 6 * 64 + lane;
    int klo, khi;
    tile_band(t, 32 * nkc, 32, klo, khi);
    for (int kc = klo + kw; kc < khi; kc += KS) {
      const v8u16* Pc = P + (int64_t)kc * 6 * 64;
      const v8u16 r0v = Pc[0], i0v = Pc[64], r1v = Pc[128], i1v = Pc[192], r2v = Pc[256], i2v = Pc[320];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 32 * kc + 8 * lk + e;
        if (k < L) {
          const double er = (double)(bf2f(r0v[e]) + bf2f(r1v[e]) + bf2f(r2v[e]));
          const double ei = (double)(bf2f(i0v[e]) + bf2f(i1v[e]) + bf2f(i2v[e]));
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const double2 x = a.X[in_row(a, r0[m] + k)];
            cmac(yr[m], yi[m], er, ei, x);
          }
        }
      }
    }
  } else {
    // groups of G k-steps, every load of a group issued before its products (state operands
    // past the fibre read the zero buffer, as in k_gemv_tile)
    using PT = typename std::conditional<FMT == PF_F64, double2, float2>::type;
    constexpr int G = M <= 2 ? 4 : (M <= 4 ? 2 : 1);
    const int nks = ((L + 15) & ~15) >> 2;
    const double2* zx = reinterpret_cast<const double2*>(a.zero);
    const PT* P = reinterpret_cast<const PT*>(Pb) + (int64_t)t.rb * nks * 64 + lane;
    int klo, khi;
    tile_band(t, 4 * nks, 4, klo, khi);
    int ks = klo + kw;
    for (; ks + (G - 1) * KS < khi; ks += G * KS) {
      PT p[G];
      double2 x[G][M];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int kk = ks + g * KS, k = 4 * kk + lk;
        const bool ok = k < L;
        p[g] = P[(int64_t)kk * 64];
#pragma unroll
        for (int m = 0; m < M; ++m) x[g][m] = *(ok ? a.X + in_row(a, r0[m] + (ok ? k : 0)) : zx);
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int m = 0; m < M; ++m) cmac(yr[m], yi[m], p[g].x, p[g].y, x[g][m]);
    }
    for (; ks < khi; ks += KS) {
      const int k = 4 * ks + lk;
      const bool ok = k < L;
      double2 x[M];
#pragma unroll
      for (int m = 0; m < M; ++m) x[m] = *(ok ? a.X + in_row(a, r0[m] + (ok ? k : 0)) : zx);
      const PT pe = P[(int64_t)ks * 64];
#pragma unroll
      for (int m = 0; m < M; ++m) cmac(yr[m], yi[m], pe.x, pe.y, x[m]);
    }
  }
  // sum the four k-lanes of each row, then the waves in order
#pragma unroll
  for (int m = 0; m < M; ++m) {
    double vr = yr[m], vi = yi[m];
    vr += __shfl_xor(vr, 16);
    vi += __shfl_xor(vi, 16);
    vr += __shfl_xor(vr, 32);
    vi += __shfl_xor(vi, 32);
    if (lk == 0) {
      red[((kw * M + m) * 2 + 0) * 16 + li] = vr;
      red[((kw * M + m) * 2 + 1) * 16 + li] = vi;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * M; idx += 64 * KS) {
    const int lr = idx & 15, m = idx >> 4;
    const int arow = 16 * t.rb + lr;
    if (m >= nm || arow >= L) continue;
    double sr = 0.0, si = 0.0;
    for (int w = 0; w < KS; ++w) {
      sr += red[((w * M + m) * 2 + 0) * 16 + lr];
      si += red[((w * M + m) * 2 + 1) * 16 + lr];
    }
    const int p = og[1 + m] + arow;
    if (FMT != PF_F64) {
      const double2 x = a.X[in_row(a, p)];
      const double2 dg = a.diag[t.d0 + arow];
      cmac(sr, si, dg.x, dg.y, x);
    }
    if (a.ph) cscale(sr, si, a.ph[a.ph_idx ? a.ph_idx[p] : p]);
    a.Y[a.out_pos ? a.out_pos[p] : p] = make_double2(sr, si);
  }
}

// ---------------------------------------------------------------- single-state passes, one row per lane
// A wave covers four 16-row blocks of a propagator (lane l: block l / 16 of the tile, row
// l % 16) and reads, for each k-step, all columns of its row from the lane slots of the
// stored chunk (four slots of one column for FP64 / FP32, four slots of eight columns for
// BF16x3), so the state operand of a k-step is the same for the whole wave: it is read once
// per wave through the scalar cache instead of once per lane.  ORB: the tile
// multiplies up to M fibres of a group with one propagator (PassArgs::orbit), else the tile's
// own fibre.  Per fibre and row the products are summed in column order, then the KS waves in a
// fixed order, so orbit and per-fibre tiles give identical results.  The k-steps run over the union
// of the four blocks' bands, and each block's lanes take zeros outside their own block's band.
template <int KS, int FMT, int M, bool ORB, bool GATHER>
__global__ __launch_bounds__(64 * KS) void k_gemv_rows(PassArgs a) {
  static_assert(ORB || M == 1, "a per-fibre tile has one fibre");
  constexpr int KR = KS > 4 ? 4 : KS;   // the waves' sums are added as pairs KR apart, then in order
  constexpr int KH = ORB ? KR : KS;     // sums held at a time
  __shared__ double red[KH * M * 2 * 64];
  const TileDesc t = a.tiles[blockIdx.x];
  if (t.f < 0) return;
  int nm = 1, r0[M];
  if constexpr (ORB) {
    const int32_t* og = a.orbit + (int64_t)t.f * kOrbitStride;
    nm = og[0];
#pragma unroll
    for (int m = 0; m < M; ++m) r0[m] = og[1 + m];
  } else {
    r0[0] = t.r0;
  }
  const int L = t.L;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, q = lane >> 4;
  const int nrb = (L + 15) >> 4;
  const int rbq = 4 * t.rb + q;
  const bool rowok = rbq < nrb;
  const char* Pb = reinterpret_cast<const char*>(a.P) + t.poff;
  // each row block's own band (fibre positions): its lanes read the zero buffer outside it
  int qlo = 0, qhi = kBandEnd;
  if (a.rb_band && t.bb >= 0 && rowok) {
    const int2 b = reinterpret_cast<const int2*>(a.rb_band)[t.bb + rbq];
    qlo = b.x;
    qhi = b.y;
  }
  double yr[M], yi[M];
#pragma unroll
  for (int m = 0; m < M; ++m) yr[m] = yi[m] = 0.0;
  if constexpr (FMT == PF_BF16X3) {
    // BF16x3 chunks of 32 columns: the row's four lane slots hold 8 consecutive columns each
    // (six planes of 8 bf16 per slot); per slot, the state operand is 8 consecutive rows of
    // every fibre (two 64-byte reads where contiguous)
    const int nkc = ((L + 31) & ~31) >> 5;
    const v8u16* zp = reinterpret_cast<const v8u16*>(a.zero);
    const v8u16* Pq = reinterpret_cast<const v8u16*>(Pb) + (int64_t)(rowok ? rbq : 0) * nkc * 6 * 64 + li;
    int klo, khi;
    tile_band(t, 32 * nkc, 32, klo, khi);
    struct X8 {
      double2 v[8];
    };
    for (int kc = klo + kw; kc < khi; kc += KS) {
      const bool in = rowok && 32 * kc >= qlo && 32 * kc < qhi;
      const v8u16* Pc = Pq + (int64_t)kc * 6 * 64;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v8u16 pl[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) pl[k] = *(in ? Pc + 64 * k + 16 * j : zp);
        double er[8], ei[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          er[e] = (double)(bf2f(pl[0][e]) + bf2f(pl[2][e]) + bf2f(pl[4][e]));
          ei[e] = (double)(bf2f(pl[1][e]) + bf2f(pl[3][e]) + bf2f(pl[5][e]));
        }
        const int c0 = 32 * kc + 8 * j;
        if (!GATHER && c0 + 7 < L) {
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const X8 x = *reinterpret_cast<const X8*>(a.X + r0[m] + c0);
#pragma unroll
            for (int e = 0; e < 8; ++e) cmac(yr[m], yi[m], er[e], ei[e], x.v[e]);
          }
        } else {
#pragma unroll
          for (int m = 0; m < M; ++m)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const double2 x = a.X[xrow<GATHER>(a, r0[m] + min(c0 + e, L - 1))];
              cmac(yr[m], yi[m], er[e], ei[e], x);
            }
        }
      }
    }
  } else {
    using PT = typename std::conditional<FMT == PF_F64, double2, float2>::type;
    const int nks = ((L + 15) & ~15) >> 2;
    const PT* zp = reinterpret_cast<const PT*>(a.zero);
    const PT* Pq = reinterpret_cast<const PT*>(Pb) + (int64_t)(rowok ? rbq : 0) * nks * 64 + li;
    int klo, khi;
    tile_band(t, 4 * nks, 4, klo, khi);
    auto src = [&](int kk, int c) { return (rowok && 4 * kk >= qlo && 4 * kk < qhi) ? Pq + (int64_t)kk * 64 + 16 * c : zp; };
    // The state operand of a k-step: four consecutive rows of every fibre, one 64-byte read per
    // fibre where its rows are contiguous (no gather, k-step inside the fibre); columns past the
    // fibre multiply zero padding and read the fibre's last row instead.  The entries of the next
    // k-step are loaded before this one's products (two steps ahead takes 87 registers and measured
    // slower: fewer waves fit).  With that and half the LDS, which let a fourth workgroup of eight
    // waves into a CU, a mixed FP32 pass of the twisted bilayer (N = 398821, 119 MB) takes 35.8 us, 40.3
    // before.
    struct X4 {
      double2 v[4];
    };
    PT f[4];  // the next k-step's entries
    if constexpr (ORB)
#pragma unroll
      for (int c = 0; c < 4; ++c) f[c] = *(klo + kw < khi ? src(klo + kw, c) : zp);
    for (int kk = klo + kw; kk < khi; kk += KS) {
      PT e[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) e[c] = ORB ? f[c] : *src(kk, c);
      if constexpr (ORB)
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = *(kk + KS < khi ? src(kk + KS, c) : zp);
      if (!GATHER && 4 * kk + 3 < L) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const X4 x = *reinterpret_cast<const X4*>(a.X + r0[m] + 4 * kk);
#pragma unroll
          for (int c = 0; c < 4; ++c) cmac(yr[m], yi[m], e[c].x, e[c].y, x.v[c]);
        }
      } else {
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double2 x = a.X[xrow<GATHER>(a, r0[m] + min(4 * kk + c, L - 1))];
            cmac(yr[m], yi[m], e[c].x, e[c].y, x);
          }
      }
    }
  }
  if constexpr (KS > KH) {  // the upper waves' sums go to the lower ones first
    if (kw >= KR)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        red[(((kw - KR) * M + m) * 2 + 0) * 64 + lane] = yr[m];
        red[(((kw - KR) * M + m) * 2 + 1) * 64 + lane] = yi[m];
      }
    __syncthreads();
    if (kw < KR)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        yr[m] += red[((kw * M + m) * 2 + 0) * 64 + lane];
        yi[m] += red[((kw * M + m) * 2 + 1) * 64 + lane];
      }
  }
  if (kw < KH)
#pragma unroll
    for (int m = 0; m < M; ++m) {
      red[((kw * M + m) * 2 + 0) * 64 + lane] = yr[m];
      red[((kw * M + m) * 2 + 1) * 64 + lane] = yi[m];
    }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 64 * M; idx += 64 * KS) {
    const int ln = idx & 63, m = idx >> 6;
    const int arow = 16 * (4 * t.rb + (ln >> 4)) + (ln & 15);
    if (m >= nm || arow >= L) continue;
    double sr = 0.0, si = 0.0;
    for (int w = 0; w < KR; ++w) {
      double vr = red[((w * M + m) * 2 + 0) * 64 + ln], vi = red[((w * M + m) * 2 + 1) * 64 + ln];
      if constexpr (KH > KR) {
        vr += red[(((w + KR) * M + m) * 2 + 0) * 64 + ln];
        vi += red[(((w + KR) * M + m) * 2 + 1) * 64 + ln];
      }
      sr += vr;
      si += vi;
    }
    const int p = (ORB ? a.orbit[(int64_t)t.f * kOrbitStride + 1 + m] : t.r0) + arow;
    if (FMT != PF_F64) {
      const double2 x = a.X[in_row(a, p)];
      const double2 dg = a.diag[t.d0 + arow];
      cmac(sr, si, dg.x, dg.y, x);
    }
    if (a.ph) cscale(sr, si, a.ph[a.ph_idx ? a.ph_idx[p] : p]);
    a.Y[a.out_pos ? a.out_pos[p] : p] = make_double2(sr, si);
  }
}

// ================================================================ launchers
// Prefetch depth of the FP64/FP32 passes (k-steps per register group); LSX_PREFETCH
// selects 1, 2 or 4 (default 2).
static int prefetch_depth() {
  static int u = [] {
    const char* v = std::getenv("LSX_PREFETCH");
    const int x = v ? std::atoi(v) : 2;
    return (x == 1 || x == 4) ? x : 2;
  }();
  return u;
}

// Set while prepare_persistent() runs: persistent launchers compute their grid (and so query
// the kernel's occupancy) and return without launching.
static thread_local bool g_prepare_only = false;

// Grid of a persistent launch: the kernel's resident workgroups per CU times the CU count,
// rounded down to a multiple of 8 (whole XCD rounds), at most the tile count rounded up to 8.
// The occupancy of each kernel is queried once.
static unsigned persistent_grid(const void* fn, int threads, size_t shm, int ntiles) {
  static std::map<const void*, int> cap;
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  auto it = cap.find(fn);
  if (it == cap.end()) {
    int dev = 0, ncu = 256, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      ncu = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, threads, shm) != hipSuccess || per < 1) per = 1;
    it = cap.emplace(fn, std::max(8, (per * ncu) / 8 * 8)).first;
  }
  const int want = (ntiles + 7) / 8 * 8;
  return (unsigned)std::max(8, std::min(want, it->second));
}

template <int NB, int KS, int U, bool G>
static hipError_t launch_mfma_persist(hipStream_t s, int fmt, int ntiles, const PassArgs& a0) {
  PassArgs a = a0;
  a.ntiles = ntiles;
  const size_t shm = KS > 1 ? (size_t)KS * NB * 2 * 4 * 64 * sizeof(double) : 0;
  const void* fn = fmt == PF_F64   ? reinterpret_cast<const void*>(&k_pass_f64_persist<NB, KS, U, G>)
                   : fmt == PF_F32 ? reinterpret_cast<const void*>(&k_pass_f32_persist<NB, KS, U, G>)
                                   : reinterpret_cast<const void*>(&k_pass_bf16x3_persist<NB, KS, 1, G>);
  const dim3 grid(persistent_grid(fn, 64 * KS, shm, ntiles));
  if (g_prepare_only) return hipSuccess;
  if (fmt == PF_F64)
    hipLaunchKernelGGL((k_pass_f64_persist<NB, KS, U, G>), grid, dim3(64 * KS), shm, s, a);
  else if (fmt == PF_F32)
    hipLaunchKernelGGL((k_pass_f32_persist<NB, KS, U, G>), grid, dim3(64 * KS), shm, s, a);
  else
    hipLaunchKernelGGL((k_pass_bf16x3_persist<NB, KS, 1, G>), grid, dim3(64 * KS), shm, s, a);
  return hipGetLastError();
}

template <int NB, int KS, int U, bool G, bool B>
static hipError_t launch_mfma_u(hipStream_t s, int fmt, int ntiles, const PassArgs& a) {
  const size_t shm = KS > 1 ? (size_t)KS * NB * 2 * 4 * 64 * sizeof(double) : 0;
  if constexpr (B) {
    if (a.persist) return launch_mfma_persist<NB, KS, U, G>(s, fmt, ntiles, a);
  }
  if (fmt == PF_F64)
    hipLaunchKernelGGL((k_pass_f64<NB, KS, U, G, B>), dim3(ntiles), dim3(64 * KS), shm, s, a);
  else if (fmt == PF_F32)
    hipLaunchKernelGGL((k_pass_f32<NB, KS, U, G, B>), dim3(ntiles), dim3(64 * KS), shm, s, a);
  else
    hipLaunchKernelGGL((k_pass_bf16x3<NB, KS, 1, G, B>), dim3(ntiles), dim3(64 * KS), shm, s, a);
  return hipGetLastError();
}

template <int NB, int KS, bool G>
static hipError_t launch_mfma_g(hipStream_t s, int fmt, int ntiles, const PassArgs& a, bool batched) {
  if (batched)
    return (fmt != PF_BF16X3 && a.u == 1) ? launch_mfma_u<NB, KS, 1, G, true>(s, fmt, ntiles, a)
                                          : launch_mfma_u<NB, KS, 2, G, true>(s, fmt, ntiles, a);
  switch (fmt == PF_BF16X3 ? 1 : (a.u == 1 || a.u == 2 || a.u == 4) ? a.u : prefetch_depth()) {
    case 1: return launch_mfma_u<NB, KS, 1, G, false>(s, fmt, ntiles, a);
    case 4: return launch_mfma_u<NB, KS, 4, G, false>(s, fmt, ntiles, a);
    default: return launch_mfma_u<NB, KS, 2, G, false>(s, fmt, ntiles, a);
  }
}

template <int NB, int KS>
static hipError_t launch_mfma(hipStream_t s, int fmt, int ntiles, const PassArgs& a, bool batched, bool gather) {
  return gather ? launch_mfma_g<NB, KS, true>(s, fmt, ntiles, a, batched)
                : launch_mfma_g<NB, KS, false>(s, fmt, ntiles, a, batched);
}

template <int FMT, int KS, int U>
static hipError_t launch_slots_k(hipStream_t s, int nunits, int max_slots, const SlotArgs& a) {
  constexpr int NB = 2;
  const size_t shm = (size_t)KS * NB * 2 * 4 * 64 * sizeof(double);
  // few classes of many slots: their 32-slot blocks go to workgroups of their own, up to 64 waves a
  // compute unit (1660 units of four waves, up to 2048 slots: 138 us a pass with one workgroup a unit,
  // 123 with two); with many classes a class has few slots and one workgroup takes them
  const int64_t want = std::max(1, 16384 / (KS * nunits)), most = ((int64_t)max_slots + 16 * NB - 1) / (16 * NB);
  const dim3 g(nunits, (unsigned)std::max<int64_t>(1, std::min(want, most)));
  hipLaunchKernelGGL((k_pass_slots<FMT, KS, U>), g, dim3(64 * KS), shm, s, a);
  return hipGetLastError();
}

template <int KS>
static hipError_t launch_slots_mix(hipStream_t s, int fmt, int nunits, int max_slots, const SlotArgs& a) {
  if (fmt == PF_BF16X3) return launch_slots_k<PF_BF16X3, KS, 1>(s, nunits, max_slots, a);
  switch (prefetch_depth()) {
    case 1: return launch_slots_k<PF_F32, KS, 1>(s, nunits, max_slots, a);
    case 4: return launch_slots_k<PF_F32, KS, 4>(s, nunits, max_slots, a);
    default: return launch_slots_k<PF_F32, KS, 2>(s, nunits, max_slots, a);
  }
}

// ks: waves that split the fibre length (mixed formats).  FP64 sums round at 1e-16 however they are
// split, and four waves are the fastest.
hipError_t launch_pass_slots(hipStream_t s, int fmt, int nunits, int max_slots, int ks, const SlotArgs& a) {
  if (nunits == 0) return hipSuccess;
  if (fmt == PF_F64) return launch_slots_k<PF_F64, 4, 2>(s, nunits, max_slots, a);
  switch (ks) {
    case 1: return launch_slots_mix<1>(s, fmt, nunits, max_slots, a);
    case 2: return launch_slots_mix<2>(s, fmt, nunits, max_slots, a);
    case 4: return launch_slots_mix<4>(s, fmt, nunits, max_slots, a);
    default: return hipErrorInvalidValue;
  }
}

template <int KS, bool B>
static hipError_t launch_gemv(hipStream_t s, int fmt, int ntiles, const PassArgs& a0) {
  PassArgs a = a0;
  if constexpr (B) {
    if (a.persist) {
      a.ntiles = ntiles;
      const void* fn = fmt == PF_F64   ? reinterpret_cast<const void*>(&k_gemv_persist<KS, PF_F64>)
                       : fmt == PF_F32 ? reinterpret_cast<const void*>(&k_gemv_persist<KS, PF_F32>)
                                       : reinterpret_cast<const void*>(&k_gemv_persist<KS, PF_BF16X3>);
      const dim3 grid(persistent_grid(fn, 64 * KS, 0, ntiles));
      if (g_prepare_only) return hipSuccess;
      if (fmt == PF_F64)
        hipLaunchKernelGGL((k_gemv_persist<KS, PF_F64>), grid, dim3(64 * KS), 0, s, a);
      else if (fmt == PF_F32)
        hipLaunchKernelGGL((k_gemv_persist<KS, PF_F32>), grid, dim3(64 * KS), 0, s, a);
      else
        hipLaunchKernelGGL((k_gemv_persist<KS, PF_BF16X3>), grid, dim3(64 * KS), 0, s, a);
      return hipGetLastError();
    }
  }
  if (fmt == PF_F64)
    hipLaunchKernelGGL((k_gemv<KS, PF_F64, B>), dim3(ntiles), dim3(64 * KS), 0, s, a);
  else if (fmt == PF_F32)
    hipLaunchKernelGGL((k_gemv<KS, PF_F32, B>), dim3(ntiles), dim3(64 * KS), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemv<KS, PF_BF16X3, B>), dim3(ntiles), dim3(64 * KS), 0, s, a);
  return hipGetLastError();
}

// single-state orbit tiles of one row block: KS waves, M the layer's largest group rounded up
// to an instantiated size
template <int KS>
static hipError_t launch_gemv_orbit_m(hipStream_t s, int fmt, int ntiles, const PassArgs& a) {
  const int gm = a.orbit_max;
#define LSX_ORBIT_M(M_)                                                                           \
  if (gm <= M_) {                                                                                 \
    if (fmt == PF_F64)                                                                            \
      hipLaunchKernelGGL((k_gemv_orbit<KS, PF_F64, M_>), dim3(ntiles), dim3(64 * KS), 0, s, a);    \
    else if (fmt == PF_F32)                                                                       \
      hipLaunchKernelGGL((k_gemv_orbit<KS, PF_F32, M_>), dim3(ntiles), dim3(64 * KS), 0, s, a);    \
    else                                                                                          \
      hipLaunchKernelGGL((k_gemv_orbit<KS, PF_BF16X3, M_>), dim3(ntiles), dim3(64 * KS), 0, s, a); \
    return hipGetLastError();                                                                     \
  }
  LSX_ORBIT_M(2)
  LSX_ORBIT_M(4)
  LSX_ORBIT_M(6)
  LSX_ORBIT_M(8)
#undef LSX_ORBIT_M
  return hipErrorInvalidValue;
}

// single-state tiles of four row blocks, one row per lane (every storage format): per-fibre
// tiles (orbit = false) or orbit tiles with M the layer's largest group rounded up
template <int KS, int FMT, int M, bool ORB>
static hipError_t launch_gemv_rows_g(hipStream_t s, int ntiles, const PassArgs& a) {
  if (a.in_pos)
    hipLaunchKernelGGL((k_gemv_rows<KS, FMT, M, ORB, true>), dim3(ntiles), dim3(64 * KS), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemv_rows<KS, FMT, M, ORB, false>), dim3(ntiles), dim3(64 * KS), 0, s, a);
  return hipGetLastError();
}

template <int KS, int M, bool ORB>
static hipError_t launch_gemv_rows_m(hipStream_t s, int fmt, int ntiles, const PassArgs& a) {
  if (fmt == PF_F64) return launch_gemv_rows_g<KS, PF_F64, M, ORB>(s, ntiles, a);
  if (fmt == PF_F32) return launch_gemv_rows_g<KS, PF_F32, M, ORB>(s, ntiles, a);
  return launch_gemv_rows_g<KS, PF_BF16X3, M, ORB>(s, ntiles, a);
}

template <int KS>
static hipError_t launch_gemv_rows(hipStream_t s, int fmt, int ntiles, bool orbit, const PassArgs& a) {
  if (!orbit) return launch_gemv_rows_m<KS, 1, false>(s, fmt, ntiles, a);
  if (!a.orbit || a.orbit_max < 1 || a.orbit_max > kOrbitMax || a.wt || a.tcount) return hipErrorInvalidValue;
  const int gm = a.orbit_max;
  if (gm <= 2) return launch_gemv_rows_m<KS, 2, true>(s, fmt, ntiles, a);
  if (gm <= 4) return launch_gemv_rows_m<KS, 4, true>(s, fmt, ntiles, a);
  if (gm <= 6) return launch_gemv_rows_m<KS, 6, true>(s, fmt, ntiles, a);
  return launch_gemv_rows_m<KS, 8, true>(s, fmt, ntiles, a);
}

static hipError_t launch_gemv_orbit(hipStream_t s, int fmt, int ntiles, int ksplit, const PassArgs& a) {
  if (!a.orbit || a.orbit_max < 1 || a.orbit_max > kOrbitMax || a.wt || a.tcount) return hipErrorInvalidValue;
  switch (ksplit) {
    case 1: return launch_gemv_orbit_m<1>(s, fmt, ntiles, a);
    case 2: return launch_gemv_orbit_m<2>(s, fmt, ntiles, a);
    case 4: return launch_gemv_orbit_m<4>(s, fmt, ntiles, a);
    default: return hipErrorInvalidValue;
  }
}

// batched: tile.f is a system index into a.batch and every system has its own W; the
// caller passes gather = whether the systems' in_pos tables are set (uniform per pass)
hipError_t launch_pass(hipStream_t s, int fmt, int W, int ntiles, int nb, int ksplit, const PassArgs& a,
                       bool batched) {
  if (ntiles == 0) return hipSuccess;
  const bool gather = a.in_pos != nullptr;
  if (W == 1) {
    if (batched) return launch_gemv<4, true>(s, fmt, ntiles, a);
    if (ksplit < 0) {  // tiles of four row blocks, one row per lane, -ksplit waves
      const bool orbit = nb == kOrbitNB;
      switch (-ksplit) {
        case 1: return launch_gemv_rows<1>(s, fmt, ntiles, orbit, a);
        case 2: return launch_gemv_rows<2>(s, fmt, ntiles, orbit, a);
        case 4: return launch_gemv_rows<4>(s, fmt, ntiles, orbit, a);
        case 8: return launch_gemv_rows<8>(s, fmt, ntiles, orbit, a);
        default: return hipErrorInvalidValue;
      }
    }
    if (nb == kOrbitNB) return launch_gemv_orbit(s, fmt, ntiles, ksplit, a);
    switch (ksplit) {
      case 1: return launch_gemv<1, false>(s, fmt, ntiles, a);
      case 2: return launch_gemv<2, false>(s, fmt, ntiles, a);
      default: return launch_gemv<4, false>(s, fmt, ntiles, a);
    }
  }
  if (ksplit < 0) {
    if (batched) return hipErrorInvalidValue;
    return launch_rowsplit(s, fmt, ntiles, nb, -ksplit, a);
  }
#define LSX_MFMA_CASE(NB_, KS_) \
  if (nb == NB_ && ksplit == KS_) return launch_mfma<NB_, KS_>(s, fmt, ntiles, a, batched, gather);
  LSX_MFMA_CASE(1, 1)
  LSX_MFMA_CASE(1, 2)
  LSX_MFMA_CASE(1, 4)
  LSX_MFMA_CASE(2, 1)
  LSX_MFMA_CASE(2, 2)
  LSX_MFMA_CASE(2, 4)
  LSX_MFMA_CASE(4, 1)
  LSX_MFMA_CASE(4, 2)
  LSX_MFMA_CASE(4, 4)
#undef LSX_MFMA_CASE
  return hipErrorInvalidValue;
}

hipError_t prepare_persistent(int fmt, int W, int nb, int ksplit, const PassArgs& a) {
  if (!a.persist) return hipSuccess;
  g_prepare_only = true;
  const hipError_t e = launch_pass(nullptr, fmt, W, 1, nb, ksplit, a, true);
  g_prepare_only = false;
  return e;
}

}  // namespace lsx

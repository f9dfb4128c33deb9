// Small systems: every pass of a call in one launch, one workgroup per wavepacket.
//
// The passes of a step couple the rows of a wavepacket but never two wavepackets, so a workgroup
// that holds one column of the state in LDS can run any number of passes with workgroup barriers
// between them, where separate launches cost 2.4 us each (1.5 from a graph) whatever the pass
// does.  Four lanes share a row: lane kl takes the band's columns kl, kl + 4, ... (FP64 / FP32
// propagators) or eight of every 32 (BF16x3), so that sixteen rows read each stored propagator
// chunk in its own order; the four sums are added by shuffles.  The arithmetic is the single-state
// passes': stored entries times the FP64 state, FP64 accumulation, the FP64 diagonal term.
// A pass is a latency chain (descriptor, propagator entries, state from LDS, products, shuffles,
// LDS store, barrier); the next pass's descriptor is loaded before a thread's first row and its
// first entries before the barrier, and a two-pass body whose rows and bands allow it keeps both
// passes' entries in registers (PAIR).
// Tiny chain (N = 53, W = 1, FP64): 5.6 us per Strang step as launches, 2.3 without PAIR, 1.05 with it.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lsx_pass.h"

namespace lsx {

// sum += p x as fused multiply-adds in a fixed order
__device__ __forceinline__ void res_mac(double& yr, double& yi, double pr, double pi, double2 x) {
  yr = __builtin_fma(pr, x.x, yr);
  yr = __builtin_fma(-pi, x.y, yr);
  yi = __builtin_fma(pr, x.y, yi);
  yi = __builtin_fma(pi, x.x, yi);
}

// What a pass needs for one row before its products: descriptor, output position, phase, diagonal
// entry and the first propagator entries.
template <int FMT, int U>
struct ResidentHead {
  using PT = typename std::conditional<FMT == PF_F64, double2, float2>::type;
  ResidentRow r;
  int32_t out;
  double2 ph, dg;
  PT e[U];
};

template <int FMT, bool PAIR>
__global__ __launch_bounds__(1024) void k_resident(ResidentArgs a) {
  constexpr int U = kResidentU;
  using Head = ResidentHead<FMT, U>;
  using PT = typename Head::PT;
  extern __shared__ double2 lds[];
  double2* xa = lds;
  double2* xb = lds + a.N;
  const int t = threadIdx.x, kl = t & 3, row0 = t >> 2, nrow = blockDim.x >> 2;
  const int64_t w = blockIdx.x;
  const int W = a.W;
  for (int p = t; p < a.N; p += blockDim.x) xa[p] = a.X[(int64_t)(a.in_pos ? a.in_pos[p] : p) * W + w];
  // position in the sequence head, body x reps, tail: entry of pass i in a.pass
  int64_t i = a.begin;
  const int64_t tail0 = a.nhead + (int64_t)a.nbody * a.reps;
  int at;
  if (i < a.nhead) at = (int)i;
  else if (i < tail0) at = a.nhead + (int)((i - a.nhead) % a.nbody);
  else at = a.nhead + a.nbody + (int)(i - tail0);
  auto next_at = [&](int64_t j, int c) {  // entry of pass j + 1 when pass j's is c
    if (j + 1 == tail0) return a.nhead + a.nbody;
    if (j + 1 < tail0 && j + 1 > a.nhead && c + 1 == a.nhead + a.nbody) return (int)a.nhead;
    return c + 1;
  };
  // the head of row p in two steps, the second once the descriptor has arrived
  auto load_row = [&](const ResidentPass& d, int p, Head& h) {
    h.r = d.rows[p];
    h.out = d.out_pos ? d.out_pos[p] : p;
  };
  auto load_entries = [&](const ResidentPass& d, Head& h) {
    if (d.ph) h.ph = d.ph[h.r.canon];
    if (FMT != PF_F64) h.dg = d.diag[h.r.d];
    if constexpr (FMT != PF_BF16X3) {
      const PT* P = reinterpret_cast<const PT*>(d.P) + h.r.base + 16 * kl;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u < h.r.n) h.e[u] = P[(int64_t)u * 64];
    }
  };
  // row p of a pass: products, sum over the row's lanes, diagonal term, phase
  auto row_pass = [&](const ResidentPass& d, Head& h, int p) {
    const ResidentRow r = h.r;
    double yr = 0.0, yi = 0.0;
    if constexpr (FMT == PF_BF16X3) {
      const v8u16* P = reinterpret_cast<const v8u16*>(d.P) + r.base + 16 * kl;
      for (int c = 0; c < r.n; ++c) {
        v8u16 pl[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) pl[k] = P[((int64_t)c * 6 + k) * 64];
#pragma unroll
        for (int el = 0; el < 8; ++el) {
          const int k = r.x0 + 32 * c + 8 * kl + el;
          if (k < r.lim)
            res_mac(yr, yi, (double)(bf2f(pl[0][el]) + bf2f(pl[2][el]) + bf2f(pl[4][el])),
                    (double)(bf2f(pl[1][el]) + bf2f(pl[3][el]) + bf2f(pl[5][el])), xa[k]);
        }
      }
    } else {
      auto group = [&](int c) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = r.x0 + 4 * (c + u) + kl;
          if (c + u < r.n && k < r.lim) res_mac(yr, yi, h.e[u].x, h.e[u].y, xa[k]);
        }
      };
      group(0);
      if constexpr (!PAIR) {
        const PT* P = reinterpret_cast<const PT*>(d.P) + r.base + 16 * kl;
        for (int c = U; c < r.n; c += U) {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (c + u < r.n) h.e[u] = P[(int64_t)(c + u) * 64];
          group(c);
        }
      }
    }
    yr += __shfl_xor(yr, 1);
    yi += __shfl_xor(yi, 1);
    yr += __shfl_xor(yr, 2);
    yi += __shfl_xor(yi, 2);
    if (kl == 0) {
      if (FMT != PF_F64) res_mac(yr, yi, h.dg.x, h.dg.y, xa[p]);
      if (d.ph) {
        const double zr = __builtin_fma(h.ph.x, yr, -(h.ph.y * yi));
        yi = __builtin_fma(h.ph.x, yi, h.ph.y * yr);
        yr = zr;
      }
      xb[h.out] = make_double2(yr, yi);
    }
  };
  auto turn = [&]() {
    __syncthreads();
    double2* const s = xa;
    xa = xb;
    xb = s;
  };
  const bool has = row0 < a.N;
  if constexpr (PAIR) {
    // one row per four lanes, every band within U entries a lane: a body of two passes keeps both
    // its heads in registers and reads nothing but LDS
    auto single = [&](int64_t n) {  // n passes one by one
      for (; n > 0; --n, ++i) {
        const ResidentPass d = a.pass[at];
        Head h;
        if (has) {
          load_row(d, row0, h);
          load_entries(d, h);
        }
        if (i == a.begin) __syncthreads();  // the column is in LDS (every thread, so outside the branch)
        if (has) row_pass(d, h, row0);
        turn();
        at = next_at(i, at);
      }
    };
    if (i < a.nhead) single(min(a.end, (int64_t)a.nhead) - i);
    else if (i < a.end && i < tail0 && ((i - a.nhead) & 1)) single(1);
    const int64_t pairs = i < tail0 ? (min(a.end, tail0) - i) / 2 : 0;
    if (pairs > 0) {
      const ResidentPass d0 = a.pass[a.nhead], d1 = a.pass[a.nhead + 1];
      Head h0, h1;
      if (has) {
        load_row(d0, row0, h0);
        load_row(d1, row0, h1);
        load_entries(d0, h0);
        load_entries(d1, h1);
      }
      if (i == a.begin) __syncthreads();
      for (int64_t q = 0; q < pairs; ++q) {
        if (has) row_pass(d0, h0, row0);
        turn();
        if (has) row_pass(d1, h1, row0);
        turn();
      }
      i += 2 * pairs;
      at = i == tail0 ? a.nhead + a.nbody : a.nhead;
    }
    single(a.end - i);
  } else {
    Head cur, nxt;
    if (has) {
      load_row(a.pass[at], row0, nxt);
      load_entries(a.pass[at], nxt);
    }
    __syncthreads();
    for (; i < a.end; ++i) {
      const ResidentPass d = a.pass[at];
      const int nat = i + 1 < a.end ? next_at(i, at) : at;
      cur = nxt;
      if (has) load_row(a.pass[nat], row0, nxt);
      for (int p = row0; p < a.N; p += nrow) {
        if (p != row0) {
          load_row(d, p, cur);
          load_entries(d, cur);
        }
        row_pass(d, cur, p);
      }
      if (has) load_entries(a.pass[nat], nxt);
      turn();
      at = nat;
    }
  }
  for (int p = t; p < a.N; p += blockDim.x) a.Y[(int64_t)p * W + w] = xa[p];
}

hipError_t launch_resident(hipStream_t s, int fmt, const ResidentArgs& a, bool pair) {
  const int threads = a.N * 4 >= 1024 ? 1024 : round_up(a.N * 4, 64);
  const size_t shm = (size_t)2 * a.N * sizeof(double2);
  const dim3 grid(a.W), block(threads);
  if (fmt == PF_F64) {
    if (pair) hipLaunchKernelGGL((k_resident<PF_F64, true>), grid, block, shm, s, a);
    else hipLaunchKernelGGL((k_resident<PF_F64, false>), grid, block, shm, s, a);
  } else if (fmt == PF_F32) {
    if (pair) hipLaunchKernelGGL((k_resident<PF_F32, true>), grid, block, shm, s, a);
    else hipLaunchKernelGGL((k_resident<PF_F32, false>), grid, block, shm, s, a);
  } else {
    hipLaunchKernelGGL((k_resident<PF_BF16X3, false>), grid, block, shm, s, a);
  }
  return hipGetLastError();
}

}  // namespace lsx

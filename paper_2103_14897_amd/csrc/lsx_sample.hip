// Stochastic steps of liblsx: the semi-implicit step (Alg. 1) and its random batch form
// (Alg. 4) as one neighbour-stencil kernel, per-column fibre sampling (subsets without
// replacement, importance draws from a proposal), compaction of the sampled fibres, and the
// per-fibre features and increment norms the proposal is trained on.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cstdlib>

#include "lsx_block.h"
#include "lsx_internal.h"

namespace lsx {

// ---------------------------------------------------------------- semi-implicit / random batch
// out[i][w] = (x - i tau (a1 (V^1 x)_i + a2 (V^2 x)_i)) / (1 + i tau |K_i|^2 / 2), where
// (V^j x)_i = sum_p v_p x[nbr_j(i, p)] (the layer-j potential inside row i's fibre) and
// a_j = wt_j[fibre_j(i)][w] (1 when wt_j is null: Alg. 1).  One thread per (row, column).
//
// Cache blocking: every neighbour row is read again by nv other rows, the layer-1 ones
// (m - p, n) from far away in canonical order.  Workgroup b runs on XCD b % 8, so XCD x
// takes part x of the rows (Sweep), and sweeps it in blocks of CW columns: the rows
// between a neighbour's first and last use then fit in that XCD's own L2, which the output of a
// large state does not displace (non-temporal stores).  Twisted bilayer, N = 398821, W = 128: 0.93
// ms a step in contiguous slabs with 8-column sweeps and ordinary stores, 0.87 ms now, 1.9 of 4.9
// TB/s of state read and written once; L2 read misses (34 to 22 million lines, 2.85 GB) bound it.
// Measured and not used: the next row's indices loaded ahead of the current row's values (0.98 ms).
//
// Stencil sizes NV1, NV2 are compile-time for the common cases (1D cosine: 2, 2D first shell:
// 6) so every neighbour index and value is loaded before any is used; a missing neighbour
// (index -1) reads a zero row instead of branching.  NV1 = 0 selects runtime loops.
template <int NVC>
__device__ __forceinline__ void si_stencil(int64_t i, int w, int W, int nv, const int32_t* __restrict__ nbr,
                                           const double2* __restrict__ v, const double2* __restrict__ X,
                                           const double2* __restrict__ zero, double& sr, double& si) {
  if (NVC > 0) {
    int j[8];
    double2 y[8];
#pragma unroll
    for (int p = 0; p < NVC; ++p) j[p] = nbr[i * NVC + p];
#pragma unroll
    for (int p = 0; p < NVC; ++p) y[p] = *(j[p] >= 0 ? X + (int64_t)j[p] * W + w : zero);
#pragma unroll
    for (int p = 0; p < NVC; ++p) {
      const double2 c = v[p];
      sr += c.x * y[p].x - c.y * y[p].y;
      si += c.x * y[p].y + c.y * y[p].x;
    }
  } else {
    for (int p = 0; p < nv; ++p) {
      const int jj = nbr[i * nv + p];
      const double2 y = *(jj >= 0 ? X + (int64_t)jj * W + w : zero), c = v[p];
      sr += c.x * y.x - c.y * y.y;
      si += c.x * y.y + c.y * y.x;
    }
  }
}

template <int NV1, int NV2>
__global__ __launch_bounds__(256) void k_si_step(Sweep sweep, int W, int CW, double tau, const double* __restrict__ K2,
                                                 int nv1, const int32_t* __restrict__ nbr1,
                                                 const double2* __restrict__ v1, const double* __restrict__ wt1,
                                                 const int32_t* __restrict__ fid1, int nv2,
                                                 const int32_t* __restrict__ nbr2, const double2* __restrict__ v2,
                                                 const double* __restrict__ wt2, const int32_t* __restrict__ fid2,
                                                 const double2* __restrict__ X, double2* __restrict__ Y,
                                                 const double2* __restrict__ zero) {
  const int xcd = blockIdx.x & 7;
  const int G = gridDim.x >> 3, lb = blockIdx.x >> 3;
  const int r0 = sweep.start[xcd], r1 = sweep.start[xcd + 1];
  const int rpi = 256 / CW;  // rows per workgroup iteration
  const int tr = threadIdx.x / CW, tc = threadIdx.x - tr * CW;
  for (int cb = (int)blockIdx.y * CW; cb < W; cb += (int)gridDim.y * CW) {
    const int w = cb + tc;
    if (w >= W) continue;
    for (int k = r0 + lb * rpi + tr; k < r1; k += G * rpi) {
      const int64_t i = sweep.order ? sweep.order[k] : k;
      double s1r = 0.0, s1i = 0.0, s2r = 0.0, s2i = 0.0;
      si_stencil<NV1>(i, w, W, nv1, nbr1, v1, X, zero, s1r, s1i);
      si_stencil<NV2>(i, w, W, nv2, nbr2, v2, X, zero, s2r, s2i);
      const double a1 = wt1 ? wt1[(int64_t)fid1[i] * W + w] : 1.0;
      const double a2 = wt2 ? wt2[(int64_t)fid2[i] * W + w] : 1.0;
      const double2 x = X[i * W + w];
      // z = x - i tau (a1 s1 + a2 s2)
      const double zr = x.x + tau * (a1 * s1i + a2 * s2i);
      const double zi = x.y - tau * (a1 * s1r + a2 * s2r);
      // z / (1 + i b) = z (1 - i b) / (1 + b^2)
      const double b = 0.5 * tau * K2[i];
      const double den = 1.0 + b * b;
      const double2 out = make_double2((zr + b * zi) / den, (zi - b * zr) / den);
      if (sweep.order) {  // empty compiler barriers keep the two branches' stores apart
        asm volatile("" ::: "memory");
        __builtin_nontemporal_store(out.x, &Y[i * W + w].x);
        __builtin_nontemporal_store(out.y, &Y[i * W + w].y);
        asm volatile("" ::: "memory");
      } else {
        Y[i * W + w] = out;
      }
    }
  }
}

// ---------------------------------------------------------------- per-column sampling
// Random subset of p of the nf fibres for column w = blockIdx.x (Alg. 4): partial
// Fisher-Yates with the uniforms u[w][0..p-1] (position s swaps with
// s + floor(u (nf - s))), weight nf/p on the chosen fibres, 0 elsewhere; wt is [nf][W].
__global__ __launch_bounds__(256) void k_subset_weights(int nf, int W, int p, int ustride, const double* u,
                                                        double* wt) {
  extern __shared__ int32_t perm[];
  const int w = blockIdx.x;
  for (int f = threadIdx.x; f < nf; f += blockDim.x) perm[f] = f;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double* uw = u + (int64_t)w * ustride;
    for (int s = 0; s < p; ++s) {
      int j = s + (int)floor(uw[s] * (double)(nf - s));
      j = j < nf - 1 ? j : nf - 1;
      const int tmp = perm[s];
      perm[s] = perm[j];
      perm[j] = tmp;
    }
  }
  __syncthreads();
  for (int f = threadIdx.x; f < nf; f += blockDim.x) wt[(int64_t)f * W + w] = 0.0;
  __syncthreads();
  const double g = (double)nf / (double)p;
  for (int s = threadIdx.x; s < p; s += blockDim.x) wt[(int64_t)perm[s] * W + w] = g;
}

// Importance draws for column w = blockIdx.x: q = (1 - eps) softmax(z[w]) + eps / nf
// (uniform when z is null), cdf = running sum of q in fibre order, draw s lands on the
// first fibre whose cdf exceeds u[w][s] (the last fibre if none), and adds 1 / (p q_f)
// to that fibre's weight.  All draws of a fibre add the same value, so the sum does not
// depend on their order.  Dynamic LDS: 3 * nf doubles.  256 threads.
__global__ __launch_bounds__(256) void k_sample_weights(int nf, int W, int p, int ustride, const double* u,
                                                        const float* z, double eps, double* wt) {
  extern __shared__ double sm[];
  double* q = sm;
  double* cdf = sm + nf;
  double* acc = sm + 2 * nf;
  __shared__ double red[256];
  const int w = blockIdx.x;
  if (z) {
    const float* zw = z + (int64_t)w * nf;
    double mx = -INFINITY;
    for (int f = threadIdx.x; f < nf; f += blockDim.x) mx = fmax(mx, (double)zw[f]);
    mx = block_max(mx, red);
    double s = 0.0;
    for (int f = threadIdx.x; f < nf; f += blockDim.x) {
      const double e = exp((double)zw[f] - mx);
      q[f] = e;
      s += e;
    }
    s = block_sum(s, red);
    for (int f = threadIdx.x; f < nf; f += blockDim.x) q[f] = (1.0 - eps) * q[f] / s + eps / nf;
  } else {
    for (int f = threadIdx.x; f < nf; f += blockDim.x) q[f] = 1.0 / nf;
  }
  for (int f = threadIdx.x; f < nf; f += blockDim.x) acc[f] = 0.0;
  __syncthreads();
  // Summed in fibre order by one thread, which fixes every draw.  Sixteen entries are read before
  // they are added: with one read and one write an entry, the LDS latency of each was the kernel's
  // time (889 fibres, 128 wavepackets: 39 us, now 19).
  if (threadIdx.x == 0) {
    double c = 0.0;
    int f = 0;
    for (; f + 16 <= nf; f += 16) {
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = q[f + i];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        c += v[i];
        v[i] = c;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) cdf[f + i] = v[i];
    }
    for (; f < nf; ++f) {
      c += q[f];
      cdf[f] = c;
    }
  }
  __syncthreads();
  const double* uw = u + (int64_t)w * ustride;
  for (int s = threadIdx.x; s < p; s += blockDim.x) {
    const double us = uw[s];
    int lo = 0, hi = nf;  // first f with cdf[f] > us
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cdf[mid] > us)
        hi = mid;
      else
        lo = mid + 1;
    }
    const int f = lo < nf ? lo : nf - 1;
    atomicAdd(&acc[f], 1.0 / ((double)p * q[f]));
  }
  __syncthreads();
  for (int f = threadIdx.x; f < nf; f += blockDim.x) wt[(int64_t)f * W + w] = acc[f];
}

// Column list of every fibre: the columns (in increasing order) whose weight on it is
// nonzero.  One wave per fibre compacts 64 columns at a time with a ballot.
__global__ __launch_bounds__(256) void k_fibre_cols(int nf, int W, const double* wt, int32_t* cols, int32_t* ncols) {
  const int f = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (f >= nf) return;
  int base = 0;
  for (int w0 = 0; w0 < W; w0 += 64) {
    const int w = w0 + lane;
    const bool on = w < W && wt[(int64_t)f * W + w] != 0.0;
    const unsigned long long m = __ballot(on);
    const int pos = __popcll(m & ((1ull << lane) - 1ull));
    if (on) cols[(int64_t)f * W + base + pos] = w;
    base += __popcll(m);
  }
  if (lane == 0) ncols[f] = base;
}

// Slots of the classes (SlotBuild): the fibres' column counts summed in class order give every
// fibre's slot offset inside its class and the class sizes; class sizes times fibre lengths summed
// over the classes give the places of the compacted columns.  One workgroup of 1024 threads, dynamic
// LDS (nf + 1) int32.
__global__ __launch_bounds__(1024) void k_slot_scan(SlotBuild b) {
  extern __shared__ int32_t S[];  // S[q]: slots before fibre qfib[q]
  __shared__ int64_t scan[1024];
  const int t = threadIdx.x;
  auto block_scan = [&](int64_t mine) {  // exclusive sum over the threads
    scan[t] = mine;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int64_t v = t >= o ? scan[t - o] : 0;
      __syncthreads();
      scan[t] += v;
      __syncthreads();
    }
    const int64_t before = scan[t] - mine;
    __syncthreads();
    return before;
  };
  const int fc = (b.nf + 1023) / 1024, q0 = min(b.nf, t * fc), q1 = min(b.nf, q0 + fc);
  int mine = 0;
  for (int q = q0; q < q1; ++q) mine += b.ncols[b.qfib[q]];
  int at = (int)block_scan(mine);
  for (int q = q0; q < q1; ++q) {
    S[q] = at;
    at += b.ncols[b.qfib[q]];
  }
  if (q1 == b.nf) S[b.nf] = at;  // every thread past the end has the same sum
  __syncthreads();
  for (int q = q0; q < q1; ++q) b.off[b.qfib[q]] = S[q] - S[b.cstart[b.fcls[b.qfib[q]]]];
  const int cc = (b.nc + 1023) / 1024, c0 = min(b.nc, t * cc), c1 = min(b.nc, c0 + cc);
  int64_t elems = 0;
  for (int c = c0; c < c1; ++c) elems += (int64_t)b.clen[c] * (S[b.cstart[c + 1]] - S[b.cstart[c]]);
  int64_t xat = block_scan(elems);
  for (int c = c0; c < c1; ++c) {
    const int n = S[b.cstart[c + 1]] - S[b.cstart[c]];
    b.n[c] = n;
    b.sbase[c] = S[b.cstart[c]];
    b.xbase[c] = xat;
    xat += (int64_t)b.clen[c] * n;
  }
}

// Compacted columns and slots of fibre f = blockIdx.x; workgroup y takes every gridDim.y-th share of
// its elements, so that the reads of a fibre (one 16-byte entry per row and drawn wavepacket, each in
// a line of its own) are in flight together (889 fibres, 2048 drawn pairs: 42 us with one, 32 with four).
__global__ __launch_bounds__(256) void k_slot_gather(SlotBuild b) {
  const int f = blockIdx.x, nc = b.ncols[f];
  if (nc == 0) return;
  const int c = b.fcls[f], n = b.n[c], off = b.off[f];
  const int r0 = b.ptr[f], L = b.ptr[f + 1] - r0;
  const int32_t* cols = b.cols + (int64_t)f * b.W;
  if (blockIdx.y == 0)
    for (int s = threadIdx.x; s < nc; s += blockDim.x) {
      Slot sl;
      sl.r0 = r0;
      sl.w = cols[s];
      sl.g = b.wt[(int64_t)f * b.W + sl.w];
      b.slot[b.sbase[c] + off + s] = sl;
    }
  double2* out = b.Xc + b.xbase[c] + off;
  // thread t takes elements t, t + nt, ... of the [L][nc] block, stepping (row, slot) along
  const int t = blockIdx.y * blockDim.x + threadIdx.x, nt = gridDim.y * blockDim.x;
  const int dk = nt / nc, ds = nt - dk * nc;
  int s = t % nc;
  for (int k = t / nc; k < L;) {
    const int64_t row = b.pos ? b.pos[r0 + k] : r0 + k;
    double2 x = b.X[row * b.W + cols[s]];
    if (b.pend) {
      const double2 h = b.pend[row];
      x = make_double2(h.x * x.x - h.y * x.y, h.x * x.y + h.y * x.x);
    }
    out[(int64_t)k * n + s] = x;
    k += dk;
    s += ds;
    if (s >= nc) {
      s -= nc;
      ++k;
    }
  }
}

// Tile offsets of a single state's sampled fibres (weight nonzero): ceil(L_f / 16) row blocks
// each; off = exclusive scan in fibre order.  One workgroup of 1024 threads; thread t scans fibres
// [t chunk, (t + 1) chunk).
__global__ __launch_bounds__(1024) void k_scan_tiles(int nf, const double* wt, const int32_t* ptr, int32_t* off,
                                                     int32_t* count) {
  __shared__ int32_t scan[1024];
  const int t = threadIdx.x;
  const int chunk = (nf + 1023) / 1024;
  const int f0 = min(nf, t * chunk), f1 = min(nf, f0 + chunk);
  int mine = 0;
  for (int f = f0; f < f1; ++f) mine += wt[f] != 0.0 ? (ptr[f + 1] - ptr[f] + 15) / 16 : 0;
  scan[t] = mine;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {  // inclusive Hillis-Steele scan
    const int v = t >= o ? scan[t - o] : 0;
    __syncthreads();
    scan[t] += v;
    __syncthreads();
  }
  int pos = scan[t] - mine;
  for (int f = f0; f < f1; ++f) {
    off[f] = pos;
    pos += wt[f] != 0.0 ? (ptr[f + 1] - ptr[f] + 15) / 16 : 0;
  }
  if (t == 1023) *count = scan[1023];
}

// Tiles of sampled fibre f = blockIdx.x at off[f], one per row block, each with its row block's
// band when the band table is given (else the whole fibre).
__global__ __launch_bounds__(64) void k_emit_tiles(const double* wt, const int32_t* ptr, const int64_t* poff,
                                                   const int32_t* d0, const int32_t* bptr, const int32_t* band,
                                                   const int32_t* off, TileDesc* out) {
  const int f = blockIdx.x;
  if (wt[f] == 0.0) return;
  const int r0 = ptr[f], L = ptr[f + 1] - r0;
  const int n = (L + 15) / 16;
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    TileDesc t;
    t.r0 = r0;
    t.L = L;
    t.rb = k;
    t.wb = 0;
    t.poff = poff ? poff[f] : 0;
    t.f = f;
    t.d0 = d0 ? d0[f] : r0;
    t.k0 = band ? band[2 * (bptr[f] + t.rb)] : 0;
    t.k1 = band ? band[2 * (bptr[f] + t.rb) + 1] : kBandEnd;
    t.bb = -1;
    t.pad_ = 0;
    out[off[f] + k] = t;
  }
}

// Copies the rows of every listed tile of a single state from src to dst (through pos when set);
// tiles at or past *count are skipped.  16 threads per tile.
__global__ __launch_bounds__(256) void k_copy_rows(const TileDesc* tiles, const int32_t* count, const int32_t* pos,
                                                   const double2* src, double2* dst) {
  const int ti = blockIdx.x * 16 + (threadIdx.x >> 4);
  if (ti >= *count) return;
  const TileDesc t = tiles[ti];
  const int a = 16 * t.rb + (threadIdx.x & 15);
  if (a >= t.L) return;
  const int64_t row = pos ? pos[t.r0 + a] : t.r0 + a;
  dst[row] = src[row];
}

// ---------------------------------------------------------------- training data
// b[w][f] = sum over the fibre's rows of |Y - X|^2 (one workgroup per fibre)
__global__ __launch_bounds__(256) void k_fibre_incr(const int32_t* ptr, const int32_t* rows, int nf, int W,
                                                    const double2* X, const double2* Y, double* out) {
  __shared__ double red[256];
  const int f = blockIdx.x;
  const int r0 = ptr[f], L = ptr[f + 1] - r0;
  const int WB = W < 256 ? W : 256;
  const int S = 256 / WB;
  const int tid = threadIdx.x;
  for (int w0 = 0; w0 < W; w0 += WB) {
    const int w = w0 + tid % WB, s = tid / WB;
    double acc = 0.0;
    if (w < W && s < S)
      for (int a = s; a < L; a += S) {
        const int64_t e = (int64_t)rows[r0 + a] * W + w;
        const double dr = Y[e].x - X[e].x, di = Y[e].y - X[e].y;
        acc += dr * dr + di * di;
      }
    red[tid] = acc;
    __syncthreads();
    if (tid < WB && w0 + tid < W) {
      double sum = 0.0;
      for (int j = 0; j < S; ++j) sum += red[j * WB + tid];
      out[(int64_t)(w0 + tid) * nf + f] = sum;
    }
    __syncthreads();
  }
}

// X[w][f][:] = (shift / Kmax (d), |shift / Kmax|^2, log10(max(mass, 1e-30)) / 10, layer sign)
// from sfeat[f] = (shift / Kmax, |shift / Kmax|^2) and mass [nf][W].
__global__ __launch_bounds__(256) void k_features(int nf, int W, int d, const double* sfeat, const double* mass,
                                                  float sign, float* X) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)nf * W) return;
  const int w = (int)(e / nf), f = (int)(e - (int64_t)w * nf);
  const int nin = d + 3;
  float* x = X + e * nin;
  for (int k = 0; k <= d; ++k) x[k] = (float)sfeat[f * (d + 1) + k];
  x[d + 1] = (float)(log10(fmax(mass[(int64_t)f * W + w], 1e-30)) / 10.0);
  x[d + 2] = sign;
}

// ================================================================ launchers
static unsigned grid_for(int64_t n, int64_t cap) {
  const int64_t g = (n + 255) / 256;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

// Whether a semi-implicit step takes the row parts (Sweep::order) in sweeps of up to 32 columns with
// non-temporal output, or slabs of the canonical order in sweeps of 8 with ordinary stores.  The state and
// its output stay in the 256 MB last-level cache up to about 144 MB each, and there ordinary stores are
// the faster ones; beyond it the parts are, where most lanes of their sweeps have a column.  Rows of a
// number of columns that is no multiple of 8 do not fill whole lines, and their 8-column sweeps share a
// line each: there the parts pay at almost any size.  Microseconds a step, slabs / parts, N = 58837, 150193
// and 398821: W = 16 14.0 / 15.4, 28.7 / 34.1, 77 / 84; W = 48 36.5 / 47.6, 85 / 118, 312 / 342; W = 64 46.7 /
// 51.4, 140 / 134, 423 / 397; W = 128 95 / 101, 303 / 290, 842 / 784.  N = 150193 and 398821: W = 31 86 / 65,
// 335 / 193; W = 127 515 / 345, 1728 / 964; W = 36 80 / 122, 316 / 350.  Every element is summed alike on both
// ways.
static bool si_parts(int64_t N, int W) {
  const int cw = W > 16 ? kSweepCW : 16, blocks = (W + cw - 1) / cw;
  const double bytes = 16.0 * (double)N * W, lanes = (double)W / (cw * blocks);
  if (W % 8 == 0) return W >= kSweepCW && bytes >= 144e6 && lanes >= 0.9;
  return W > 8 && (W < 16 || lanes >= 0.75 || (W % 4 != 0 && bytes >= (W < kSweepCW ? 60e6 : 96e6)));
}

hipError_t launch_si_step(hipStream_t s, const Sweep& rows, int W, double tau, const double* K2, int nv1,
                          const int32_t* nbr1, const double2* v1, const double* wt1, const int32_t* fid1, int nv2,
                          const int32_t* nbr2, const double2* v2, const double* wt2, const int32_t* fid2,
                          const double2* X, double2* Y, const double2* zero) {
  const int64_t N = rows.start[8];
  if (N == 0) return hipSuccess;
  Sweep sweep = rows;
  if (sweep.order && !si_parts(N, W)) {
    sweep.order = nullptr;
    for (int x = 0; x <= 8; ++x) sweep.start[x] = (int32_t)std::min(N, x * ((N + 7) / 8));
  }
  // column block: LSX_SI_CW (1..256, a power of two) or the sweep's; 256 workgroups per XCD
  static const int cw_env = [] {
    const char* v = std::getenv("LSX_SI_CW");
    const int x = v ? std::atoi(v) : 0;
    return (x >= 1 && x <= 256 && (x & (x - 1)) == 0) ? x : 0;
  }();
  int CW = cw_env ? cw_env : sweep.order ? kSweepCW : 8;
  while (CW > 1 && CW / 2 >= W) CW /= 2;  // narrow states: no idle lanes beyond W
  int64_t rows_per_xcd = 0;
  for (int x = 0; x < 8; ++x) rows_per_xcd = std::max<int64_t>(rows_per_xcd, sweep.start[x + 1] - sweep.start[x]);
  const int64_t G = std::min<int64_t>(256, std::max<int64_t>(1, (rows_per_xcd * CW + 255) / 256));
  // few rows: the column blocks go to workgroups of their own, up to one a CU (random batch step of N = 79,
  // W = 128: 28 to 11 us); the elements are the same
  const int64_t ny = std::max<int64_t>(1, std::min<int64_t>((W + CW - 1) / CW, 256 / (8 * G)));
  const dim3 grid((unsigned)(8 * G), (unsigned)ny);
  if (nv1 == 2 && nv2 == 2)
    hipLaunchKernelGGL((k_si_step<2, 2>), grid, dim3(256), 0, s, sweep, W, CW, tau, K2, nv1, nbr1, v1, wt1, fid1, nv2,
                       nbr2, v2, wt2, fid2, X, Y, zero);
  else if (nv1 == 6 && nv2 == 6)
    hipLaunchKernelGGL((k_si_step<6, 6>), grid, dim3(256), 0, s, sweep, W, CW, tau, K2, nv1, nbr1, v1, wt1, fid1, nv2,
                       nbr2, v2, wt2, fid2, X, Y, zero);
  else
    hipLaunchKernelGGL((k_si_step<0, 0>), grid, dim3(256), 0, s, sweep, W, CW, tau, K2, nv1, nbr1, v1, wt1, fid1, nv2,
                       nbr2, v2, wt2, fid2, X, Y, zero);
  return hipGetLastError();
}

hipError_t launch_subset_weights(hipStream_t s, int nf, int W, int p, int ustride, const double* u, double* wt) {
  hipLaunchKernelGGL(k_subset_weights, dim3(W), dim3(256), (size_t)nf * sizeof(int32_t), s, nf, W, p, ustride, u,
                     wt);
  return hipGetLastError();
}

hipError_t launch_sample_weights(hipStream_t s, int nf, int W, int p, int ustride, const double* u, const float* z,
                                 double eps, double* wt) {
  hipLaunchKernelGGL(k_sample_weights, dim3(W), dim3(256), (size_t)3 * nf * sizeof(double), s, nf, W, p, ustride,
                     u, z, eps, wt);
  return hipGetLastError();
}

hipError_t launch_slots(hipStream_t s, const SlotBuild& b) {
  if (b.nf == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fibre_cols, dim3((b.nf + 3) / 4), dim3(256), 0, s, b.nf, b.W, b.wt, b.cols, b.ncols);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_slot_scan, dim3(1), dim3(1024), (size_t)(b.nf + 1) * sizeof(int32_t), s, b);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_slot_gather, dim3(b.nf, 4), dim3(256), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_sampled_tiles(hipStream_t s, int nf, const double* wt, const int32_t* ptr, const int64_t* poff,
                                const int32_t* d0, const int32_t* bptr, const int32_t* band, int32_t* off,
                                TileDesc* tiles, int32_t* count) {
  if (nf == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(1024), 0, s, nf, wt, ptr, off, count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_emit_tiles, dim3(nf), dim3(64), 0, s, wt, ptr, poff, d0, bptr, band, off, tiles);
  return hipGetLastError();
}

hipError_t launch_copy_rows(hipStream_t s, int ntiles, const TileDesc* tiles, const int32_t* count,
                            const int32_t* pos, const double2* src, double2* dst) {
  if (ntiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_rows, dim3((ntiles + 15) / 16), dim3(256), 0, s, tiles, count, pos, src, dst);
  return hipGetLastError();
}

hipError_t launch_fibre_incr(hipStream_t s, int nf, const int32_t* ptr, const int32_t* rows, int W,
                             const double2* X, const double2* Y, double* out) {
  if (nf == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fibre_incr, dim3(nf), dim3(256), 0, s, ptr, rows, nf, W, X, Y, out);
  return hipGetLastError();
}

hipError_t launch_features(hipStream_t s, int nf, int W, int d, const double* sfeat, const double* mass,
                           float sign, float* X) {
  const int64_t n = (int64_t)nf * W;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, nf, W, d, sfeat, mass, sign,
                     X);
  return hipGetLastError();
}

}  // namespace lsx

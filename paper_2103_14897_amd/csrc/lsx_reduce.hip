// Elementwise and reduction kernels of liblsx: the kinetic phase, mass, energy and fibre masses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "lsx_internal.h"

namespace lsx {

// ---------------------------------------------------------------- kinetic phase
__global__ void k_phase_table(int64_t N, const double* K2, double scale, double2* ph) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) {
    double s, c;
    sincos(scale * K2[i], &s, &c);
    ph[i] = make_double2(c, -s);
  }
}

// Thread (r, w) of a workgroup takes column w (and w + TW, ...) of rows r, r + RPB, ... of a
// grid-stride sweep, TW = W rounded up to a power of two (at most 256), RPB = 256 / TW: no
// per-element index division, and every row's phase is loaded once per thread.
__global__ __launch_bounds__(256) void k_phase_apply(int64_t N, int W, int TW, const double2* __restrict__ ph,
                                                     double2* __restrict__ c) {
  const int rpb = 256 / TW;
  const int r = threadIdx.x / TW, w0 = threadIdx.x - r * TW;
  for (int64_t i = (int64_t)blockIdx.x * rpb + r; i < N; i += (int64_t)gridDim.x * rpb) {
    const double2 p = ph[i];
    for (int w = w0; w < W; w += TW) {
      const double2 x = c[i * W + w];
      c[i * W + w] = make_double2(p.x * x.x - p.y * x.y, p.x * x.y + p.y * x.x);
    }
  }
}

// ---------------------------------------------------------------- grouped copies
// A batch's results after an odd number of passes, every system's array in one launch instead of
// one copy each (16 chains of W = 16: 353 to 326 us for 20 steps).
__global__ __launch_bounds__(256) void k_copy_home(const CopyItem* items) {
  const CopyItem it = items[blockIdx.y];
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < it.elems; e += (int64_t)gridDim.x * 256)
    it.to[e] = it.from[e];
}

// A single state's rows in another order: dst[p] = src[pos[p]].
__global__ __launch_bounds__(256) void k_gather_rows(int64_t N, const int32_t* pos, const double2* src, double2* dst) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p < N) dst[p] = src[pos[p]];
}

// ---------------------------------------------------------------- FP64 reductions
// Mass sum_i |c_iw|^2 and energy sum_i 1/2 |K_i|^2 |c_iw|^2 + Re conj(c_iw) (V c)_iw of every
// column, as partial sums of one workgroup's rows.  V is Hermitian, so the terms of a coefficient
// and of its partner at the opposite index have equal real parts once summed over the rows: one
// term per pair (EnergyTerm) reads half the neighbours of the stencil.
//
// Bound by the neighbour reads: each row is read again by every term, the first layers' from far
// away.  As in the semi-implicit step, XCD x (workgroup b runs on XCD b % 8) takes part x of the
// rows (Sweep) and sweeps it in blocks of CW columns, so that those reads hit its L2; a
// thread loads the indices, then the values, of up to kTermsPerLoad terms together.  Twisted
// bilayer, N = 398821, W = 128: mass and energy 2.48 ms as separate sweeps of whole rows over all
// twelve neighbours, 0.73 ms as one sweep over six (mass alone 0.19 ms both ways).
constexpr int kReduceThreads = 512;
constexpr int kTermsPerLoad = kEnergyTermGroup;
template <bool MASS, bool ENERGY>
__global__ __launch_bounds__(kReduceThreads) void k_reduce_partial(ReduceArgs a) {
  __shared__ double red[2][kReduceThreads / 64][64];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nx = (int)gridDim.x >= 64 ? 8 : 1;  // a small grid takes the parts as one
  const int x = b % nx, lb = b / nx;
  const int G = ((int)gridDim.x - x + nx - 1) / nx;  // workgroups of this part
  const int r0 = nx == 8 ? a.sweep.start[x] : 0, r1 = nx == 8 ? a.sweep.start[x + 1] : a.sweep.start[8];
  const int rpi = kReduceThreads / a.CW;
  const int tr = threadIdx.x / a.CW, tc = threadIdx.x - tr * a.CW;
  const int W = a.W;
  for (int cb = (int)blockIdx.y * a.CW; cb < W; cb += (int)gridDim.y * a.CW) {
    const int w = cb + tc;
    const bool ok = w < W;
    double am = 0.0, ae = 0.0;
    for (int k = r0 + lb * rpi + tr; ok && k < r1; k += G * rpi) {
      const int64_t i = a.sweep.order ? a.sweep.order[k] : k;
      const double2 c = a.c[i * W + w];
      const double m2 = c.x * c.x + c.y * c.y;
      if (MASS) am += m2;
      if (ENERGY) {
        double hr = 0.0, hi = 0.0;
        for (int t0 = 0; t0 < a.nterms; t0 += kTermsPerLoad) {
          int32_t j[kTermsPerLoad];
          double2 y[kTermsPerLoad];
#pragma unroll
          for (int t = 0; t < kTermsPerLoad; ++t) {
            const EnergyTerm e = a.terms[t0 + t];  // the list is padded to whole groups
            j[t] = e.nbr[i * e.nv + e.col];
          }
#pragma unroll
          for (int t = 0; t < kTermsPerLoad; ++t) y[t] = *(j[t] >= 0 ? a.c + (int64_t)j[t] * W + w : a.zero);
#pragma unroll
          for (int t = 0; t < kTermsPerLoad; ++t) {
            const double2 v = a.terms[t0 + t].v;
            hr += v.x * y[t].x - v.y * y[t].y;
            hi += v.x * y[t].y + v.y * y[t].x;
          }
        }
        ae += (0.5 * a.K2[i] + a.v0) * m2 + (c.x * hr + c.y * hi);
      }
    }
    // sum over the rows of a column: lanes CW apart, then the waves in order
    for (int o = a.CW; o < 64; o <<= 1) {
      if (MASS) am += __shfl_xor(am, o);
      if (ENERGY) ae += __shfl_xor(ae, o);
    }
    if (lane < a.CW) {
      red[0][wave][lane] = am;
      red[1][wave][lane] = ae;
    }
    __syncthreads();
    const int tw = threadIdx.x;
    if (tw < a.CW && cb + tw < W) {
      double sm = 0.0, se = 0.0;
      for (int k = 0; k < kReduceThreads / 64; ++k) {
        sm += red[0][k][tw];
        se += red[1][k][tw];
      }
      if (MASS) a.pmass[(int64_t)b * W + cb + tw] = sm;
      if (ENERGY) a.penergy[(int64_t)b * W + cb + tw] = se;
    }
    __syncthreads();
  }
}

// out[w] = sum over the workgroups of partial[b][w]: eight columns per workgroup, 32 threads
// per column each taking every 32nd partial, then a fixed-order sum
__global__ __launch_bounds__(256) void k_reduce_final(int nblocks, int W, const double* partial, double* out) {
  __shared__ double red[32][8];
  const int tc = threadIdx.x & 7, tr = threadIdx.x >> 3;
  const int w = blockIdx.x * 8 + tc;
  double s = 0.0;
  if (w < W)
    for (int b = tr; b < nblocks; b += 32) s += partial[(int64_t)b * W + w];
  red[tr][tc] = s;
  __syncthreads();
  if (tr == 0 && w < W) {
    double t = 0.0;
    for (int k = 0; k < 32; ++k) t += red[k][tc];
    out[w] = t;
  }
}

__global__ __launch_bounds__(256) void k_fibre_mass(const int32_t* ptr, const int32_t* rows, int W,
                                                    const double2* c, double* out) {
  __shared__ double red[256];
  const int f = blockIdx.x;
  const int r0 = ptr[f], L = ptr[f + 1] - r0;
  const int WB = W < 256 ? W : 256;
  const int S = 256 / WB;
  const int tid = threadIdx.x;
  for (int w0 = 0; w0 < W; w0 += WB) {
    const int w = w0 + tid % WB, s = tid / WB;
    // four independent partial sums keep four rows in flight per thread
    double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
    if (w < W && s < S) {
      int a = s;
      for (; a + 3 * S < L; a += 4 * S) {
        const double2 x0 = c[(int64_t)rows[r0 + a] * W + w];
        const double2 x1 = c[(int64_t)rows[r0 + a + S] * W + w];
        const double2 x2 = c[(int64_t)rows[r0 + a + 2 * S] * W + w];
        const double2 x3 = c[(int64_t)rows[r0 + a + 3 * S] * W + w];
        acc0 += x0.x * x0.x + x0.y * x0.y;
        acc1 += x1.x * x1.x + x1.y * x1.y;
        acc2 += x2.x * x2.x + x2.y * x2.y;
        acc3 += x3.x * x3.x + x3.y * x3.y;
      }
      for (; a < L; a += S) {
        const double2 x = c[(int64_t)rows[r0 + a] * W + w];
        acc0 += x.x * x.x + x.y * x.y;
      }
    }
    red[tid] = (acc0 + acc1) + (acc2 + acc3);
    __syncthreads();
    if (tid < WB && w0 + tid < W) {
      double sum = 0.0;
      for (int j = 0; j < S; ++j) sum += red[j * WB + tid];
      out[(int64_t)f * W + w0 + tid] = sum;
    }
    __syncthreads();
  }
}

// ================================================================ launchers
hipError_t launch_phase_table(hipStream_t s, int64_t N, const double* K2, double scale, double2* ph) {
  hipLaunchKernelGGL(k_phase_table, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, N, K2, scale, ph);
  return hipGetLastError();
}

hipError_t launch_phase_apply(hipStream_t s, int64_t N, int W, const double2* ph, double2* c) {
  int TW = 1;
  while (TW < W && TW < 256) TW <<= 1;
  const int64_t rows_per_block = 256 / TW;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((N + rows_per_block - 1) / rows_per_block,
                                                                        256 * 64));
  hipLaunchKernelGGL(k_phase_apply, dim3(grid), dim3(256), 0, s, N, W, TW, ph, c);
  return hipGetLastError();
}

hipError_t launch_reduce(hipStream_t s, const ReduceArgs& a0, int nblocks, double* mass, double* energy) {
  if (!mass && !energy) return hipSuccess;
  ReduceArgs a = a0;
  a.CW = a.sweep.order ? kSweepCW : 8;
  while (a.CW > 1 && a.CW / 2 >= a.W) a.CW /= 2;  // narrow states: no idle lanes beyond W
  // Up to 64 row workgroups (small systems) spread the column blocks over the chip instead of sweeping
  // them one after the other (mass of N = 53, W = 128 with its copy to the host: 35.8 to 28.7 us); beyond,
  // an XCD sweeps a part of the rows block by block.  The sums are the same.
  const int ny = nblocks < 64 ? std::min((a.W + a.CW - 1) / a.CW, 512 / nblocks) : 1;
  const dim3 grid(nblocks, ny), block(kReduceThreads);
  if (mass && energy)
    hipLaunchKernelGGL((k_reduce_partial<true, true>), grid, block, 0, s, a);
  else if (mass)
    hipLaunchKernelGGL((k_reduce_partial<true, false>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_reduce_partial<false, true>), grid, block, 0, s, a);
  hipError_t e = hipGetLastError();
  const dim3 fgrid((a.W + 7) / 8);
  if (e == hipSuccess && mass) {
    hipLaunchKernelGGL(k_reduce_final, fgrid, dim3(256), 0, s, nblocks, a.W, a.pmass, mass);
    e = hipGetLastError();
  }
  if (e == hipSuccess && energy) {
    hipLaunchKernelGGL(k_reduce_final, fgrid, dim3(256), 0, s, nblocks, a.W, a.penergy, energy);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_copy_home(hipStream_t s, int n, const CopyItem* items, int64_t max_elems) {
  if (n == 0 || max_elems == 0) return hipSuccess;
  // about 4096 workgroups over the systems, at least one and at most what the longest needs
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>((max_elems + 255) / 256, 4096 / n + 1));
  for (int i = 0; i < n; i += 65535)  // grid.y limit
    hipLaunchKernelGGL(k_copy_home, dim3((unsigned)want, (unsigned)std::min(65535, n - i)), dim3(256), 0, s, items + i);
  return hipGetLastError();
}

hipError_t launch_gather_rows(hipStream_t s, int64_t N, const int32_t* pos, const double2* src, double2* dst) {
  if (N == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, N, pos, src, dst);
  return hipGetLastError();
}

hipError_t launch_fibre_mass(hipStream_t s, int nf, const int32_t* ptr, const int32_t* rows, int W,
                             const double2* c, double* out) {
  if (nf == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fibre_mass, dim3(nf), dim3(256), 0, s, ptr, rows, W, c, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- allocation-free scratch
// Reduction partials of the allocation-free observables entry point live in this array, one
// copy per GPU for the life of the process.  Host code never passes the array's name to a
// kernel (on the host it is a stand-in, not a device address): the address is looked up once
// per device with that device current and kept.
static __device__ __align__(256) double scratch[kStaticScratchDoubles];

hipError_t static_scratch(double** ptr) {
  static std::mutex mu;
  static double* per_device[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    per_device[dev] = static_cast<double*>(p);
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

}  // namespace lsx

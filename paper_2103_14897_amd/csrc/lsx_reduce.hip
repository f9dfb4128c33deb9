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

// ---------------------------------------------------------------- FP64 reductions
// kind 0: |c|^2;  kind 1: 1/2 K2 |c|^2 + Re conj(c_iw) sum_p v_p c_{nbr(i,p), w} (both layers)
__global__ __launch_bounds__(256) void k_reduce_partial(int kind, int64_t N, int W, const double2* c,
                                                        const double* K2, int nv1, const int32_t* nbr1,
                                                        const double2* v1, int nv2, const int32_t* nbr2,
                                                        const double2* v2, int nv3, const int32_t* nbr3,
                                                        const double2* v3, double* partial, int R) {
  __shared__ double red[256];
  const int b = blockIdx.x;
  const int64_t i0 = (int64_t)b * R;
  const int64_t i1 = min(N, i0 + R);
  const int WB = W < 256 ? W : 256;
  const int S = 256 / WB;
  const int tid = threadIdx.x;
  for (int w0 = 0; w0 < W; w0 += WB) {
    const int w = w0 + tid % WB, s = tid / WB;
    double acc = 0.0;
    if (w < W && s < S) {
      for (int64_t i = i0 + s; i < i1; i += S) {
        const double2 x = c[i * W + w];
        const double m2 = x.x * x.x + x.y * x.y;
        if (kind == 0) {
          acc += m2;
        } else {
          double hr = 0.0, hi = 0.0;
          for (int p = 0; p < nv1; ++p) {
            const int j = nbr1[i * nv1 + p];
            if (j >= 0) {
              const double2 y = c[(int64_t)j * W + w], v = v1[p];
              hr += v.x * y.x - v.y * y.y;
              hi += v.x * y.y + v.y * y.x;
            }
          }
          for (int p = 0; p < nv2; ++p) {
            const int j = nbr2[i * nv2 + p];
            if (j >= 0) {
              const double2 y = c[(int64_t)j * W + w], v = v2[p];
              hr += v.x * y.x - v.y * y.y;
              hi += v.x * y.y + v.y * y.x;
            }
          }
          for (int p = 0; p < nv3; ++p) {
            const int j = nbr3[i * nv3 + p];
            if (j >= 0) {
              const double2 y = c[(int64_t)j * W + w], v = v3[p];
              hr += v.x * y.x - v.y * y.y;
              hi += v.x * y.y + v.y * y.x;
            }
          }
          acc += 0.5 * K2[i] * m2 + (x.x * hr + x.y * hi);
        }
      }
    }
    red[tid] = acc;
    __syncthreads();
    if (tid < WB && w0 + tid < W) {
      double sum = 0.0;
      for (int j = 0; j < S; ++j) sum += red[j * WB + tid];
      partial[(int64_t)b * W + w0 + tid] = sum;
    }
    __syncthreads();
  }
}

__global__ void k_reduce_final(int nblocks, int W, const double* partial, double* out) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w < W) {
    double s = 0.0;
    for (int b = 0; b < nblocks; ++b) s += partial[(int64_t)b * W + w];
    out[w] = s;
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

hipError_t launch_reduce(hipStream_t s, int kind, int64_t N, int W, const double2* c, const double* K2, int nv1,
                         const int32_t* nbr1, const double2* v1, int nv2, const int32_t* nbr2, const double2* v2,
                         int nv3, const int32_t* nbr3, const double2* v3, double* partial, int nblocks,
                         double* out) {
  const int R = (int)((N + nblocks - 1) / nblocks);
  hipLaunchKernelGGL(k_reduce_partial, dim3(nblocks), dim3(256), 0, s, kind, N, W, c, K2, nv1, nbr1, v1, nv2,
                     nbr2, v2, nv3, nbr3, v3, partial, R);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_reduce_final, dim3((W + 255) / 256), dim3(256), 0, s, nblocks, W, partial, out);
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

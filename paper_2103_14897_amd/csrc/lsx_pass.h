// Device code shared by the fibre-pass kernels of liblsx: operand types, bf16 splits, tile
// addressing and the epilogue.
#pragma once

#include <hip/hip_runtime.h>

#include "lsx_internal.h"

namespace lsx {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned short v8u16 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ unsigned short f2bf(float f) {
  // round to nearest even (finite inputs only)
  unsigned int u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

// three-term bf16 split of a double: x ~= t0 + t1 + t2
__device__ __forceinline__ void split3(double x, unsigned short& t0, unsigned short& t1, unsigned short& t2) {
  t0 = f2bf((float)x);
  double r = x - (double)bf2f(t0);
  t1 = f2bf((float)r);
  r = r - (double)bf2f(t1);
  t2 = f2bf((float)r);
}
// exact three-term bf16 split of an fp32 value: t0 is x with the low 16 bits cleared, t1 the
// same for the remainder x - t0 (exact in fp32, at most 16 significant bits), and the second
// remainder has at most 8 significant bits, so it is a bf16 itself: t0 + t1 + t2 = x exactly.
// Three masks and two subtractions, against three roundings for split3f.
__device__ __forceinline__ void split3x(float x, unsigned short& t0, unsigned short& t1, unsigned short& t2) {
  const unsigned u = __float_as_uint(x);
  const float r1 = x - __uint_as_float(u & 0xFFFF0000u);
  const unsigned v = __float_as_uint(r1);
  const float r2 = r1 - __uint_as_float(v & 0xFFFF0000u);
  t0 = (unsigned short)(u >> 16);
  t1 = (unsigned short)(v >> 16);
  t2 = (unsigned short)(__float_as_uint(r2) >> 16);
}

// same split from an fp32 value (all residuals exact in fp32)
__device__ __forceinline__ void split3f(float x, unsigned short& t0, unsigned short& t1, unsigned short& t2) {
  t0 = f2bf(x);
  float r = x - bf2f(t0);
  t1 = f2bf(r);
  r = r - bf2f(t1);
  t2 = f2bf(r);
}

// ---------------------------------------------------------------- tile columns
// State column of this lane in each of the tile's NB column blocks ((wb NB + nb) 16 + lane % 16),
// and whether it exists.
template <int NB>
__device__ __forceinline__ void tile_cols(const PassArgs& a, const TileDesc& t, int li, int (&wc)[NB],
                                          bool (&wok)[NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    wc[nb] = (t.wb * NB + nb) * 16 + li;
    wok[nb] = wc[nb] < a.W;
  }
}

// ---------------------------------------------------------------- fibre-pass epilogue
// acc[nb][0/1][r]: this lane's part of the 16x16 output blocks, column lane%16 and
// row 4*(lane/16)+r for the FP32-accumulating MFMAs, row 4*r+lane/16 for
// v_mfma_f64_16x16x4f64 (ROWS_F64).  Summed over the KS waves in fixed order; mixed
// formats add the FP64 diagonal term d_a x_a; an optional kinetic phase multiplies
// the output row (the phase sub-step that follows this pass, fused).
// With a.nt set the output is stored non-temporally.  The next pass reads it in the other
// layer's fibre order, mostly on other XCDs, so keeping it in this XCD's L2 can only add
// write-back work at the end of the launch; but for states that fit the last-level cache,
// ordinary stores leave it there for the next pass.  The host measures which is faster.
template <int NB, int KS, bool MIX, bool ROWS_F64>
__device__ __forceinline__ void pass_epilogue(const PassArgs& a, const TileDesc& t, double (&acc)[NB][2][4],
                                              double* red, const int (&wc)[NB], const bool (&wok)[NB]) {
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lk = lane >> 4;
  const int r0 = t.r0, L = t.L, rb = t.rb;
  const int W = a.W;
  if (KS > 1) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(((kw * NB + nb) * 2 + c) * 4 + r) * 64 + lane] = acc[nb][c][r];
    __syncthreads();
  }
  for (int r = (KS > 1 ? kw : 0); r < 4; r += KS) {
    const int arow = 16 * rb + (ROWS_F64 ? 4 * r + lk : 4 * lk + r);
    if (arow >= L) continue;
    const int p = r0 + arow;
    const int64_t orow = a.out_pos ? a.out_pos[p] : p;
    const int64_t irow = a.in_pos ? a.in_pos[p] : p;
    double2 ph = make_double2(1.0, 0.0);
    if (a.ph) ph = a.ph[a.ph_idx ? a.ph_idx[p] : p];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int w = wc[nb];
      if (!wok[nb]) continue;
      double yr, yi;
      if (KS > 1) {
        yr = 0.0;
        yi = 0.0;
        for (int j = 0; j < KS; ++j) {
          yr += red[(((j * NB + nb) * 2 + 0) * 4 + r) * 64 + lane];
          yi += red[(((j * NB + nb) * 2 + 1) * 4 + r) * 64 + lane];
        }
      } else {
        yr = acc[nb][0][r];
        yi = acc[nb][1][r];
      }
      if (MIX) {
        const double2 x = a.X[irow * W + w];
        const double2 dg = a.diag[t.d0 + arow];
        yr += dg.x * x.x - dg.y * x.y;
        yi += dg.x * x.y + dg.y * x.x;
      }
      if (a.ph) {
        const double zr = ph.x * yr - ph.y * yi;
        yi = ph.x * yi + ph.y * yr;
        yr = zr;
      }
      double2* y = a.Y + orow * W + w;
      if (a.nt) {
        // empty compiler barriers (no instruction) around the stores keep them from being
        // hoisted or sunk together with the other branch's, which would drop the hint
        asm volatile("" ::: "memory");
        __builtin_nontemporal_store(yr, &y->x);
        __builtin_nontemporal_store(yi, &y->y);
        asm volatile("" ::: "memory");
      } else {
        *y = make_double2(yr, yi);
      }
    }
  }
}

__device__ __forceinline__ int64_t in_row(const PassArgs& a, int p) { return a.in_pos ? a.in_pos[p] : p; }

// Band of a tile in units of `unit` fibre positions (4 for a k-step of the FP64 / FP32
// products, 32 for a BF16x3 chunk): [lo, hi), clamped to the padded fibre length Lp.
__device__ __forceinline__ void tile_band(const TileDesc& t, int Lp, int unit, int& lo, int& hi) {
  lo = t.k0 / unit;
  hi = (min(t.k1, Lp) + unit - 1) / unit;
}

// GATHER: element k of the fibre is row in_pos[r0 + k] of X, else row r0 + k.
template <bool GATHER>
__device__ __forceinline__ int64_t xrow(const PassArgs& a, int p) {
  return GATHER ? (int64_t)a.in_pos[p] : (int64_t)p;
}

__device__ __forceinline__ v8bf as_bf(const v8u16& u) { return __builtin_bit_cast(v8bf, u); }

// acc += A (3 bf16 terms) * B (3 bf16 terms), six cross products, smallest first
__device__ __forceinline__ v4f mma3(v4f c, const v8bf& a0, const v8bf& a1, const v8bf& a2, const v8bf& b0,
                                    const v8bf& b1, const v8bf& b2) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b0, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b2, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b0, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b1, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, c, 0, 0, 0);
  return c;
}

}  // namespace lsx

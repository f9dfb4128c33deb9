// Row-split fibre passes of liblsx: the waves of a workgroup take consecutive 16-row blocks of
// one fibre and share the state operand, staged once per workgroup in LDS.
#include "lsx_pass.h"

namespace lsx {

// ---------------------------------------------------------------- row-split passes, LDS-staged state
// Workgroup = MS waves on MS consecutive 16-row blocks of one fibre (tile rb counts groups
// of MS blocks) and the same 16 NB columns.  The state operand of every 16-row chunk of
// the fibre is read from memory once per workgroup, converted once (FP32 and the 3M sums
// x_r, x_i - x_r, x_r + x_i) into double-buffered LDS and read there by all MS waves, so
// each state row is fetched once per row-block group instead of once per row block.  Each
// wave streams its own propagator rows, one chunk ahead in registers.  No cross-wave
// reduction: every wave owns its output rows.  Needs MS <= 4 NB.  Chunks are KC k-steps
// (4 KC fibre positions); four- and eight-wave groups take 32-row chunks, which halves the
// barriers and doubles the work that hides each chunk's loads without costing occupancy.
// With band-limited products the staged chunks cover the union of the group's bands, and
// each wave multiplies only the chunks of its own row block's band (PassArgs::rb_band), so
// larger groups read the state operand fewer times without adding products.
template <int NB, int MS>
struct StageMap {
  static constexpr int KC = MS >= 4 ? 8 : 4;   // k-steps per chunk
  static constexpr int CR = 4 * KC;            // rows of a chunk
  static constexpr int CW = 16 * NB;           // columns of a chunk
  static constexpr int PER = CR * CW / (64 * MS);  // elements per thread per chunk
  static constexpr int RSTEP = 64 * MS / CW;   // chunk rows between a thread's elements
};

template <int PER, int RSTEP, int CR, bool GATHER>
__device__ __forceinline__ void stage_load_f32(double2 (&v)[PER], const PassArgs& a, int ch, int r0, int L, int w,
                                               bool wok, int rr0) {
  const double2* zx = reinterpret_cast<const double2*>(a.zero);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int k = CR * ch + rr0 + j * RSTEP;
    const bool ok = wok && k < L;
    const int64_t row = xrow<GATHER>(a, r0 + (ok ? k : 0));
    v[j] = *(ok ? a.X + row * a.W + w : zx);
  }
}

template <int NB, int MS, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * MS, true) void k_pass_f32m(PassArgs a) {
  using SM = StageMap<NB, MS>;
  constexpr int KC = SM::KC;
  __shared__ float4 xs[2][SM::CR][SM::CW];
  if (a.tcount && (int)blockIdx.x >= *a.tcount) return;
  const TileDesc t0 = a.tiles[blockIdx.x];
  if (t0.f < 0) return;
  const int r0 = t0.r0, L = t0.L;
  const int nks = ((L + 15) & ~15) >> 2;
  // chunks [clo, clo + nch) cover the tile's band; k-steps past nks read zeros
  int clo, nch;
  tile_band(t0, 4 * nks, SM::CR, clo, nch);
  nch -= clo;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  TileDesc t = t0;
  t.rb = t0.rb * MS + kw;
  const bool act = t.rb < ((L + 15) >> 4);
  const float2* zp = reinterpret_cast<const float2*>(a.zero);
  const float2* P = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                    (int64_t)(act ? t.rb : 0) * nks * 64 + lane;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  // this thread's staging slot: column c (fixed), rows rr0 + j RSTEP of each chunk
  const int c = threadIdx.x % SM::CW, rr0 = threadIdx.x / SM::CW;
  int sw;
  bool sok;
  {
    const int nc = a.cols ? a.ncols[t.f] : a.W;
    const int sl = t.wb * SM::CW + c;
    sok = sl < nc;
    sw = a.cols ? (sok ? a.cols[(int64_t)t.f * a.W + sl] : 0) : sl;
  }
  v4f k1[NB], k2[NB], k3[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  double2 sv[SM::PER];
  float2 Ac[KC], An[KC];
  // chunks of the band in the order c0, c0 + 1, ... (cyclically), with the workgroup's own
  // rows last: the epilogue's FP64 reload of those rows then finds them in this XCD's L2,
  // just staged
  const int c0 = (((t0.rb + 1) * MS * 16 / SM::CR - clo) % nch + nch) % nch;
  auto chunk = [&](int i) { return clo + (i + c0 < nch ? i + c0 : i + c0 - nch); };
  // this wave's own band [wlo, whi) of chunks (its row block's), inside the staged ones
  int wlo = clo, whi = clo + nch;
  if (a.rb_band && t0.bb >= 0 && act) {
    const int2 wb = reinterpret_cast<const int2*>(a.rb_band)[t0.bb + t.rb];
    wlo = wb.x / SM::CR;
    whi = (min(wb.y, 4 * nks) + SM::CR - 1) / SM::CR;
  }
  auto mine = [&](int cc) { return act && cc >= wlo && cc < whi; };
  stage_load_f32<SM::PER, SM::RSTEP, SM::CR, GATHER>(sv, a, chunk(0), r0, L, sw, sok, rr0);
  {
    const bool in = mine(chunk(0));
#pragma unroll
    for (int u = 0; u < KC; ++u) {
      const int ks = KC * chunk(0) + u;
      Ac[u] = (in && ks < nks) ? P[(int64_t)ks * 64] : *zp;
    }
  }
#pragma unroll
  for (int j = 0; j < SM::PER; ++j) {
    const float xr = (float)sv[j].x, xi = (float)sv[j].y;
    xs[0][rr0 + j * SM::RSTEP][c] = make_float4(xr, xi - xr, xr + xi, 0.f);
  }
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int buf = ch & 1;
    const bool more = ch + 1 < nch;
    if (more) {
      stage_load_f32<SM::PER, SM::RSTEP, SM::CR, GATHER>(sv, a, chunk(ch + 1), r0, L, sw, sok, rr0);
      const bool in = mine(chunk(ch + 1));
#pragma unroll
      for (int u = 0; u < KC; ++u) {
        const int ks = KC * chunk(ch + 1) + u;
        An[u] = (in && ks < nks) ? P[(int64_t)ks * 64] : *zp;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (mine(chunk(ch))) {
#pragma unroll
      for (int u = 0; u < KC; ++u) {
        const float ps = Ac[u].x + Ac[u].y;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float4 b = xs[buf][4 * u + lk][nb * 16 + li];
          k1[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ps, b.x, k1[nb], 0, 0, 0);
          k2[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ac[u].x, b.y, k2[nb], 0, 0, 0);
          k3[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ac[u].y, b.z, k3[nb], 0, 0, 0);
        }
      }
    }
    if (more) {
#pragma unroll
      for (int j = 0; j < SM::PER; ++j) {
        const float xr = (float)sv[j].x, xi = (float)sv[j].y;
        xs[buf ^ 1][rr0 + j * SM::RSTEP][c] = make_float4(xr, xi - xr, xr + xi, 0.f);
      }
#pragma unroll
      for (int u = 0; u < KC; ++u) Ac[u] = An[u];
    }
    __syncthreads();
  }
  if (!act) return;
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = (double)k1[nb][r] - (double)k3[nb][r];
      acc[nb][1][r] = (double)k1[nb][r] + (double)k2[nb][r];
    }
  pass_epilogue<NB, 1, true, false>(a, t, acc, nullptr, wc, wok);
}

// Row-split FP64 pass: MS waves on consecutive row blocks, chunks of KC k-steps (4 KC rows) of the
// state staged in double-buffered LDS as the three B operands of the 3M products (x_r, x_i - x_r,
// x_r + x_i).  FP64 matrix instructions and vector instructions do not overlap on a SIMD (64
// cycles each; four integer additions between them measured 82), so the loop is laid out to
// have next to no vector instructions: the sums are formed once per staged element instead of
// once per wave, propagator chunks are read at a uniform address plus the lane, each into the
// registers its predecessor just left (a whole chunk of products ahead of its use, and no second
// set of registers), and the chunks a wave only stages are separate loops, without a branch
// around the products (which copied every accumulator).  Five vector instructions per 24
// products, 92 registers (NB = 2): five waves per SIMD.
// Twisted bilayer, N = 398821, W = 128, tau = 5e-3, layer 1 / 2: 1688 / 1515 us a pass, 59 TF of
// matrix work; the fastest K-split shape takes 2030 / 1800, as did this kernel when it formed the
// sums in every wave with addresses in vector registers (1970 / 1790).  Measured slower: MS = 2
// and 8 (1890, 1744), two waves' register buffers in turn (1962), next k-step's LDS reads ahead
// (1745: 108 registers).
template <int NB, int MS, int KC, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * MS, true) void k_pass_f64m(PassArgs a) {
  constexpr int CW = 16 * NB, CR = 4 * KC;
  constexpr int PER = CR * CW / (64 * MS), RSTEP = 64 * MS / CW;
  static_assert(PER >= 1, "at least one staged element per thread");
  __shared__ double xs[2][3][NB][CR][16];
  const TileDesc t0 = a.tiles[blockIdx.x];
  if (t0.f < 0) return;
  const int r0 = t0.r0, L = t0.L;
  const int nks = ((L + 15) & ~15) >> 2;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  TileDesc t = t0;
  t.rb = t0.rb * MS + kw;
  const bool act = t.rb < ((L + 15) >> 4);
  const double2* zp = reinterpret_cast<const double2*>(a.zero);
  const double2* P = reinterpret_cast<const double2*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                     (int64_t)(act ? t.rb : 0) * nks * 64;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  const int c = threadIdx.x % CW, rr0 = threadIdx.x / CW;
  const int sw = t.wb * CW + c;
  const bool sok = sw < a.W;
  v4d k1[NB], k2[NB], k3[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (v4d){0.0, 0.0, 0.0, 0.0};
  int klo, khi;  // staged chunks of CR rows: the union of the group's bands
  tile_band(t0, 4 * nks, CR, klo, khi);
  int wlo = klo * KC, whi = min(khi * KC, nks);  // this wave's own band in k-steps
  if (a.rb_band && t0.bb >= 0 && act) {
    const int2 wb = reinterpret_cast<const int2*>(a.rb_band)[t0.bb + t.rb];
    wlo = wb.x >> 2;
    whi = min(wb.y, 4 * nks) >> 2;
  }
  if (!act) whi = wlo;
  double2 sv[PER];
  const double2* xp = a.X + (int64_t)(r0 + rr0) * a.W + sw;  // this thread's element of chunk 0
  auto load_state = [&](int ch) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int k = CR * ch + rr0 + j * RSTEP;
      const bool ok = sok && k < L;
      if (GATHER) {
        int64_t off = xrow<GATHER>(a, r0 + (ok ? k : 0)) * a.W + sw;
        asm volatile("" : "+v"(off));
        sv[j] = *(ok ? a.X + off : zp);
      } else {
        const double2* q = xp + (int64_t)(CR * ch + j * RSTEP) * a.W;
        sv[j] = *(ok ? q : zp);
      }
    }
  };
  const int sb = c >> 4, sc = c & 15;
  auto store_state = [&](int buf) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      xs[buf][0][sb][rr0 + j * RSTEP][sc] = sv[j].x;
      xs[buf][1][sb][rr0 + j * RSTEP][sc] = sv[j].y - sv[j].x;
      xs[buf][2][sb][rr0 + j * RSTEP][sc] = sv[j].x + sv[j].y;
    }
  };
  // propagator chunk of k-step ks (zeros outside the wave's band; the address is uniform)
  auto load_p = [&](int ks) {
    const double2* q = (ks >= wlo && ks < whi) ? P + (int64_t)ks * 64 : zp;
    return q[(unsigned)lane];
  };
  // chunks this wave multiplies: [alo, ahi), inside the staged [klo, khi)
  const int alo = act ? min(max(wlo / KC, klo), khi) : khi;
  const int ahi = act ? min(max((whi + KC - 1) / KC, alo), khi) : khi;
  double2 E[KC];
  int ch = klo;
  load_state(klo);
  if (alo < ahi)
#pragma unroll
    for (int u = 0; u < KC; ++u) E[u] = load_p(KC * alo + u);
  store_state(0);
  __syncthreads();
  // stage chunk ch + 1 while chunk ch is multiplied (or passed over)
  auto next = [&](int cn) {
    if (cn < khi) {
      store_state((cn - klo) & 1);
      __syncthreads();
    }
  };
  for (; ch < alo; ++ch) {
    load_state(ch + 1);
    next(ch + 1);
  }
  for (; ch < ahi; ++ch) {
    load_state(ch + 1);
    const int buf = (ch - klo) & 1;
#pragma unroll
    for (int u = 0; u < KC; ++u) {
      const double2 p = E[u];
      const double ps = p.x + p.y;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        k1[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ps, xs[buf][0][nb][4 * u + lk][li], k1[nb], 0, 0, 0);
        k2[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(p.x, xs[buf][1][nb][4 * u + lk][li], k2[nb], 0, 0, 0);
        k3[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(p.y, xs[buf][2][nb][4 * u + lk][li], k3[nb], 0, 0, 0);
      }
      E[u] = load_p(KC * (ch + 1) + u);
      __builtin_amdgcn_sched_barrier(0);
    }
    next(ch + 1);
  }
  for (; ch < khi; ++ch) {
    load_state(ch + 1);
    next(ch + 1);
  }
  if (!act) return;
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = k1[nb][r] - k3[nb][r];
      acc[nb][1][r] = k1[nb][r] + k2[nb][r];
    }
  pass_epilogue<NB, 1, false, true>(a, t, acc, nullptr, wc, wok);
}

// Row-split BF16x3 pass: as k_pass_f32m, with 32-row chunks.  The staging threads split each
// state value once (x~ = fp32(x) into three bf16 terms, real and imaginary parts) into six
// LDS planes stored column-major (a lane's 8 consecutive k values are one 16-byte read);
// every wave multiplies its own propagator rows (six bf16 planes, one chunk ahead in
// registers) with the shared planes.  Needs MS <= 8 NB.
template <int NB>
struct StageBF {
  static constexpr int CW = 16 * NB;
  static constexpr int KP = 40;  // padded k stride of a column (32 used)
};

template <int NB, int MS, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * MS, true) void k_pass_bf16m(PassArgs a) {
  constexpr int CW = StageBF<NB>::CW, KP = StageBF<NB>::KP;
  constexpr int PER = 32 * CW / (64 * MS), RSTEP = 64 * MS / CW;
  __shared__ __attribute__((aligned(16))) unsigned short xb[2][6][CW][KP];
  if (a.tcount && (int)blockIdx.x >= *a.tcount) return;
  const TileDesc t0 = a.tiles[blockIdx.x];
  if (t0.f < 0) return;
  const int r0 = t0.r0, L = t0.L;
  const int nkc = ((L + 31) & ~31) >> 5;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  TileDesc t = t0;
  t.rb = t0.rb * MS + kw;
  const bool act = t.rb < ((L + 15) >> 4);
  const v8bf* zb = reinterpret_cast<const v8bf*>(a.zero);
  const v8bf* P = reinterpret_cast<const v8bf*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                  (int64_t)(act ? t.rb : 0) * nkc * 6 * 64 + lane;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  const int c = threadIdx.x % CW, rr0 = threadIdx.x / CW;
  int sw;
  bool sok;
  {
    const int nc = a.cols ? a.ncols[t.f] : a.W;
    const int sl = t.wb * CW + c;
    sok = sl < nc;
    sw = a.cols ? (sok ? a.cols[(int64_t)t.f * a.W + sl] : 0) : sl;
  }
  const double2* zx = reinterpret_cast<const double2*>(a.zero);
  v4f rr[NB], ii[NB], ri[NB], ir[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) rr[nb] = ii[nb] = ri[nb] = ir[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  double2 sv[PER];
  // State operands of chunk kc (rows past the fibre read the zero buffer).  The offset is
  // computed unconditionally and pinned by an empty asm operand, so the pointer select stays a
  // select: a load under a branch makes the compiler wait for every outstanding load at the
  // join, including the next chunk's prefetch.  (Pinning the pointer itself would lose its
  // address space and turn the loads into flat loads, which LDS waits also wait for.)
  auto load_state = [&](int kc) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int k = 32 * kc + rr0 + j * RSTEP;
      const bool ok = sok && k < L;
      int64_t off = xrow<GATHER>(a, r0 + (ok ? k : 0)) * a.W + sw;
      asm volatile("" : "+v"(off));
      sv[j] = *(ok ? a.X + off : zx);
    }
  };
  // fp32(x) split exactly into three bf16 terms, six planes [term re/im][column][k]
  auto store_state = [&](int buf) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      unsigned short q0, q1, q2, q3, q4, q5;
      split3x((float)sv[j].x, q0, q1, q2);
      split3x((float)sv[j].y, q3, q4, q5);
      const int k = rr0 + j * RSTEP;
      xb[buf][0][c][k] = q0;
      xb[buf][1][c][k] = q1;
      xb[buf][2][c][k] = q2;
      xb[buf][3][c][k] = q3;
      xb[buf][4][c][k] = q4;
      xb[buf][5][c][k] = q5;
    }
  };
  // the tile's band of chunks [klo, khi), and this wave's own [wlo, whi) inside it (its row
  // block's band; the staged chunks cover the union)
  int klo, khi;
  tile_band(t0, 32 * nkc, 32, klo, khi);
  int wlo = klo, whi = khi;
  if (a.rb_band && t0.bb >= 0 && act) {
    const int2 wb = reinterpret_cast<const int2*>(a.rb_band)[t0.bb + t.rb];
    wlo = wb.x / 32;
    whi = (min(wb.y, 32 * nkc) + 31) / 32;
  }
  auto mine = [&](int kc) { return act && kc >= wlo && kc < whi; };
  // this wave's propagator planes of chunk kc (E re/im terms 0..2), zeros outside its band
  auto load_e = [&](v8bf (&E)[6], int kc) {
    const bool in = mine(kc);
#pragma unroll
    for (int pl = 0; pl < 6; ++pl) {
      int64_t off = ((int64_t)kc * 6 + pl) * 64;
      asm volatile("" : "+v"(off));
      E[pl] = *(in ? P + off : zb);
    }
  };
  auto mma = [&](const v8bf (&E)[6], int buf) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      // one column block's operands at a time (keeps the next block's LDS reads from being
      // hoisted, which would hold twice the registers)
      if (nb > 0) __builtin_amdgcn_sched_barrier(0);
      const int col = nb * 16 + li;
      const v8bf Xr0 = *reinterpret_cast<const v8bf*>(&xb[buf][0][col][8 * lk]);
      const v8bf Xr1 = *reinterpret_cast<const v8bf*>(&xb[buf][1][col][8 * lk]);
      const v8bf Xr2 = *reinterpret_cast<const v8bf*>(&xb[buf][2][col][8 * lk]);
      const v8bf Xi0 = *reinterpret_cast<const v8bf*>(&xb[buf][3][col][8 * lk]);
      const v8bf Xi1 = *reinterpret_cast<const v8bf*>(&xb[buf][4][col][8 * lk]);
      const v8bf Xi2 = *reinterpret_cast<const v8bf*>(&xb[buf][5][col][8 * lk]);
      rr[nb] = mma3(rr[nb], E[0], E[2], E[4], Xr0, Xr1, Xr2);
      ii[nb] = mma3(ii[nb], E[1], E[3], E[5], Xi0, Xi1, Xi2);
      ri[nb] = mma3(ri[nb], E[0], E[2], E[4], Xi0, Xi1, Xi2);
      ir[nb] = mma3(ir[nb], E[1], E[3], E[5], Xr0, Xr1, Xr2);
    }
  };
  // Ping-pong operand buffers over pairs of chunks: chunk kc multiplies EA (or EB) while the
  // next chunk's state values and planes load into sv and EB (or EA); no register copies.
  v8bf EA[6], EB[6];
  load_state(klo);
  load_e(EA, klo);
  store_state(0);
  __syncthreads();
  for (int kc = klo; kc < khi; kc += 2) {
    load_state(kc + 1);
    load_e(EB, kc + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (mine(kc)) mma(EA, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (kc + 1 >= khi) break;
    store_state(1);
    __syncthreads();
    load_state(kc + 2);
    load_e(EA, kc + 2);
    __builtin_amdgcn_sched_barrier(0);
    if (mine(kc + 1)) mma(EB, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (kc + 2 >= khi) break;
    store_state(0);
    __syncthreads();
  }
  if (!act) return;
  double acc[NB][2][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc[nb][0][r] = (double)rr[nb][r] - (double)ii[nb][r];
      acc[nb][1][r] = (double)ri[nb][r] + (double)ir[nb][r];
    }
  pass_epilogue<NB, 1, true, false>(a, t, acc, nullptr, wc, wok);
}

// Row-split tiles of nb column blocks and ms waves (PassArgs::in_pos null: no gather)
hipError_t launch_rowsplit(hipStream_t s, int fmt, int ntiles, int nb, int ms, const PassArgs& a) {
  const bool gather = a.in_pos != nullptr;
  if (fmt == PF_F64) {
#define LSX_ROWSPLIT_F64(NB_, MS_, KC_)                                                             \
  if (nb == NB_ && ms == MS_) {                                                                     \
    if (gather)                                                                                     \
      hipLaunchKernelGGL((k_pass_f64m<NB_, MS_, KC_, true>), dim3(ntiles), dim3(64 * MS_), 0, s, a);  \
    else                                                                                            \
      hipLaunchKernelGGL((k_pass_f64m<NB_, MS_, KC_, false>), dim3(ntiles), dim3(64 * MS_), 0, s, a); \
    return hipGetLastError();                                                                       \
  }
    LSX_ROWSPLIT_F64(1, 4, 4)
    LSX_ROWSPLIT_F64(2, 4, 4)
#undef LSX_ROWSPLIT_F64
    return hipErrorInvalidValue;
  }
  if (fmt == PF_BF16X3) {
#define LSX_ROWSPLIT_BF(NB_, MS_)                                                                       \
  if (nb == NB_ && ms == MS_) {                                                                    \
  if (gather)                                                                                         \
      hipLaunchKernelGGL((k_pass_bf16m<NB_, MS_, true>), dim3(ntiles), dim3(64 * MS_), 0, s, a);        \
    else                                                                                              \
      hipLaunchKernelGGL((k_pass_bf16m<NB_, MS_, false>), dim3(ntiles), dim3(64 * MS_), 0, s, a);       \
    return hipGetLastError();                                                                         \
  }
    LSX_ROWSPLIT_BF(1, 2)
    LSX_ROWSPLIT_BF(1, 4)
    LSX_ROWSPLIT_BF(1, 8)
    LSX_ROWSPLIT_BF(2, 2)
    LSX_ROWSPLIT_BF(2, 4)
    LSX_ROWSPLIT_BF(2, 8)
#undef LSX_ROWSPLIT_BF
    return hipErrorInvalidValue;
  }
#define LSX_ROWSPLIT_CASE(NB_, MS_)                                                                      \
  if (nb == NB_ && ms == MS_) {                                                                    \
  if (gather)                                                                                         \
      hipLaunchKernelGGL((k_pass_f32m<NB_, MS_, true>), dim3(ntiles), dim3(64 * MS_), 0, s, a);         \
    else                                                                                              \
      hipLaunchKernelGGL((k_pass_f32m<NB_, MS_, false>), dim3(ntiles), dim3(64 * MS_), 0, s, a);        \
    return hipGetLastError();                                                                         \
  }
  LSX_ROWSPLIT_CASE(1, 2)
  LSX_ROWSPLIT_CASE(1, 4)
  LSX_ROWSPLIT_CASE(2, 2)
  LSX_ROWSPLIT_CASE(2, 4)
  LSX_ROWSPLIT_CASE(2, 8)
  LSX_ROWSPLIT_CASE(4, 2)
  LSX_ROWSPLIT_CASE(4, 4)
  LSX_ROWSPLIT_CASE(4, 8)
#undef LSX_ROWSPLIT_CASE
  return hipErrorInvalidValue;
}

}  // namespace lsx

// Row-split fibre passes of liblsx: the waves of a workgroup take consecutive 16-row blocks of
// one fibre and share the state operand, staged once per workgroup in LDS.
#include "lsx_pass.h"

namespace lsx {

// State element at byte offset `off` from X, or a zero: both as one load from a selected offset
// (`zoff`: the zero buffer's distance from X), so that no branch surrounds the load
__device__ __forceinline__ double2 load_or_zero(const double2* X, bool ok, int64_t off, int64_t zoff) {
  const int64_t o = ok ? off : zoff;
  return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(X) + o);
}
__device__ __forceinline__ int64_t byte_distance(const void* from, const void* to) {
  return (int64_t)(reinterpret_cast<uintptr_t>(to) - reinterpret_cast<uintptr_t>(from));
}

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
// Vector instructions take issue time from the matrix ones (32 cycles each, about 1.7 more per
// vector instruction between them), so the propagator chunks are read at a uniform address plus
// the lane, each into the registers its predecessor just left.  Twisted bilayer, N = 398821,
// W = 128, tau = 1e-3, 2 column blocks and 8 waves, layer 1 / 2: 945 / 843 us a pass with a second
// register set and addresses in vector registers, 779 / 691 now; Example 3, W = 100, best shape,
// 447 to 390 us a step.
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
                                               bool wok, int rr0, int64_t zoff) {
  // the thread's element of the chunk's first rows, and rows RSTEP apart from there
  const int64_t row_bytes = (int64_t)a.W * 16;
  const int64_t off0 = (int64_t)(r0 + CR * ch + rr0) * row_bytes + (int64_t)w * 16;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int k = CR * ch + rr0 + j * RSTEP;
    const bool ok = wok && k < L;
    const int64_t off = GATHER ? xrow<GATHER>(a, r0 + (ok ? k : 0)) * row_bytes + (int64_t)w * 16
                               : off0 + (int64_t)(j * RSTEP) * row_bytes;
    v[j] = load_or_zero(a.X, ok, off, zoff);
  }
}

template <int NB, int MS, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * MS, true) void k_pass_f32m(PassArgs a) {
  using SM = StageMap<NB, MS>;
  constexpr int KC = SM::KC;
  __shared__ float4 xs[2][SM::CR][SM::CW];
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
  static_assert(64 * sizeof(float2) <= kZeroBytes, "load_p reads a zero for every lane");
  const float2* zp = reinterpret_cast<const float2*>(a.zero);
  const float2* P = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                    (int64_t)(act ? t.rb : 0) * nks * 64;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  // this thread's staging slot: column c (fixed), rows rr0 + j RSTEP of each chunk
  const int c = threadIdx.x % SM::CW, rr0 = threadIdx.x / SM::CW;
  const int sw = t.wb * SM::CW + c;
  const bool sok = sw < a.W;
  v4f k1[NB], k2[NB], k3[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) k1[nb] = k2[nb] = k3[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  double2 sv[SM::PER];
  float2 E[KC];
  const int64_t zoff = byte_distance(a.X, a.zero);
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
  // propagator chunk of k-step ks (zeros outside the wave's band): a uniform address and the lane
  auto load_p = [&](bool in, int ks) {
    const float2* q = (in && ks < nks) ? P + (int64_t)ks * 64 : zp;
    return q[(unsigned)lane];
  };
  stage_load_f32<SM::PER, SM::RSTEP, SM::CR, GATHER>(sv, a, chunk(0), r0, L, sw, sok, rr0, zoff);
  {
    const bool in = mine(chunk(0));
#pragma unroll
    for (int u = 0; u < KC; ++u) E[u] = load_p(in, KC * chunk(0) + u);
  }
  auto stage_store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < SM::PER; ++j) {
      const float xr = (float)sv[j].x, xi = (float)sv[j].y;
      xs[buf][rr0 + j * SM::RSTEP][c] = make_float4(xr, xi - xr, xr + xi, 0.f);
    }
  };
  stage_store(0);
  __syncthreads();
  for (int ch = 0; ch < nch; ++ch) {
    const int buf = ch & 1;
    const int cn = ch + 1 < nch ? chunk(ch + 1) : 0;
    const bool more = ch + 1 < nch, in = more && mine(cn);
    if (more) stage_load_f32<SM::PER, SM::RSTEP, SM::CR, GATHER>(sv, a, cn, r0, L, sw, sok, rr0, zoff);
    __builtin_amdgcn_sched_barrier(0);
    if (mine(chunk(ch))) {
#pragma unroll
      for (int u = 0; u < KC; ++u) {
        const float2 p = E[u];
        const float ps = p.x + p.y;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const float4 b = xs[buf][4 * u + lk][nb * 16 + li];
          k1[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ps, b.x, k1[nb], 0, 0, 0);
          k2[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(p.x, b.y, k2[nb], 0, 0, 0);
          k3[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(p.y, b.z, k3[nb], 0, 0, 0);
        }
        // the next chunk's entries into the registers these products have just read
        E[u] = load_p(in, KC * cn + u);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < KC; ++u) E[u] = load_p(in, KC * cn + u);
    }
    if (more) stage_store(buf ^ 1);
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
// products, 94 registers (NB = 2): five waves per SIMD.
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
  static_assert(64 * sizeof(double2) <= kZeroBytes, "load_p reads a zero for every lane");
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
  // this thread's element of the chunk that load_state reads next (chunks in order from klo)
  const double2* xp = a.X + (int64_t)(r0 + CR * klo + rr0) * a.W + sw;
  const int64_t step = (int64_t)CR * a.W;
  auto load_state = [&](int ch) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int k = CR * ch + rr0 + j * RSTEP;
      const bool ok = sok && k < L;
      const double2* q = GATHER ? a.X + xrow<GATHER>(a, r0 + (ok ? k : 0)) * a.W + sw : xp + (int64_t)(j * RSTEP) * a.W;
      sv[j] = *(ok ? q : zp);
    }
    xp += step;
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
// LDS planes in B-operand order (lane = column + 16 (k / 8), element k % 8: a lane's operand is one
// 16-byte read, a wave's 1 KiB in a row), two rows of a column at a time where a thread has two;
// every wave multiplies its own propagator rows (six bf16 planes in registers) with the shared
// planes.  Needs MS <= 8 NB.
// Twisted bilayer, N = 398821, W = 128, tau = 1e-3, 2 column blocks and 8 waves, layer 1 / 2: 718 /
// 651 us a pass with planes for two chunks in registers (124), their addresses in vector
// registers and two-byte staging stores into padded columns (28% of the cycles lost to bank
// conflicts); 690 / 624 now, with 94 registers; the trilayer's best shape 564 to 505 us.
template <int NB, int MS, bool GATHER>
__global__ LSX_MFMA_BOUNDS(64 * MS, true) void k_pass_bf16m(PassArgs a) {
  constexpr int CW = 16 * NB;
  constexpr int PER = 32 * CW / (64 * MS), RSTEP = 64 * MS / CW;
  constexpr int RP = PER > 1 ? 2 : 1;  // consecutive rows a thread stages together
  __shared__ __attribute__((aligned(16))) unsigned short xb[2][6][NB][64][8];
  const TileDesc t0 = a.tiles[blockIdx.x];
  if (t0.f < 0) return;
  const int r0 = t0.r0, L = t0.L;
  const int nkc = ((L + 31) & ~31) >> 5;
  const int lane = threadIdx.x & 63, kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  TileDesc t = t0;
  t.rb = t0.rb * MS + kw;
  const bool act = t.rb < ((L + 15) >> 4);
  static_assert(64 * sizeof(v8bf) <= kZeroBytes, "load_e reads a zero for every lane");
  const v8bf* zb = reinterpret_cast<const v8bf*>(a.zero);
  const v8bf* P = reinterpret_cast<const v8bf*>(reinterpret_cast<const char*>(a.P) + t.poff) +
                  (int64_t)(act ? t.rb : 0) * nkc * 6 * 64;
  int wc[NB];
  bool wok[NB];
  tile_cols<NB>(a, t, li, wc, wok);
  const int c = threadIdx.x % CW, rr0 = threadIdx.x / CW;
  const int sw = t.wb * CW + c;
  const bool sok = sw < a.W;
  v4f rr[NB], ii[NB], ri[NB], ir[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) rr[nb] = ii[nb] = ri[nb] = ir[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
  double2 sv[PER];
  // State operands of chunk kc (rows past the fibre read zeros): rows RP (rr0 + RSTEP j) + q of the
  // chunk, q < RP
  const int64_t zoff = byte_distance(a.X, a.zero), row_bytes = (int64_t)a.W * 16;
  auto row_of = [&](int e) { return RP * (rr0 + (e / RP) * RSTEP) + e % RP; };
  // fp32(x) split exactly into three bf16 terms, six planes [term re/im]
  const int sb = c >> 4, sc = c & 15;
  auto store_state = [&](int buf) {
#pragma unroll
    for (int e = 0; e < PER; e += RP) {
      unsigned short q[RP][6];
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        split3x((float)sv[e + r].x, q[r][0], q[r][1], q[r][2]);
        split3x((float)sv[e + r].y, q[r][3], q[r][4], q[r][5]);
      }
      const int k = row_of(e);
#pragma unroll
      for (int pl = 0; pl < 6; ++pl) {
        unsigned short* to = &xb[buf][pl][sb][sc + 16 * (k >> 3)][k & 7];
        if (RP == 2)
          *reinterpret_cast<unsigned*>(to) = (unsigned)q[0][pl] | ((unsigned)q[RP - 1][pl] << 16);
        else
          *to = q[0][pl];
      }
    }
  };
  // the tile's band of chunks [klo, khi), and this wave's own [wlo, whi) inside it (its row
  // block's band; the staged chunks cover the union)
  int klo, khi;
  tile_band(t0, 32 * nkc, 32, klo, khi);
  // byte offset of this thread's first element of the chunk that load_state reads next (chunks in
  // order from klo)
  int64_t off0 = (int64_t)(r0 + 32 * klo + RP * rr0) * row_bytes + (int64_t)sw * 16;
  auto load_state = [&](int kc) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int k = 32 * kc + row_of(e);
      const bool ok = sok && k < L;
      const int64_t off = GATHER ? xrow<GATHER>(a, r0 + (ok ? k : 0)) * row_bytes + (int64_t)sw * 16
                                 : off0 + (int64_t)(RP * (e / RP) * RSTEP + e % RP) * row_bytes;
      sv[e] = load_or_zero(a.X, ok, off, zoff);
    }
    off0 += 32 * row_bytes;
  };
  int wlo = klo, whi = khi;
  if (a.rb_band && t0.bb >= 0 && act) {
    const int2 wb = reinterpret_cast<const int2*>(a.rb_band)[t0.bb + t.rb];
    wlo = wb.x / 32;
    whi = (min(wb.y, 32 * nkc) + 31) / 32;
  }
  auto mine = [&](int kc) { return act && kc >= wlo && kc < whi; };
  // propagator planes of chunk kc, real (part 0) or imaginary (part 1) terms 0..2, zeros outside
  // the wave's band: a uniform address and the lane
  v8bf E[2][3];
  auto load_e = [&](int part, int kc) {
    const bool in = mine(kc);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const v8bf* p = in ? P + ((int64_t)kc * 6 + 2 * q + part) * 64 : zb;
      E[part][q] = p[(unsigned)lane];
    }
  };
  // products of one part's planes with both parts of the staged chunk: part 0 into rr and ri, part
  // 1 into ir and ii
  auto mma = [&](int part, int buf) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      // one column block's operands at a time (keeps the next block's LDS reads from being
      // hoisted, which would hold twice the registers)
      if (nb > 0) __builtin_amdgcn_sched_barrier(0);
      v8bf X[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) X[q] = *reinterpret_cast<const v8bf*>(&xb[buf][q][nb][lane][0]);
      if (part == 0) {
        rr[nb] = mma3(rr[nb], E[0][0], E[0][1], E[0][2], X[0], X[1], X[2]);
        ri[nb] = mma3(ri[nb], E[0][0], E[0][1], E[0][2], X[3], X[4], X[5]);
      } else {
        ii[nb] = mma3(ii[nb], E[1][0], E[1][1], E[1][2], X[3], X[4], X[5]);
        ir[nb] = mma3(ir[nb], E[1][0], E[1][1], E[1][2], X[0], X[1], X[2]);
      }
    }
  };
  // Chunk kc: its real planes' products, then the next chunk's real planes into the same
  // registers, then the imaginary ones alike: each set of planes is loaded half a chunk of
  // products ahead of its use, without a second set of registers.
  load_state(klo);
  load_e(0, klo);
  load_e(1, klo);
  store_state(0);
  __syncthreads();
  for (int kc = klo; kc < khi; ++kc) {
    const int buf = (kc - klo) & 1;
    const bool in = mine(kc);
    load_state(kc + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (in) mma(0, buf);
    __builtin_amdgcn_sched_barrier(0);
    load_e(0, kc + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (in) mma(1, buf);
    __builtin_amdgcn_sched_barrier(0);
    load_e(1, kc + 1);
    if (kc + 1 >= khi) break;
    store_state(buf ^ 1);
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

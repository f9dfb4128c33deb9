// Internal declarations shared by the host library and the HIP kernels of liblsx.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "lsx.h"

namespace lsx {

// ---------------------------------------------------------------- errors
void set_error(const std::string& msg);
#define LSX_HIP_TRY(expr)                                                                   \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      ::lsx::set_error(std::string(#expr) + ": " + hipGetErrorString(e_));                  \
      return LSX_E_HIP;                                                                     \
    }                                                                                       \
  } while (0)

// Launch bounds of the kernels with matrix instructions.  Left to itself the compiler gives a
// workgroup of up to four waves the whole register file (512 per lane), selects the matrix
// instructions' accumulation-register form and then copies every accumulator to and from the
// ordinary registers around each loop pass.  Asking for two waves per SIMD caps a lane at 256
// registers, which selects the form that accumulates in ordinary registers, with no copies:
// a loop of six independent FP64 accumulator chains ran at 32.5 TF with them and at 67.6 TF
// without at one wave per SIMD, 47.8 and 77.7 TF at four.  `cap` is false for the shapes whose
// accumulators and operands do not fit 256 registers (they would spill in the loop).
#define LSX_MFMA_BOUNDS(threads, cap) __launch_bounds__(threads, (cap) ? 2 : 1)

// ---------------------------------------------------------------- storage formats
// Propagator storage, per fibre f of length L (all formats zero-padded):
//  PF_F64    : complex128 P, Lp = roundup(L,16); chunk (rb, ks) = rows 16rb.., cols 4ks..
//              holds 64 double2, lane l = (row%16) + 16*(col%4).  Chunk index rb*(Lp/4)+ks.
//              This is exactly the A-operand order of v_mfma_f64_16x16x4f64.
//  PF_F32    : the off-diagonal part E of P as complex64 in the same chunk order
//              (A-operand order of v_mfma_f32_16x16x4f32), diagonal held in FP64 separately.
//  PF_BF16X3 : E split into three bf16 terms; Lp = roundup(L,32); chunk (rb, kc) = rows
//              16rb.., cols 32kc..; per chunk 6 planes (term*2 + {re,im}) of 64 lanes x 8
//              bf16, lane l = (row%16) + 16*((col%32)/8), element col%8 -- the A-operand
//              order of v_mfma_f32_16x16x32_bf16.
enum PropFormat { PF_F64 = 0, PF_F32 = 1, PF_BF16X3 = 2 };

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
inline int prop_pad(int fmt) { return fmt == PF_BF16X3 ? 32 : 16; }
// size in bytes of one fibre's propagator storage
inline int64_t prop_bytes(int fmt, int L) {
  int64_t Lp = round_up(L, prop_pad(fmt));
  switch (fmt) {
    case PF_F64: return Lp * Lp * 16;
    case PF_F32: return Lp * Lp * 8;
    default: return Lp * Lp * 12;  // 3 terms x (re, im) x bf16
  }
}

// Tile of a fibre pass (48 bytes, read with scalar loads): fibre f starting at fibre
// position r0 with length L, output rows 16*rb.., columns 16*NB*wb.., the byte offset of
// the fibre's propagator and of its diagonal, and the band [k0, k1) of fibre positions
// whose propagator columns hold an entry above the plan's band tolerance for any of the
// tile's rows (multiples of the format's column chunk; the kernels clamp k1 to the padded
// fibre length, so k1 = INT32_MAX means "to the end").  bb: entry of the propagator's first
// 16-row block in the per-block band table (PassArgs::rb_band), -1 when the tile has none.
// f < 0 marks a padding tile.
struct TileDesc {
  int32_t r0, L, rb, wb;
  int64_t poff;
  int32_t f;
  int32_t d0;  // mixed formats: position of this propagator's diagonal (fibres may share one)
  int32_t k0, k1;
  int32_t bb, pad_;
};
constexpr int32_t kBandEnd = 0x7fffffff;
// columns per propagator chunk of a format (the unit of the band)
inline int band_chunk(int fmt) { return fmt == PF_BF16X3 ? 32 : 4; }
// Fibres sharing a stored propagator are grouped by up to kOrbitMax; single-state passes
// over such groups use the tile shape nb = kOrbitNB (PassArgs::orbit).
constexpr int kOrbitMax = 8;
constexpr int kOrbitStride = 1 + kOrbitMax;
constexpr int kOrbitNB = 8;

struct PassArgs;
// Size of a plan's buffer of zeros: the widest load from it is a 16-byte operand for each of the 64 lanes
// (the row-split passes read it at the lane, as they read a propagator chunk).
constexpr int kZeroBytes = 64 * 16;

// Arguments of every fibre-pass kernel.  Element k of fibre f (fibre position
// p = r0 + k) is row in_pos[p] of X and row out_pos[p] of Y (identity when null),
// so a pass can read one array layout and write another.
// Weighted single-state passes (wt set): the output is x + wt[f] (P_f x - x) per fibre f, i.e. a
// weighted fibre increment; tcount (device) bounds the tiles a launch runs.
struct PassArgs {
  const TileDesc* tiles = nullptr;
  const int32_t* in_pos = nullptr;
  const int32_t* out_pos = nullptr;
  const int32_t* ph_idx = nullptr;  // canonical index of fibre position p (identity when null)
  const double2* ph = nullptr;      // kinetic phase applied to the output rows (none when null)
  const void* P = nullptr;          // propagator storage (format per kernel)
  const double2* diag = nullptr;    // mixed formats: diagonal of P at fibre position p
  const double2* X = nullptr;       // input state  [rows][W]
  double2* Y = nullptr;             // output state [rows][W]
  const void* zero = nullptr;       // kZeroBytes zero bytes: target of every out-of-range operand load
  const PassArgs* batch = nullptr;  // batched launches: per-system arguments, indexed by TileDesc::f
  const double* wt = nullptr;       // weighted single-state passes: [fibre] increment weights
  const int32_t* tcount = nullptr;  // device tile count: workgroups at or past it exit
  // row-split passes: band of every 16-row block of the layer's stored propagators, (k0, k1)
  // fibre positions at [2 (TileDesc::bb + block)]; each wave of a tile then skips the chunks
  // outside its own block's band (null: the tile's band for every wave)
  const int32_t* rb_band = nullptr;
  // persistent batched launches: mode (0 none, 1 per-XCD tile queues on device counters,
  // 2 static stride), 9 device counters that are zero between launches (mode 1) and the
  // number of tiles in `tiles`
  int32_t persist = 0;
  int32_t* queue = nullptr;
  int32_t ntiles = 0;
  int32_t W = 0;
  // output stores: 0 ordinary (lines kept in the writer's L2), 1 non-temporal (streamed out);
  // the faster one depends on the state's size and is measured per state
  int32_t nt = 0;
  // K-split FP64 / FP32 passes: groups of k-steps each wave keeps in flight (1, 2 or 4; 0: the
  // library default), chosen per state by the tile tuner
  int32_t u = 0;
  // single-state orbit passes (W = 1, tile shape nb = kOrbitNB): TileDesc::f indexes this
  // table of fibre groups that share one stored propagator, kOrbitStride entries per group:
  // the member count, then the fibre position of every member's first row (entries past the
  // count repeat the first member's); orbit_max is the largest group of the layer
  const int32_t* orbit = nullptr;
  int32_t orbit_max = 0;
};

// ---------------------------------------------------------------- kernel launchers (lsx_kernels.hip)
hipError_t launch_assemble(hipStream_t s, int nb, int maxn, const int32_t* fid, const int32_t* ptr, const int32_t* rows,
                           const int32_t* mn, int d, int stride, int own, double kfac, const double* K2, int nv,
                           const int32_t* vidx, const double* vre, const double* vim, int embed, double* A,
                           const int64_t* moff, const int32_t* ndim);
// Blocked two-sided Jacobi (long fibres): arguments of one round.  Matrices are indexed by their
// slot m (moff, ndim: padded size, a multiple of 32).  mat lists this sweep's unconverged
// matrices by size, largest first; a round runs on the first `count` of them (those with more
// than `round` + 1 blocks of 16), maxn the largest.  pfx_pairs is the prefix sum over mat of nb/2
// pairs (nb = n/16); Q holds every pair's 32x32 rotation (row-major) at its pfx_pairs index,
// rotated[] whether it has any rotation; flag[m] is set to 1 when matrix m was rotated; tiny[m] is
// its skip threshold.
struct BJArgs {
  double* A = nullptr;
  double* VT = nullptr;
  const int64_t* moff = nullptr;
  const int32_t* ndim = nullptr;
  double* tiny = nullptr;
  const int32_t* mat = nullptr;
  const int32_t* pfx_pairs = nullptr;
  int round = 0;
  double* Q = nullptr;
  int32_t* rotated = nullptr;
  int32_t* flag = nullptr;
};
hipError_t launch_bj_init(hipStream_t s, int nsel, const int32_t* sel, const BJArgs& g);
hipError_t launch_bj_round(hipStream_t s, int count, int maxn, const BJArgs& g);
hipError_t launch_bj_finish(hipStream_t s, int nsel, const int32_t* sel, const BJArgs& g, double* lam,
                            const int64_t* loff);

// Scalar cyclic Jacobi, one workgroup per matrix; sel (nullable) lists the matrices to solve.
hipError_t launch_jacobi(hipStream_t s, int nf, int maxn, double* A, double* VT, const int64_t* moff,
                         const int32_t* ndim, double* lam, const int64_t* loff, int32_t* info,
                         int maxsweeps, const int32_t* sel = nullptr);
hipError_t launch_eig_fn(hipStream_t s, int64_t nlam, const double* lam, double t, int flow, double2* gh);
hipError_t launch_form(hipStream_t s, int fmt, int nb, int maxL, const int32_t* fid, const int32_t* ptr,
                       const double* VT, const int64_t* moff, const int32_t* ndim, const int32_t* embed,
                       const double2* gh, const int64_t* loff, void* P, const int64_t* poff, double2* diag);
// Band of every 16-row block of every stored propagator (k_band): band[2 (boff[b] + rb)] and
// band[2 (boff[b] + rb) + 1] = first and one past the last column chunk with an entry whose
// |Re| + |Im| >= tol (a block with none keeps its diagonal chunk).
hipError_t launch_band(hipStream_t s, int fmt, int nb, int maxL, const int32_t* fid, const int32_t* ptr, const void* P,
                       const int64_t* poff, const int64_t* boff, double tol, int32_t* band);
hipError_t launch_phase_table(hipStream_t s, int64_t N, const double* K2, double theta_scale, double2* ph);
hipError_t launch_phase_apply(hipStream_t s, int64_t N, int W, const double2* ph, double2* c);
hipError_t launch_pass(hipStream_t s, int fmt, int W, int ntiles, int nb, int ksplit, const PassArgs& a,
                       bool batched = false);
// Sampled passes of several wavepackets (k_pass_slots).  The drawn (fibre, wavepacket) pairs of all
// fibres that share a stored propagator are its class's slots; their columns lie compacted in Xc,
// class c as [L][n[c]] at xbase[c], slot s with its fibre's first position, wavepacket and weight at
// slot[sbase[c] + s].  A unit is one 16-row block of one class's propagator.
struct SlotUnit {
  int64_t poff;
  int32_t cls, L, rb, d0, k0, k1;  // k0, k1 as TileDesc
};
struct Slot {
  int32_t r0, w;
  double g;
};
struct SlotArgs {
  const SlotUnit* units = nullptr;
  const int32_t* n = nullptr;
  const int64_t* xbase = nullptr;
  const int32_t* sbase = nullptr;
  const Slot* slot = nullptr;
  const double2* Xc = nullptr;
  double2* Y = nullptr;             // the state [rows][W], canonical order, updated in place
  const int32_t* pos = nullptr;     // canonical index of a fibre position (identity when null)
  const double2* pend = nullptr;    // pending phase: the state's true value is pend[row] times the stored one
  const void* P = nullptr;
  const double2* diag = nullptr;
  const void* zero = nullptr;
  int W = 0;
};
// max_slots: most slots a class can have; ks: waves splitting the fibre length (1, 2 or 4)
hipError_t launch_pass_slots(hipStream_t s, int fmt, int nunits, int max_slots, int ks, const SlotArgs& a);
// row-split tiles (lsx_rowsplit.hip): ms waves on consecutive row blocks of 16 nb columns
hipError_t launch_rowsplit(hipStream_t s, int fmt, int ntiles, int nb, int ms, const PassArgs& a);
// Batched launches with a.persist set: computes (once per kernel) the persistent grid of the pass
// kernel launch_pass would use, launching nothing, so no occupancy query runs under capture.
hipError_t prepare_persistent(int fmt, int W, int nb, int ksplit, const PassArgs& a);
// The rows as eight parts, part x = positions [start[x], start[x + 1]) of the row list `order` (null:
// the canonical order): the kernels that read every row's potential neighbours let XCD x sweep part
// x, kSweepCW columns at a time.  A part holds the rows of a range of layer-1 fibres, in canonical
// order, so that the layer-1 neighbours, up to tens of thousands of rows away, lie in the same
// part, and the rows between a neighbour's first and last use are an eighth of what a contiguous
// slab of the canonical order would have between them: they fit the XCD's 4 MB of L2.
struct Sweep {
  const int32_t* order = nullptr;
  int32_t start[9] = {};
};
constexpr int kSweepCW = 32;

// One term of the energy's potential part: neighbour nbr[i * nv + col] of row i with value v (the
// coefficient plus the conjugate of its partner at the opposite index)
struct EnergyTerm {
  const int32_t* nbr;
  int32_t nv, col;
  double2 v;
};
constexpr int kEnergyTermGroup = 6;  // the term lists are padded to a multiple of this
// Mass and energy of every column: partial sums of nblocks workgroups into pmass / penergy
// ([nblocks][W] each), then the sums into mass / energy (either null: not computed).  v0: the
// potentials' coefficient at index zero.
struct ReduceArgs {
  Sweep sweep;
  int W = 0;
  int CW = 0;  // columns per sweep (set by the launcher)
  const double2* c = nullptr;
  const double2* zero = nullptr;
  const double* K2 = nullptr;
  const EnergyTerm* terms = nullptr;
  int nterms = 0;
  double v0 = 0.0;
  double* pmass = nullptr;
  double* penergy = nullptr;
};
// Resident steps (lsx_resident.hip).  Row p of a layer's order: its propagator's first stored
// element of the row's band (lane 0 of the four that share the row), the state position of the
// band's first column, one past the fibre's last, the number of k-steps (chunks for BF16x3), the
// position of its diagonal entry and its canonical index.
struct ResidentRow {
  int64_t base;
  int32_t x0, lim, n, d;
  int32_t canon, pad_;
};
struct ResidentPass {
  const ResidentRow* rows;
  const int32_t* out_pos;  // as PassArgs
  const double2* ph;
  const void* P;
  const double2* diag;
};
constexpr int kResidentPasses = 32;  // distinct entries of a sequence
// Passes [begin, end) of the sequence pass[0 .. nhead), the following nbody entries reps times, then
// the ntail after them, on state X (gathered through in_pos: the first pass's order) into Y in the
// last pass's output order; X and Y may be the same array.
struct ResidentArgs {
  ResidentPass pass[kResidentPasses];
  int nhead = 0, nbody = 0, ntail = 0;
  int64_t reps = 0, begin = 0, end = 0;
  int N = 0, W = 0;
  const int32_t* in_pos = nullptr;
  const double2* X = nullptr;
  double2* Y = nullptr;
};
constexpr int kResidentU = 6;  // propagator entries a lane loads together: 24 columns of the band
// pair: a body of two passes, at most 256 rows, bands of at most kResidentU k-steps (not BF16x3)
hipError_t launch_resident(hipStream_t s, int fmt, const ResidentArgs& a, bool pair);
hipError_t launch_reduce(hipStream_t s, const ReduceArgs& a, int nblocks, double* mass, double* energy);
// n copies of whole arrays in one launch (max_elems: the longest)
struct CopyItem {
  const double2* from;
  double2* to;
  int64_t elems;
};
hipError_t launch_gather_rows(hipStream_t s, int64_t N, const int32_t* pos, const double2* src, double2* dst);
hipError_t launch_copy_home(hipStream_t s, int n, const CopyItem* items, int64_t max_elems);
hipError_t launch_fibre_mass(hipStream_t s, int nf, const int32_t* ptr, const int32_t* rows, int W,
                             const double2* c, double* out);
// Device address of this GPU's static scratch array (kStaticScratchDoubles doubles), looked up
// once per device on first use; never allocates.
constexpr int64_t kStaticScratchDoubles = int64_t(1) << 20;  // 8 MiB per GPU
constexpr int kMaxDevices = 64;
hipError_t static_scratch(double** ptr);

// ---------------------------------------------------------------- stochastic steps (lsx_sample.hip, lsx_mlp.hip)
hipError_t launch_si_step(hipStream_t s, const Sweep& sweep, int W, double tau, const double* K2, int nv1,
                          const int32_t* nbr1, const double2* v1, const double* wt1, const int32_t* fid1, int nv2,
                          const int32_t* nbr2, const double2* v2, const double* wt2, const int32_t* fid2,
                          const double2* X, double2* Y, const double2* zero);
hipError_t launch_subset_weights(hipStream_t s, int nf, int W, int p, int ustride, const double* u, double* wt);
hipError_t launch_sample_weights(hipStream_t s, int nf, int W, int p, int ustride, const double* u, const float* z,
                                 double eps, double* wt);
// single-state sampled passes: tiles of the sampled fibres
// bptr, band (nullable): band of fibre f's row block rb at band[2 (bptr[f] + rb)] (k0, then k1)
hipError_t launch_sampled_tiles(hipStream_t s, int nf, const double* wt, const int32_t* ptr, const int64_t* poff,
                                const int32_t* d0, const int32_t* bptr, const int32_t* band, int32_t* off,
                                TileDesc* tiles, int32_t* count);
hipError_t launch_copy_rows(hipStream_t s, int ntiles, const TileDesc* tiles, const int32_t* count,
                            const int32_t* pos, const double2* src, double2* dst);
// Slots of the sampled fibres (SlotArgs): fibres in class order qfib, class c of them at
// [cstart[c], cstart[c + 1]), its fibre length clen[c]; fcls: class of a fibre.  Fills the column
// lists cols [nf][W] / ncols, the slot offset of every fibre inside its class (off), the class tables
// n, xbase, sbase, the slots and the compacted columns Xc (times pend where set).
struct SlotBuild {
  int nf = 0, nc = 0, W = 0;
  const double* wt = nullptr;
  const int32_t* ptr = nullptr;
  const int32_t* qfib = nullptr;
  const int32_t* cstart = nullptr;
  const int32_t* clen = nullptr;
  const int32_t* fcls = nullptr;
  const int32_t* pos = nullptr;
  const double2* pend = nullptr;
  const double2* X = nullptr;
  int32_t* cols = nullptr;
  int32_t* ncols = nullptr;
  int32_t* off = nullptr;
  int32_t* n = nullptr;
  int64_t* xbase = nullptr;
  int32_t* sbase = nullptr;
  Slot* slot = nullptr;
  double2* Xc = nullptr;
};
hipError_t launch_slots(hipStream_t s, const SlotBuild& b);
hipError_t launch_fibre_incr(hipStream_t s, int nf, const int32_t* ptr, const int32_t* rows, int W,
                             const double2* X, const double2* Y, double* out);
hipError_t launch_features(hipStream_t s, int nf, int W, int d, const double* sfeat, const double* mass,
                           float sign, float* X);
// proposal network (width 64, FP32)
int mlp_nparams(int nin);
int mlp_bwd_blocks(int64_t M);
hipError_t launch_mlp_fwd(hipStream_t s, const float* theta, int nin, const float* X, int64_t M, float* z);
hipError_t launch_mlp_bwd(hipStream_t s, const float* theta, int nin, const float* X, int64_t M, const float* dz,
                          const double* gscale, float* partial, float* grad);
hipError_t launch_loss(hipStream_t s, const float* z, const double* b, const int64_t* gptr, int64_t G, double eps,
                       double* lg, int32_t* active, float* dz, double* out);
hipError_t launch_scale_f32(hipStream_t s, int64_t n, const double* scale, float* x);
hipError_t launch_adam(hipStream_t s, int n, float* theta, float* m, float* v, const float* grad, double lr,
                       double b1, double b2, double eps, double c1, double c2);

}  // namespace lsx

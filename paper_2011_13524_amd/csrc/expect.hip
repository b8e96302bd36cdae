// Tiled evaluation of <psi|O|psi> for a Pauli-string observable (section 4.5).
//
// A term with flip mask F pairs amplitude x with x ^ F, so it can be evaluated
// from any tile of the state whose local qubits include every qubit of F: both
// members of each pair are then in the same tile. The host groups the
// observable's flip masks into passes: a pass fixes L local qubits (always the
// low b ones, for contiguous HBM runs) chosen to hold as many flip masks as it
// can (pick_pass_local below); a mask with more flip qubits than a tile holds
// is evaluated on its own, its pairs read straight from the state. Each pass reads the
// state once into LDS, tile by tile, and evaluates every group of the pass on
// it. Workgroups are persistent and prefetch their next tile while computing
// on the current one; each sums its tiles in a fixed order into one FP64
// partial (passes run in order on one stream, so each partial has a single
// writer in a fixed order), and one final fixed-order reduction gives the
// value: bitwise reproducible. Compared with one pass per flip mask, HBM
// traffic drops by the number of masks per pass. Z/Y signs on non-local qubits
// are constants per tile. The same passes give lambda = O psi (adjoint).
#include <algorithm>
#include <cstdlib>
#include <initializer_list>
#include <mutex>

#include "dev_common.h"
#include "observable.h"
#include "prof.h"
#include "qsv_internal.h"

namespace qsv {

constexpr int kExpThreads = 512;
// largest tiles (expectation and lambda passes): 2^13 amplitudes, 64 KiB of
// complex64
constexpr int kExpTileMax = 8192;
// expectation workgroups: 512 threads over a 2^13-amplitude tile, so a
// single-term group gives each thread 8 pairs per tile (the group's scalar
// setup repeats per wave) and two workgroups (64 KiB of LDS each) keep 16
// waves on a compute unit; measured at 30 qubits complex64 against 256
// threads over 2^12 tiles (21 passes: 52.7 ms) and 256 over 2^13 (18
// passes but 8 waves per compute unit: 62.4 ms): 18 passes, 50.9 ms
constexpr int kExpThreadsE = 512;
constexpr int kExpMaxHigh = 16;
constexpr int kExpMaxGlobal = 40;

struct ExpPassDev {
  int L, b, nh, ng;
  int grp_begin, grp_count;
  int single_count;            // the first records of the pass: those of one term
  int span_begin, span_count;  // the same in spans (full tiles)
  int obs_begin, obs_real;     // the same for lambda: real coefficients first
  int obs_last;                // flip bits above the thread's of the last record
  int hq[kExpMaxHigh];
  int gpos[kExpMaxGlobal];
};

constexpr int kExpSteps = kExpTileMax / kExpThreadsE;  // per-thread steps over the largest tile

// A flip-mask group of a pass, with its first term folded in and, for
// expectation workgroups of kExpThreadsE threads, the workgroup-uniform parts
// of each step's indices and signs (the same for every tile of the pass).
struct ExpGroupDev {
  double re, im;   // first term: alpha * i^nY
  uint64_t zg;     // first term: sign mask on non-local qubits (global index space)
  uint32_t lf;     // flip mask in the tile's local index space
  uint32_t zl;     // first term: sign mask on local qubits
  int hbit;        // a set bit of lf (pairs are enumerated with it clear)
  int term_begin, term_count;
  uint32_t kind;  // ExpKind: which loop evaluates the record
  // lf != 0, kExpThreadsE-thread workgroups: bits below hbit, and the flip
  // bits inside the thread part of x = ins0(pair index, hbit)
  uint32_t hmask, lft;
  // lf != 0, step k (pair index k * kExpThreadsE + thread): the step part of
  // x = ins0(pair index, hbit) and of y = x ^ lf outside the thread's bits
  uint32_t offx[kExpSteps / 2], offy[kExpSteps / 2];
  // bit 31: parity of (step part of x) & zl (complex64 plans, lf != 0: as
  // the float +-1.0); for lf == 0 the step part of x is k * kExpThreadsE
  uint32_t sgn[kExpSteps];
};

// A span: the records whose flip masks lie in the linear span of `dim` basis
// masks (2^dim amplitudes per thread of a full tile: 4 complex64, 3 complex128).
// Every thread reads one coset into registers -- its representative XOR off[e],
// byte offsets -- and evaluates all of the records there: a tile is read from LDS
// once per span instead of once per record.
struct ExpSpanDev {
  uint32_t off[16];
  int pv[4];  // pivot bits, ascending (representatives have them clear)
  int rec_begin, rec_count;
};

// A record of a span.
struct alignas(16) ExpRecDev {
  uint32_t sgn[8];  // sign of the k-th pair's first element (flip mask 0: of element k), as in ExpGroupDev
  uint32_t s8;      // flip mask 0: bit 31, sign of the elements from 8 on against those before
  uint32_t zl;      // sign mask on local qubits
  uint32_t code;    // flip mask as a combination of the basis; bit 4: imaginary
  uint32_t pad;
  double c;         // factor of the sum over pairs (flip mask: 2 re or -2 im; none: re)
  uint64_t zg;      // sign mask on non-local qubits
};
constexpr int kSpanRecs = 512;  // records of a pass, at most (their factors for a tile sit in LDS)

// A single-term record of a lambda pass over a full tile. A thread's outputs y =
// thread + k x threads gather the amplitudes thread ^ lf + j x threads, j = k ^ (the
// flip bits above the thread's): the accumulators are kept in the order of j,
// exchanged where those bits change from one record to the next.
struct alignas(32) ObsRecDev {
  uint32_t lfb;    // flip bits inside the thread part, as a byte offset
  uint32_t zt;     // sign mask on the thread part
  uint32_t swap;   // bits b: exchange the accumulators j and j ^ (1 << b) first
  uint32_t s[3];   // bit 31: sign of the amplitudes with bit b of j set
  uint32_t pad[2];
};
struct ObsCoefDev {
  double c;     // alpha i^nY (its real or imaginary part) with the record's constant signs
  uint64_t zg;  // sign mask on non-local qubits
};

// Record kinds (set by the planner): one term with flip mask 0; several
// terms with flip mask 0; one term with a flip mask and a real (REAL) or
// imaginary (IMAG) coefficient alpha i^nY; several terms with a flip mask.
enum ExpKind : uint32_t { kExpZ1 = 0, kExpZN = 1, kExpFlipRe = 2, kExpFlipIm = 3, kExpFlipN = 4 };

struct ExpTermDev {
  double re, im;  // alpha * i^nY
  uint64_t zg;    // sign mask on non-local qubits (global index space)
  uint32_t zl;    // sign mask on local qubits (local index space)
  uint32_t pad;
};

// A term as staged in LDS for one tile: coefficient with the tile's sign on
// non-local qubits folded in, and the local sign mask.
struct ExpTermLds {
  double re, im;
  uint32_t zl;
};
constexpr int kExpLdsTerms = 128;
// Flip-mask groups of at most this many terms are split into single-term
// records: a shared multi-term record (FP64 sign sums per pair, terms staged
// in LDS) costs about six single-term ones or more; splitting masks of up to
// eight terms (not only up to four) took the 24-qubit 500-term lambda pass
// from 0.279 to 0.254 ms (complex64). Larger groups share the pair products.
constexpr int kExpSplitTerms = 8;
// persistent workgroups per observable pass: 8 per compute unit (2 resident
// at a time for the 512-thread expectation workgroups over 64 KiB tiles, 1
// for the lambda workgroups, which their registers limit); measured at 30
// qubits complex64: 2048 beats 1024 (shorter ranges even out the tail);
// QSV_EXPECT_GRID overrides
constexpr int kExpGrid = 2048;

// Workgroups that an expectation's launch aims at where the state has few tiles
// (a pass's groups are split until there are this many).
constexpr uint64_t kExpSplitGrid = 1024;

// Persistent grid of the expectation and lambda passes: kExpGrid, or the
// QSV_EXPECT_GRID override (tuning, and tests that give every workgroup a
// ragged range of several tiles at small sizes).
uint64_t exp_grid_max() {
  if (const char* e = std::getenv("QSV_EXPECT_GRID")) return uint64_t(std::max(1, std::atoi(e)));
  return kExpGrid;
}

// Persistent grid of the lambda passes: one workgroup per compute unit (all that
// its registers and LDS let in), so that each has several tiles and reads the
// next one while it computes. Measured, one lambda of 500 strings at 24 qubits
// complex64: 2048 workgroups (a tile each) 4.89 ms, 1024 4.17, 512 3.88, 256 3.75.
constexpr int kObsGrid = 256;
uint64_t obs_grid_max() {
  if (std::getenv("QSV_EXPECT_GRID")) return exp_grid_max();
  return kObsGrid;
}

// A group whose flip mask has more qubits than a tile holds (with the low
// ones): its terms are wide_terms[term_begin, term_begin + term_count), with
// zg the whole sign mask.
struct ExpWide {
  uint64_t flip;
  int hbit;  // highest bit of flip
  int term_begin, term_count;
};

struct ExpPlan {
  int n = 0, L = 0, b = 0;
  std::vector<ExpPassDev> passes;
  std::vector<ExpGroupDev> groups;
  std::vector<ExpTermDev> terms;
  // full tiles only, made for the first expectation / lambda: the records in spans /
  // for lambda, and the passes with their ranges (passes itself never changes)
  std::vector<ExpPassDev> span_passes, obs_passes;
  std::vector<ExpSpanDev> spans;
  std::vector<ExpRecDev> recs;
  std::vector<ObsRecDev> orecs;
  std::vector<ObsCoefDev> ocoef;
  std::vector<ExpWide> wide;
  std::vector<ExpTermDev> wide_terms;
  // device copies, each made once per device and kept: what one call uses is never
  // replaced by another kind of call
  struct Copy {
    void* p = nullptr;
    int device = -1;
  };
  Copy dev;        // passes | groups | terms | wide_terms
  Copy dev_spans;  // span_passes | spans | recs
  Copy dev_obs;    // obs_passes | orecs | ocoef
  bool spans_tried = false, orecs_tried = false;
};
// Guards the lazy parts of every observable's plans (building, upload); a plan's
// host tables and device copies do not change once made.
std::mutex g_plan_mu;

void free_exp_plan(ExpPlan* p) {
  if (!p) return;
  for (ExpPlan::Copy* c : {&p->dev, &p->dev_spans, &p->dev_obs})
    if (c->p) (void)hipFree(c->p);
  delete p;
}

// Local index -> global index bits of a pass (bit placement: linear over OR
// for local indices with disjoint bits, so per-thread and per-iteration parts
// are placed once and combined with one OR).
__device__ __forceinline__ uint64_t exp_place(const ExpPassDev& P, uint32_t j) {
  uint64_t x = j & ((1u << P.b) - 1);
  for (int i = 0; i < P.nh; ++i) x |= uint64_t((j >> (P.b + i)) & 1) << P.hq[i];
  return x;
}

__device__ __forceinline__ uint64_t exp_tile_base(const ExpPassDev& P, uint64_t g) {
  uint64_t base = 0;
  for (int j = 0; j < P.ng; ++j) base |= ((g >> j) & 1) << P.gpos[j];
  return base;
}

// -v when s is 1, v when 0 (one XOR into the sign bit).
__device__ __forceinline__ double flip_sign(double v, uint32_t s) {
  return __hiloint2double(__double2hiint(v) ^ int(s << 31), __double2loint(v));
}

// v with its sign bit XOR-ed with bit 31 of m.
__device__ __forceinline__ double xor_sign(double v, uint32_t m) {
  return __hiloint2double(__double2hiint(v) ^ int(m), __double2loint(v));
}
__device__ __forceinline__ float xor_sign(float v, uint32_t m) {
  return __uint_as_float(__float_as_uint(v) ^ m);
}

__device__ __forceinline__ uint32_t ins0(uint32_t i, int hb) {
  return ((i >> hb) << (hb + 1)) | (i & ((1u << hb) - 1));
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uni(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ uint64_t uni(uint64_t v) {
  // (readfirstlane yields a signed int: widen through uint32_t, no sign extension)
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v >> 32)));
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(v)));
  return (uint64_t(hi) << 32) | lo;
}

// Streaming of tiles through registers into LDS. Workgroups are persistent:
// workgroup b takes the contiguous range of tile indices [b per, (b + 1) per),
// per = ceil(tiles / grid), in increasing order (ExpTileRange below: the next
// tile's base is the current one carried within the non-local qubit mask), so
// its partial sum has a fixed order; the loads of its next tile are issued
// before it computes on the current one.
template <typename R, int NT, int LT = 0, int TMAX = kExpTileMax>
struct ExpTileStream {
  static constexpr int V = sizeof(R) == 4 ? 2 : 1;
  // loads per thread (16-byte pairs or complex128); TMAX: the largest tile in
  // 8-byte units (complex64 amplitudes)
  static constexpr int NL = TMAX / 2 / NT;
  uint64_t xt;          // per-thread part of the element addresses
  uint64_t xk[NL];      // workgroup-uniform parts
  cx<R> buf[NL * V];
  uint32_t TS;          // tile size (a constant when LT > 0: LT tile qubits)
  __device__ __forceinline__ ExpTileStream(const ExpPassDev& P) {
    TS = LT > 0 ? (1u << LT) : (1u << P.L);
    xt = exp_place(P, threadIdx.x * V);
#pragma unroll
    for (int k = 0; k < NL; ++k) xk[k] = exp_place(P, uint32_t(k) * NT * V);
  }
  __device__ __forceinline__ void fetch(const R* __restrict__ psi, uint64_t base) {
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const uint32_t e = threadIdx.x + uint32_t(k) * NT;
      if (e < TS / V) AmpIO<R, V>::load(psi, base | xt | xk[k], &buf[k * V]);
    }
  }
  __device__ __forceinline__ void to_lds(cx<R>* t) const {
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const uint32_t e = threadIdx.x + uint32_t(k) * NT;
      if (e < TS / V)
#pragma unroll
        for (int v = 0; v < V; ++v) t[e * V + v] = buf[k * V + v];
    }
  }
};

// Tiles of a workgroup: a contiguous range of tile indices (fixed order); the
// base of the next tile is the current one incremented within the mask of
// non-local qubits (a carry that skips local bit positions).
struct ExpTileRange {
  uint64_t g, end, base, gmask;
  __device__ __forceinline__ ExpTileRange(const ExpPassDev& P, uint64_t ntiles) {
    const uint64_t per = (ntiles + gridDim.x - 1) / gridDim.x;
    g = uint64_t(blockIdx.x) * per;
    end = g + per < ntiles ? g + per : ntiles;
    gmask = 0;
    for (int j = 0; j < P.ng; ++j) gmask |= uint64_t(1) << P.gpos[j];
    base = g < end ? exp_tile_base(P, g) : 0;
  }
  __device__ __forceinline__ uint64_t next_base() const { return ((base | ~gmask) + 1) & gmask; }
};

// Group gi of the pass with its first term's sign for the tile at base
// folded in (workgroup-uniform values, read through the scalar cache).
struct ExpGroup {
  double re, im;
  uint32_t lf, zl;
  int hbit, term_begin, term_count;
  uint32_t hmask, lft;
  const ExpGroupDev* d;
};

// The leading fields of a group record, read one group ahead so that their
// scalar loads overlap the current group's work; fold() gives the group with
// its first term's sign for the tile at base folded in.
struct ExpGroupHead {
  double re, im;
  uint64_t zg;
  uint32_t lf, zl;
  int hbit, term_begin, term_count;
  uint32_t kind, hmask, lft;
  __device__ __forceinline__ explicit ExpGroupHead(const ExpGroupDev& G)
      : re(G.re), im(G.im), zg(G.zg), lf(G.lf), zl(G.zl), hbit(G.hbit), term_begin(G.term_begin),
        term_count(G.term_count), kind(G.kind), hmask(G.hmask), lft(G.lft) {}
  __device__ __forceinline__ ExpGroup fold(uint64_t base, const ExpGroupDev* d) const {
    const uint32_t sg = uint32_t(__popcll(base & zg) & 1) << 31;
    return ExpGroup{xor_sign(re, sg), xor_sign(im, sg), lf, zl, hbit, term_begin, term_count, hmask, lft, d};
  }
};

// Stages the terms of a multi-term group for the tile at base (sign folded in).
__device__ __forceinline__ void exp_stage_terms(const ExpTermDev* __restrict__ terms, const ExpGroup& G,
                                                uint64_t base, ExpTermLds* et) {
  const int ns = min(G.term_count, kExpLdsTerms);
  for (int k = threadIdx.x; k < ns; k += blockDim.x) {
    const ExpTermDev T = terms[G.term_begin + k];
    const bool gneg = __popcll(base & T.zg) & 1;
    et[k] = {gneg ? -T.re : T.re, gneg ? -T.im : T.im, T.zl};
  }
}

__device__ __forceinline__ void exp_term(const ExpTermDev* __restrict__ terms, const ExpTermLds* et,
                                         const ExpGroup& G, uint64_t base, int k, double& re, double& im,
                                         uint32_t& zl) {
  if (k < kExpLdsTerms) {
    re = et[k].re;
    im = et[k].im;
    zl = et[k].zl;
  } else {
    const ExpTermDev T = terms[G.term_begin + k];
    const bool gneg = __popcll(base & T.zg) & 1;
    re = gneg ? -T.re : T.re;
    im = gneg ? -T.im : T.im;
    zl = T.zl;
  }
}

// Tile qubits of the fixed-size expectation and lambda kernel variants (64
// KiB tiles), and the lambda workgroup size and outputs per thread (1024
// threads: 8 complex64 or 4 complex128 outputs each; 512 threads with 8
// complex128 outputs took 181 VGPRs, two wavefronts per SIMD).
template <typename R>
__host__ __device__ constexpr int exp_tile_bits() {
  return sizeof(R) == 4 ? 13 : 12;
}
template <typename R>
__host__ __device__ constexpr int obs_tile_bits() {
  return sizeof(R) == 4 ? 13 : 12;
}
template <typename R>
__host__ __device__ constexpr int obs_threads() {
  return 1024;
}
template <typename R>
__host__ __device__ constexpr int obs_out() {
  return (1 << obs_tile_bits<R>()) / obs_threads<R>();
}

// Re (REAL) or Im of conj(b) a. complex64: formed in FP32 (relative error
// <= 2^-23 of |a||b|; see exp_pairs for the sums), which
// halves the vector instructions per pair against converting all four
// components first; complex128: FP64.
template <typename R, bool REAL>
__device__ __forceinline__ R pair_product(const cx<R>& a, const cx<R>& b) {
  return REAL ? fma(b.re, a.re, b.im * a.im) : fma(b.re, a.im, -(b.im * a.re));
}

// One single-term group with flip mask lf != 0 over a tile: the sum over the
// pairs (x, x ^ lf), x with bit hb clear, of Re (REAL) or Im of
// conj(psi_y) psi_x with the term's local Z/Y sign. A thread's pair products
// are summed in the amplitude precision in chunks of at most 8 (complex64:
// FP32, one conversion to FP64 per chunk instead of one per pair; with the
// products' own rounding the error is at most 9 x 2^-24 of the sum of
// |psi_x||psi_y| over the pairs, i.e. of <psi|psi>/2) and the chunks, threads
// and tiles in FP64. x is the thread
// part xt (tx = t + xt) OR-ed with a workgroup-uniform step part xs (disjoint
// bits); likewise y = (xt ^ (lf & thread bits)) | (xs ^ (lf outside them)),
// so each step adds a uniform offset to two per-thread LDS pointers. The sign
// splits the same way: pt (per thread, in bit 31) XOR the uniform parity of
// xs & zl. The uniform parts come precomputed with the group.
template <typename R, bool REAL, bool FULL, int NP, int NT>
__device__ __forceinline__ double exp_pairs(const cx<R>* tx, const cx<R>* ty, const ExpGroupDev& D, uint32_t pt,
                                            uint32_t TS, uint32_t tid) {
  // every LDS read of the group is issued before its arithmetic (one wait
  // instead of one per few pairs)
  cx<R> a[NP], b[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const uint32_t i0 = uint32_t(k) * NT;
    if (i0 < TS / 2 && (FULL || i0 + tid < TS / 2)) {
      a[k] = tx[D.offx[k]];
      b[k] = ty[D.offy[k]];
    } else {
      a[k] = b[k] = cx<R>{R(0), R(0)};  // zero product
    }
  }
  double sd = 0.0;
  R sw = R(0);
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if (uint32_t(k) * NT >= TS / 2) break;
    if constexpr (sizeof(R) == 4)  // complex64 plans store the step sign as +-1.0f
      sw = fmaf(__uint_as_float(D.sgn[k]), pair_product<R, REAL>(a[k], b[k]), sw);
    else
      sw += xor_sign(pair_product<R, REAL>(a[k], b[k]), D.sgn[k]);
    if ((k & 7) == 7) {  // sums of at most 8 products in the amplitude precision
      sd += double(sw);
      sw = R(0);
    }
  }
  sd += double(sw);  // (the loop may end early on small tiles)
  return xor_sign(sd, pt);  // the thread's part of the sign, common to every step
}

// An amplitude of a tile, by byte address (one aligned read).
__device__ __forceinline__ cx<float> lds_amp(const char* p, float) {
  const float2 t = *reinterpret_cast<const float2*>(p);
  return {t.x, t.y};
}
__device__ __forceinline__ cx<double> lds_amp(const char* p, double) {
  const double2 t = *reinterpret_cast<const double2*>(p);
  return {t.x, t.y};
}

// A span's record of flip code F: its pairs (e, e ^ F), e with F's highest bit
// clear, in registers; sums as in exp_pairs.
template <typename R, int RB, int F, bool REAL>
__device__ __forceinline__ double span_pairs(const cx<R>* v, const ExpRecDev& r) {
  constexpr int H = F >= 8 ? 3 : (F >= 4 ? 2 : (F >= 2 ? 1 : 0));
  R sw = R(0);
#pragma unroll
  for (int k = 0; k < (1 << (RB - 1)); ++k) {
    const int e = ((k >> H) << (H + 1)) | (k & ((1 << H) - 1));
    const R p = pair_product<R, REAL>(v[e], v[e ^ F]);
    if constexpr (sizeof(R) == 4) sw = fmaf(__uint_as_float(r.sgn[k]), p, sw);
    else sw += xor_sign(p, r.sgn[k]);
  }
  return double(sw);
}

template <typename R, int RB>
__device__ __forceinline__ double span_record(const cx<R>* v, const ExpRecDev& r) {
#define QSV_SPAN(F)                                             \
  case F: return span_pairs<R, RB, F, true>(v, r);              \
  case F + 16: return span_pairs<R, RB, F, false>(v, r);
#define QSV_SPAN_HI(F)                                          \
  case F:                                                       \
    if constexpr (RB == 4) return span_pairs<R, RB, F, true>(v, r); \
    break;                                                      \
  case F + 16:                                                  \
    if constexpr (RB == 4) return span_pairs<R, RB, F, false>(v, r); \
    break;
  switch (r.code) {
    QSV_SPAN(1) QSV_SPAN(2) QSV_SPAN(3) QSV_SPAN(4) QSV_SPAN(5) QSV_SPAN(6) QSV_SPAN(7)
    QSV_SPAN_HI(8) QSV_SPAN_HI(9) QSV_SPAN_HI(10) QSV_SPAN_HI(11)
    QSV_SPAN_HI(12) QSV_SPAN_HI(13) QSV_SPAN_HI(14) QSV_SPAN_HI(15)
    default: break;
  }
#undef QSV_SPAN
#undef QSV_SPAN_HI
  // flip mask 0: +-|psi_x|^2, summed in FP64
  double lo = 0.0, hi = 0.0;
#pragma unroll
  for (int e = 0; e < (1 << RB); ++e) {
    const double w = double(pair_product<R, true>(v[e], v[e]));
    if (e < 8) lo += xor_sign(w, r.sgn[e & 7] & 0x80000000u);
    else hi += xor_sign(w, r.sgn[e & 7] & 0x80000000u);
  }
  return lo + xor_sign(hi, r.s8);
}

// <psi|O|psi> over the tiles of one pass. Sums over threads and tiles are
// FP64; single-term groups form their products in the amplitude precision,
// and a flip group also sums each thread's 8 pairs per tile in it
// (complex64: |dE| <= 9 x 2^-24 sum |alpha| <psi|psi> beyond the stored
// amplitudes, see exp_pairs); multi-term groups work in FP64. Each workgroup sums its
// tiles in a fixed order into partial[blockIdx.x] (added to the value of
// earlier passes when accumulate is set). MODE 0: any tile size (per-lane
// guards); 1: the tile has at least two amplitudes per thread, so every loop
// below has a workgroup-uniform trip count; 2: the tile has exp_tile_bits<R>()
// qubits (trip counts known at compile time).
// 3: as 2, with the single-term records evaluated in spans: 200 strings of weight 4
// at 30 qubits complex64 32.0 ms reading LDS for each record, 27.5 ms in spans;
// complex128, 250 strings, 26 qubits 4.38 and 3.91 ms. What is left is the number of
// passes: 18 read 154.6 GB in 30.1 ms, 5.1 TB/s where streaming in place reaches
// 5.64 on this card (45 vector and 34 scalar instructions per record and wavefront
// keep the vector units 55% busy beside it). The records' factors with the tile's
// signs come from LDS (formed by one lane each; on the scalar unit 31.3 ms), and
// records are read where they are used (two at a time 28.2 ms).
// gridDim.y passes run in one launch, each split over gridDim.z ranges of its
// groups (workgroup b = x + gridDim.x (y + gridDim.y z) writes partial[b]).
template <typename R, int MODE>
__global__ void __launch_bounds__(kExpThreadsE)
    k_expect_tile(const R* __restrict__ psi, const ExpPassDev* __restrict__ passes, int pass_idx,
                  const ExpGroupDev* __restrict__ groups, const ExpTermDev* __restrict__ terms,
                  const ExpSpanDev* __restrict__ spans, const ExpRecDev* __restrict__ recs,
                  double* __restrict__ partial, int accumulate, uint64_t ntiles) {
  constexpr int NT = kExpThreadsE;
  constexpr int NA = kExpTileMax / NT;  // amplitudes per thread, at most
  constexpr bool FULL = MODE >= 1;
  constexpr int LT = MODE >= 2 ? exp_tile_bits<R>() : 0;
  constexpr bool SPANS = MODE == 3;
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[NT / 64];
  __shared__ ExpTermLds et[kExpLdsTerms];
  cx<R>* t = reinterpret_cast<cx<R>*>(smem);
  const ExpPassDev& P = passes[pass_idx + int(blockIdx.y)];
  // this workgroup's records: a range of the pass's groups, or of its spans and
  // then the groups that are in none
  const uint32_t items = uint32_t(SPANS ? P.span_count + P.grp_count - P.single_count : P.grp_count);
  int grp0 = int(items * blockIdx.z / gridDim.z), grp1 = int(items * (blockIdx.z + 1) / gridDim.z);
  int span0 = 0, span1 = 0;
  if (SPANS) {
    span0 = P.span_begin + min(grp0, P.span_count);
    span1 = P.span_begin + min(grp1, P.span_count);
    grp0 = max(grp0 - P.span_count, 0) + P.single_count;
    grp1 = max(grp1 - P.span_count, 0) + P.single_count;
  }
  const int grps = grp1 - grp0;
  __shared__ double cs[SPANS ? kSpanRecs : 1];  // the records' factors with the tile's signs
  const int rec0 = SPANS && span0 < span1 ? spans[span0].rec_begin : 0;
  const int nrec = SPANS && span0 < span1 ? spans[span1 - 1].rec_begin + spans[span1 - 1].rec_count - rec0 : 0;
  const uint32_t TS = LT > 0 ? (1u << LT) : (1u << P.L);
  const uint32_t tid = threadIdx.x;
  ExpTileStream<R, NT, LT> io(P);
  ExpTileRange tr(P, ntiles);
  double acc = 0.0;
  if (tr.g < tr.end) io.fetch(psi, tr.base);
  for (; tr.g < tr.end; ++tr.g) {
    const uint64_t base = tr.base;
    __syncthreads();  // previous tile consumed
    io.to_lds(t);
    if (SPANS && int(tid) < nrec) {
      const ExpRecDev& r = recs[rec0 + int(tid)];
      cs[tid] = xor_sign(r.c, uint32_t(__popcll(base & r.zg) & 1) << 31);
    }
    if (tr.g + 1 < tr.end) {
      tr.base = tr.next_base();
      io.fetch(psi, tr.base);
    }
    const ExpGroupDev* gd = groups + P.grp_begin + grp0;
    ExpGroupHead head(gd[0]);
    __syncthreads();  // tile (and, first time, the group table) in LDS
    if constexpr (SPANS) {
      constexpr int RB = exp_tile_bits<R>() - 9;  // 512 threads
      for (int si = span0; si < span1; ++si) {
        const ExpSpanDev& S = spans[si];
        uint32_t rep = tid;
#pragma unroll
        for (int j = 0; j < RB; ++j) rep = ins0(rep, S.pv[j]);
        cx<R> v[1 << RB];
#pragma unroll
        for (int e = 0; e < (1 << RB); ++e)
          v[e] = lds_amp(smem + ((rep * uint32_t(sizeof(cx<R>))) ^ S.off[e]), R(0));
        for (int ri = S.rec_begin; ri < S.rec_begin + S.rec_count; ++ri) {
          const ExpRecDev& r = recs[ri];
          const double c = cs[ri - rec0];
          // (the products of all codes are loop-invariant: formed ahead of the
          // loop they would take far more registers than there are)
#pragma unroll
          for (int e = 0; e < (1 << RB); ++e) asm volatile("" : "+v"(v[e].re), "+v"(v[e].im));
          const uint32_t pt = uint32_t(__popc(rep & r.zl)) << 31;
          acc += c * xor_sign(span_record<R, RB>(v, r), pt);
        }
      }
    }
    for (int left = grps; left > 0; --left, ++gd) {
      const ExpGroup G = head.fold(base, gd);
      const uint32_t kind = head.kind;
      head = ExpGroupHead(gd[1]);  // (after a pass's last record: the next pass's first, or the spare)
      const int nt = G.term_count;
      if (!SPANS && (kind == kExpFlipRe || kind == kExpFlipIm)) {
        // one term (the common case for random strings). A Hermitian term's
        // coefficient alpha i^nY is real (nY even) or imaginary (nY odd):
        // only Re or Im of w = conj(psi[y]) psi[x] counts
        const uint32_t xt = ((tid & ~G.hmask) << 1) | (tid & G.hmask);  // ins0(tid, hbit)
        const cx<R>* tx = t + xt;
        const cx<R>* ty = t + (xt ^ G.lft);
        uint32_t pt = uint32_t(__popc(xt & G.zl) & 1) << 31;
        if (kind == kExpFlipRe)
          acc += 2.0 * G.re * exp_pairs<R, true, FULL, NA / 2, NT>(tx, ty, *G.d, pt, TS, tid);
        else
          acc -= 2.0 * G.im * exp_pairs<R, false, FULL, NA / 2, NT>(tx, ty, *G.d, pt, TS, tid);
        continue;
      }
      if (nt > 1) {
        __syncthreads();
        exp_stage_terms(terms, G, base, et);
        __syncthreads();
      }
      if (!SPANS && kind == kExpZ1) {
        // sum of +-|psi_x|^2: thread part of the sign once, uniform part per step
        uint32_t pt = uint32_t(__popc(tid & G.zl) & 1) << 31;
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < NA; ++k) {
          const uint32_t j0 = uint32_t(k) * NT;
          if (j0 >= TS) break;
          if (FULL || j0 + tid < TS) {
            const cx<R> a = t[j0 + tid];
            sum += xor_sign(double(pair_product<R, true>(a, a)), G.d->sgn[k]);
          }
        }
        acc += G.re * xor_sign(sum, pt);
      } else if (kind == kExpZN) {
        for (uint32_t j = tid; j < TS; j += NT) {
          const cx<R> a = t[j];
          double c = 0.0;
          for (int k = 0; k < nt; ++k) {
            double re, im;
            uint32_t zl;
            exp_term(terms, et, G, base, k, re, im, zl);
            c += (__popc(j & zl) & 1) ? -re : re;
          }
          acc += (double(a.re) * a.re + double(a.im) * a.im) * c;
        }
      } else {  // kExpFlipN
        const int hb = G.hbit;
        const uint32_t lf = G.lf;
        for (uint32_t i = tid; i < TS / 2; i += NT) {
          const uint32_t x = ins0(i, hb);
          const cx<R> a = t[x], bb = t[x ^ lf];
          // w = conj(psi[y]) psi[x]
          const double wr = double(bb.re) * a.re + double(bb.im) * a.im;
          const double wi = double(bb.re) * a.im - double(bb.im) * a.re;
          double cr = 0.0, ci = 0.0;
          for (int k = 0; k < nt; ++k) {
            double re, im;
            uint32_t zl;
            exp_term(terms, et, G, base, k, re, im, zl);
            const bool neg = __popc(x & zl) & 1;
            cr += neg ? -re : re;
            ci += neg ? -im : im;
          }
          acc += 2.0 * (wr * cr - wi * ci);
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double r = 0.0;
    for (int w = 0; w < NT / 64; ++w) r += red[w];
    double* p = partial + blockIdx.x + size_t(gridDim.x) * (blockIdx.y + gridDim.y * blockIdx.z);
    *p = accumulate ? *p + r : r;
  }
}

template <typename R>
__global__ void __launch_bounds__(kExpThreads) k_zero_amps(R* __restrict__ a, uint64_t n) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    store1(a, i, cx<R>{R(0), R(0)});
}

// lambda = O psi over the tiles of one pass (the pass's flip masks only): every
// output y of a tile gathers psi[y ^ F] from LDS for each group F of the pass,
// with c(x) = sum over the group's terms of alpha i^nY (-1)^|x & z| (in FP64),
// summed per pass in the amplitude precision (that of lambda itself); the
// first pass writes lambda, later passes add to it.

// One single-term group's contribution to this thread's outputs: lambda_y +=
// c psi_{y ^ F} (REAL) or i c psi_{y ^ F} with c = +-coefficient, the sign of
// (-1)^|x & z| split into a per-thread bit (pt) and a per-step bit.
template <typename R, bool REAL, bool FIXED, int NT>
__device__ __forceinline__ void obs_single(const cx<R>* t, uint32_t tid, uint32_t lf, uint32_t zl, uint32_t pt,
                                           R cm, uint32_t TS, R* ar, R* ai) {
  constexpr int KO = obs_out<R>();
#pragma unroll
  for (int k = 0; k < KO; ++k) {
    const uint32_t y = tid + uint32_t(k) * NT;
    if (FIXED || y < TS) {
      const cx<R> v = t[y ^ lf];
      const R c = (pt ^ (__popc((uint32_t(k) * NT) & zl) & 1)) ? -cm : cm;
      if constexpr (REAL) {
        ar[k] += c * v.re;
        ai[k] += c * v.im;
      } else {
        ar[k] += -c * v.im;
        ai[k] += c * v.re;
      }
    }
  }
}

__device__ __forceinline__ void swap_regs(float& a, float& b) { asm volatile("v_swap_b32 %0, %1" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void swap_regs(double& a, double& b) {
  const double t = a;
  a = b;
  b = t;
}

// Exchanges accumulators j and j ^ (1 << b) for the bits b of m.
template <int KO, typename R>
__device__ __forceinline__ void obs_swap(uint32_t m, R* ar, R* ai) {
#pragma unroll
  for (int b = 1; b < KO; b <<= 1)
    if (m & uint32_t(b)) {
#pragma unroll
      for (int j = 0; j < KO; ++j)
        if (!(j & b)) {
          swap_regs(ar[j], ar[j | b]);
          swap_regs(ai[j], ai[j | b]);
        }
    }
}

// One record: acc_j += c_j psi (REAL) or i c_j psi, psi the thread's j-th gathered
// amplitude (one address, fixed offsets), c_j = +-c.
template <typename R, bool REAL, int NT>
__device__ __forceinline__ void obs_record(const char* smem, uint32_t tid, const ObsRecDev& r, R c, R* ar, R* ai) {
  constexpr int KO = obs_out<R>();
  const char* p = smem + ((tid * uint32_t(sizeof(cx<R>))) ^ r.lfb);
  cx<R> v[KO];
#pragma unroll
  for (int j = 0; j < KO; ++j) v[j] = lds_amp(p + j * NT * int(sizeof(cx<R>)), R(0));
  R cj[KO];
  cj[0] = xor_sign(c, uint32_t(__popc(tid & r.zt)) << 31);
#pragma unroll
  for (int j = 1; j < KO; ++j) {
    const int b = j >= 4 ? 2 : (j >= 2 ? 1 : 0);
    cj[j] = xor_sign(cj[j & ~(1 << b)], r.s[b]);
  }
#pragma unroll
  for (int j = 0; j < KO; ++j) {
    if constexpr (REAL) {
      ar[j] = fma(cj[j], v[j].re, ar[j]);
      ai[j] = fma(cj[j], v[j].im, ai[j]);
    } else {
      ar[j] = fma(-cj[j], v[j].im, ar[j]);
      ai[j] = fma(cj[j], v[j].re, ai[j]);
    }
  }
}

// RECS: the single-term records come as ObsRecDev: 28 vector instructions and
// four LDS reads of 16 bytes per record and thread (complex64), where forming
// each output's address and sign took about twice as many. One lambda, with the
// grid above: 500 strings at 24 qubits complex64 4.89 -> 2.98 ms (both grids
// alike: 3.75 -> 2.98), 200 strings at 28 qubits 31.4 -> 26.3; complex128, 250
// strings, 24 qubits 4.12 -> 3.26 ms.
// FIXED: the tile has obs_tile_bits<R>() qubits and every thread's outputs
// exist (complex64: 2^13 = 8 x 1024, complex128: 2^12 = 4 x 1024). Tiles of
// at most obs_out<R>() x NT amplitudes.
template <typename R, bool FIXED, int NT, bool RECS>
__global__ void __launch_bounds__(NT)
    k_apply_obs_tile(const R* __restrict__ psi, R* __restrict__ lam, const ExpPassDev* __restrict__ passes,
                     int pass_idx, const ExpGroupDev* __restrict__ groups,
                     const ExpTermDev* __restrict__ terms, const ObsRecDev* __restrict__ orecs,
                     const ObsCoefDev* __restrict__ ocoef, int accumulate, uint64_t ntiles) {
  constexpr int KO = obs_out<R>();
  __shared__ R cs[RECS ? kSpanRecs : 1];  // the records' coefficients with the tile's signs
  extern __shared__ __align__(16) char smem[];
  __shared__ ExpTermLds et[kExpLdsTerms];
  cx<R>* t = reinterpret_cast<cx<R>*>(smem);
  const ExpPassDev& P = passes[pass_idx];
  const uint32_t TS = FIXED ? (1u << obs_tile_bits<R>()) : (1u << P.L);
  const uint32_t tid = threadIdx.x;
  // (the stream's maximum counts 8-byte units: a complex128 tile of 4 x NT
  // amplitudes is 8 x NT of them)
  ExpTileStream<R, NT, 0, obs_out<R>() * NT * int(sizeof(R) / 4)> io(P);
  const uint64_t yt = exp_place(P, tid);
  uint64_t yk[KO];
#pragma unroll
  for (int k = 0; k < KO; ++k) yk[k] = exp_place(P, uint32_t(k) * NT);
  ExpTileRange tr(P, ntiles);
  if (tr.g < tr.end) io.fetch(psi, tr.base);
  for (; tr.g < tr.end; ++tr.g) {
    const uint64_t base = tr.base;
    __syncthreads();  // previous tile consumed
    io.to_lds(t);
    if (tr.g + 1 < tr.end) {
      tr.base = tr.next_base();
      io.fetch(psi, tr.base);
    }
    // per-pass sums in the amplitude precision (lambda is stored in it)
    R ar[KO], ai[KO];
#pragma unroll
    for (int k = 0; k < KO; ++k) ar[k] = ai[k] = R(0);
    if (RECS && int(tid) < P.single_count) {
      const ObsCoefDev& r = ocoef[P.obs_begin + int(tid)];
      cs[tid] = R(xor_sign(r.c, uint32_t(__popcll(base & r.zg) & 1) << 31));
    }
    const ExpGroupDev* gd = groups + P.grp_begin + (RECS ? P.single_count : 0);
    ExpGroupHead head(gd[0]);
    __syncthreads();  // tile (and, first time, the group table) in LDS
    if constexpr (RECS) {
      int i = 0;
      for (; i < P.obs_real; ++i) {
        const ObsRecDev& r = orecs[P.obs_begin + i];
        if (r.swap) obs_swap<KO>(r.swap, ar, ai);
        obs_record<R, true, NT>(smem, tid, r, cs[i], ar, ai);
      }
      for (; i < P.single_count; ++i) {
        const ObsRecDev& r = orecs[P.obs_begin + i];
        if (r.swap) obs_swap<KO>(r.swap, ar, ai);
        obs_record<R, false, NT>(smem, tid, r, cs[i], ar, ai);
      }
      obs_swap<KO>(uint32_t(P.obs_last), ar, ai);
    }
    for (int left = RECS ? P.grp_count - P.single_count : P.grp_count; left > 0; --left, ++gd) {
      const ExpGroup G = head.fold(base, gd);
      const uint32_t kind = head.kind;
      head = ExpGroupHead(gd[1]);  // (see k_expect_tile)
      const uint32_t lf = G.lf;
      if (!RECS && (kind == kExpZ1 || kind == kExpFlipRe || kind == kExpFlipIm)) {
        // alpha i^nY is real or imaginary (a Z-only string's is real):
        // lambda += c psi or i c psi
        const uint32_t pt = (__popc((tid ^ lf) & G.zl) & 1);
        if (kind != kExpFlipIm)
          obs_single<R, true, FIXED, NT>(t, tid, lf, G.zl, pt, R(G.re), TS, ar, ai);
        else
          obs_single<R, false, FIXED, NT>(t, tid, lf, G.zl, pt, R(G.im), TS, ar, ai);
        continue;
      }
      const int nt = G.term_count;
      __syncthreads();
      exp_stage_terms(terms, G, base, et);
      __syncthreads();
      {
#pragma unroll
        for (int k = 0; k < KO; ++k) {
          const uint32_t y = tid + uint32_t(k) * NT;
          if (y < TS) {
            const uint32_t x = y ^ lf;
            const cx<R> v = t[x];
            double cr = 0.0, ci = 0.0;
            for (int q = 0; q < nt; ++q) {
              double re, im;
              uint32_t zl;
              exp_term(terms, et, G, base, q, re, im, zl);
              const bool neg = __popc(x & zl) & 1;
              cr += neg ? -re : re;
              ci += neg ? -im : im;
            }
            ar[k] += R(cr * double(v.re) - ci * double(v.im));
            ai[k] += R(cr * double(v.im) + ci * double(v.re));
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < KO; ++k) {
      if (!FIXED && tid + uint32_t(k) * NT >= TS) continue;
      cx<R> r;
      if (accumulate) {
        const cx<R> old = load1(lam, base | yt | yk[k]);
        r = {old.re + ar[k], old.im + ai[k]};
      } else {
        r = {ar[k], ai[k]};
      }
      store1(lam, base | yt | yk[k], r);
    }
  }
}

// Groups whose flip mask F has more qubits than a tile holds: the pairs
// (x, x ^ F), x with the highest bit h of F clear, are read straight from the
// state (both members of a pair in one thread; consecutive threads read
// consecutive x). Each workgroup walks the pair indices in a fixed
// grid-stride order and adds its FP64 sum to partial[blockIdx.x], the
// partials of the tiled passes (same grid), so the value stays bitwise
// reproducible.
template <typename R>
__global__ void __launch_bounds__(kExpThreadsE)
    k_expect_wide(const R* __restrict__ psi, uint64_t flip, int hbit, const ExpTermDev* __restrict__ terms,
                  int nt, uint64_t pairs, double* __restrict__ partial, int accumulate) {
  __shared__ double red[kExpThreadsE / 64];
  const uint64_t stride = uint64_t(gridDim.x) * kExpThreadsE;
  const uint64_t lowm = (uint64_t(1) << hbit) - 1;
  double acc = 0.0;
  for (uint64_t i = uint64_t(blockIdx.x) * kExpThreadsE + threadIdx.x; i < pairs; i += stride) {
    const uint64_t x = ((i & ~lowm) << 1) | (i & lowm);
    const cx<R> a = load1(psi, x), bb = load1(psi, x ^ flip);
    // w = conj(psi[y]) psi[x]
    const double wr = double(bb.re) * a.re + double(bb.im) * a.im;
    const double wi = double(bb.re) * a.im - double(bb.im) * a.re;
    double cr = 0.0, ci = 0.0;
    for (int k = 0; k < nt; ++k) {
      const ExpTermDev T = terms[k];
      const bool neg = __popcll(x & T.zg) & 1;
      cr += neg ? -T.re : T.re;
      ci += neg ? -T.im : T.im;
    }
    acc += 2.0 * (wr * cr - wi * ci);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < kExpThreadsE / 64; ++w) r += red[w];
    partial[blockIdx.x] = accumulate ? partial[blockIdx.x] + r : r;
  }
}

// lambda_y (+)= c(x) psi_x, x = y ^ F, for one group whose flip mask F has
// more qubits than a tile holds (c(x) as in the tiled passes, in FP64; the
// sum is stored in the amplitude precision).
template <typename R>
__global__ void __launch_bounds__(kExpThreads)
    k_apply_obs_wide(const R* __restrict__ psi, R* __restrict__ lam, uint64_t flip,
                     const ExpTermDev* __restrict__ terms, int nt, uint64_t N, int accumulate) {
  const uint64_t stride = uint64_t(gridDim.x) * kExpThreads;
  for (uint64_t y = uint64_t(blockIdx.x) * kExpThreads + threadIdx.x; y < N; y += stride) {
    const uint64_t x = y ^ flip;
    const cx<R> v = load1(psi, x);
    double cr = 0.0, ci = 0.0;
    for (int k = 0; k < nt; ++k) {
      const ExpTermDev T = terms[k];
      const bool neg = __popcll(x & T.zg) & 1;
      cr += neg ? -T.re : T.re;
      ci += neg ? -T.im : T.im;
    }
    cx<R> r{R(cr * double(v.re) - ci * double(v.im)), R(cr * double(v.im) + ci * double(v.re))};
    if (accumulate) {
      const cx<R> old = load1(lam, y);
      r = {old.re + r.re, old.im + r.im};
    }
    store1(lam, y, r);
  }
}

__global__ void __launch_bounds__(kExpThreads)
    k_exp_sum(const double* __restrict__ partial, uint64_t count, double* __restrict__ out) {
  __shared__ double red[kExpThreads / 64];
  double acc = 0.0;
  for (uint64_t i = threadIdx.x; i < count; i += blockDim.x) acc += partial[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < kExpThreads / 64; ++w) r += red[w];
    out[0] = r;
  }
}

namespace {

int popc64(uint64_t x) { return __builtin_popcountll(x); }

// Local qubit set of the next pass, given the flip masks hi (low qubits
// removed) of the groups not yet evaluated; low: the always-local low qubits.
// The set is grown from a seed mask by adding, one at a time, the mask that
// needs the fewest new local qubits (ties: the one after which most masks lie
// inside the set), up to L qubits; of the sets grown from up to kPackSeeds
// seeds (spread over the list), the one holding the most masks is kept. On
// random weight-4 strings at 30 qubits this takes 21 passes where adding
// masks to one set in list order takes 26.
constexpr int kPackSeeds = 64, kPackTies = 8;

uint64_t pick_pass_local(const std::vector<uint64_t>& hi, uint64_t low, int L) {
  const size_t nm = hi.size();
  auto inside = [&](uint64_t loc) {
    int c = 0;
    for (uint64_t g : hi) c += (g & ~loc) == 0;
    return c;
  };
  uint64_t best = low;
  int best_cov = -1;
  const size_t ns = std::min<size_t>(nm, kPackSeeds);
  std::vector<uint64_t> ties;
  for (size_t si = 0; si < ns; ++si) {
    uint64_t local = low | hi[si * nm / ns];
    while (true) {
      int mn = 65;
      ties.clear();
      for (uint64_t f : hi) {
        const uint64_t nf = f & ~local;
        if (!nf || popc64(local | f) > L) continue;
        const int need = popc64(nf);
        if (need < mn) {
          mn = need;
          ties.assign(1, f);
        } else if (need == mn && int(ties.size()) < kPackTies) {
          ties.push_back(f);
        }
      }
      if (ties.empty()) break;
      uint64_t pick = ties[0];
      if (ties.size() > 1) {
        int pc = -1;
        for (uint64_t f : ties) {
          const int c = inside(local | f);
          if (c > pc) {
            pc = c;
            pick = f;
          }
        }
      }
      local |= pick;
    }
    const int c = inside(local);
    if (c > best_cov) {
      best_cov = c;
      best = local;
    }
  }
  return best;
}

// Moves flip-mask groups from heavily loaded passes to lighter ones whose
// local set also holds their mask (the packing above fills the first passes
// and leaves the last ones light). Cost of a pass in units of one
// single-term record's work (complex64, 30 qubits: 0.12 ms each), measured:
// max(10.9, 4.9 + records) -- at least its read of the state, and a fixed
// part per tile on top of its records; a shared record of more than
// kExpSplitTerms terms costs about six. A group moves when the modelled sum
// drops; deterministic (passes by load, groups in order).
void rebalance_passes(const std::vector<Group>& groups, const std::vector<uint64_t>& plocal,
                      std::vector<std::vector<int>>& pchosen) {
  const size_t np = plocal.size();
  auto weight = [&](int gi) { return groups[gi].count <= kExpSplitTerms ? double(groups[gi].count) : 6.0; };
  auto cost = [](double g) { return std::max(10.9, 4.9 + g); };
  std::vector<double> load(np, 0.0);
  for (size_t pi = 0; pi < np; ++pi)
    for (int gi : pchosen[pi]) load[pi] += weight(gi);
  for (int round = 0; round < 64; ++round) {
    bool moved = false;
    std::vector<size_t> order(np);
    for (size_t pi = 0; pi < np; ++pi) order[pi] = pi;
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return load[a] > load[b]; });
    for (size_t pa : order) {
      for (size_t k = 0; k < pchosen[pa].size();) {
        const int gi = pchosen[pa][k];
        const double w = weight(gi);
        size_t best = np;
        double bd = -1e-9;
        for (size_t pb = 0; pb < np; ++pb) {
          if (pb == pa || (groups[gi].flip & ~plocal[pb])) continue;
          const double d = cost(load[pa] - w) + cost(load[pb] + w) - cost(load[pa]) - cost(load[pb]);
          if (d < bd) {
            bd = d;
            best = pb;
          }
        }
        if (best == np) {
          ++k;
          continue;
        }
        pchosen[pa].erase(pchosen[pa].begin() + long(k));
        pchosen[best].push_back(gi);
        load[pa] -= w;
        load[best] += w;
        moved = true;
      }
    }
    if (!moved) break;
  }
}

// The single-term records of a pass in spans of `dim` basis masks: each span is
// grown from a seed mask by the mask after which most records lie inside, and the
// best of kSpanSeeds seeds is kept. With all masks reduced by the basis so far,
// the records that a new basis mask c brings in are those reduced to c.
constexpr size_t kSpanSeeds = 4;

struct SpanBasis {
  int dim = 0;
  uint32_t b[4];  // reduced: each has its highest bit (its pivot) alone
  uint32_t reduce(uint32_t m) const {
    for (int j = 0; j < dim; ++j)
      if (m >> (31 - __builtin_clz(b[j])) & 1) m ^= b[j];
    return m;
  }
  void add(uint32_t m) {  // m reduced, not 0
    const int p = 31 - __builtin_clz(m);
    for (int j = 0; j < dim; ++j)
      if (b[j] >> p & 1) b[j] ^= m;
    b[dim++] = m;
  }
};

void build_spans(ExpPlan* p, ExpPassDev& d, int dim, bool c64) {
  const ExpGroupDev* g = p->groups.data() + d.grp_begin;
  const size_t S = c64 ? 8 : 16;  // bytes per amplitude
  std::vector<int> left;
  for (int i = 0; i < d.single_count; ++i) left.push_back(i);
  d.span_begin = int(p->spans.size());
  while (!left.empty()) {
    SpanBasis best;
    int best_w = -1;
    std::vector<uint32_t> red, run;
    size_t seeds = 0;
    for (size_t a = 0; a < left.size() && seeds < kSpanSeeds; ++a) {
      uint32_t add = g[left[a]].lf;
      if (add == 0) continue;
      ++seeds;
      SpanBasis B;
      red.clear();
      for (int i : left) red.push_back(g[i].lf);
      for (;;) {
        B.add(add);
        const int pv = 31 - __builtin_clz(add);
        for (uint32_t& m : red)
          if (m >> pv & 1) m ^= add;
        if (B.dim == dim) break;
        run = red;
        std::sort(run.begin(), run.end());
        int most = 0;
        for (size_t i = 0, j = 0; i < run.size(); i = j) {
          while (j < run.size() && run[j] == run[i]) ++j;
          if (run[i] && int(j - i) > most) {
            most = int(j - i);
            add = run[i];
          }
        }
        if (most == 0) break;
      }
      const int w = int(std::count(red.begin(), red.end(), 0u));
      if (w > best_w) {
        best_w = w;
        best = B;
      }
    }
    for (int q = d.L - 1; best.dim < dim; --q)  // (few masks: any other directions)
      if (const uint32_t m = best.reduce(1u << q)) best.add(m);
    std::sort(best.b, best.b + dim);  // pivots ascending
    ExpSpanDev s{};
    for (int e = 0; e < (1 << dim); ++e)
      for (int j = 0; j < dim; ++j)
        if (e >> j & 1) s.off[e] ^= best.b[j] * uint32_t(S);
    for (int j = 0; j < dim; ++j) s.pv[j] = 31 - __builtin_clz(best.b[j]);
    s.rec_begin = int(p->recs.size());
    std::vector<int> rest;
    for (int i : left) {
      const ExpGroupDev& G = g[i];
      if (best.reduce(G.lf)) {
        rest.push_back(i);
        continue;
      }
      ExpRecDev r{};
      r.zg = G.zg;
      r.zl = G.zl;
      for (int j = 0; j < dim; ++j) r.code |= (G.lf >> s.pv[j] & 1) << j;
      const int top = r.code ? 31 - __builtin_clz(r.code) : 0;
      r.c = !r.code ? G.re : (G.kind == kExpFlipRe ? 2.0 * G.re : -2.0 * G.im);
      for (int k = 0; k < 8; ++k) {
        const int e = (r.code ? ((k >> top) << (top + 1)) | (k & ((1 << top) - 1)) : k) & ((1 << dim) - 1);
        r.sgn[k] = uint32_t(__builtin_popcount(s.off[e] / uint32_t(S) & G.zl) & 1) << 31 | (c64 ? 0x3f800000u : 0u);
      }
      if (dim == 4) r.s8 = uint32_t(__builtin_popcount(best.b[3] & G.zl) & 1) << 31;
      if (G.kind == kExpFlipIm) r.code |= 16;
      p->recs.push_back(r);
    }
    s.rec_count = int(p->recs.size()) - s.rec_begin;
    p->spans.push_back(s);
    left.swap(rest);
  }
  d.span_count = int(p->spans.size()) - d.span_begin;
}

ExpPlan* build_exp_plan(const qsv_observable* o, qsv_dtype dt) {
  std::vector<Group> groups;
  std::vector<GTerm> terms;
  build_groups(o, groups, terms);
  ExpPlan* p = new ExpPlan();
  const int n = o->n;
  p->n = n;
  // tile: 2^L amplitudes, 64 KiB (2^13 complex64, 2^12 complex128): more
  // flip masks fit a pass (18 expectation passes instead of 21 for the
  // 200-term 30-qubit observable); QSV_EXPECT_TILE lowers L, for tuning
  int Ldef = dt == QSV_C64 ? 13 : 12;
  if (const char* e = std::getenv("QSV_EXPECT_TILE")) Ldef = std::max(6, std::min(Ldef, std::atoi(e)));
  p->L = std::min(n, Ldef);
  int bdef = dt == QSV_C64 ? 4 : 3;  // 128-byte contiguous runs
  if (const char* e = std::getenv("QSV_EXPECT_LOW")) bdef = std::max(1, std::min(8, std::atoi(e)));
  p->b = std::min(p->L, bdef);
  const int L = p->L, b = p->b;
  const uint64_t low = (uint64_t(1) << b) - 1;
  std::vector<int> rem;
  for (size_t i = 0; i < groups.size(); ++i) {
    if (popc64(groups[i].flip | low) <= L) {
      rem.push_back(int(i));
      continue;
    }
    // more flip qubits than a tile holds: evaluated on its own, pairs read
    // straight from the state
    const Group& G = groups[i];
    ExpWide w{G.flip, 63 - __builtin_clzll(G.flip), int(p->wide_terms.size()), G.count};
    for (int k = G.begin; k < G.begin + G.count; ++k)
      p->wide_terms.push_back(ExpTermDev{terms[k].re, terms[k].im, terms[k].z, 0u, 0u});
    p->wide.push_back(w);
  }
  std::vector<uint64_t> plocal;
  std::vector<std::vector<int>> pchosen;
  while (!rem.empty()) {
    std::vector<uint64_t> hi;
    for (int r : rem) hi.push_back(groups[r].flip & ~low);
    const uint64_t local0 = pick_pass_local(hi, low, L);
    std::vector<int> chosen, rest;
    for (int r : rem) ((groups[r].flip & ~local0) == 0 ? chosen : rest).push_back(r);
    rem.swap(rest);
    uint64_t local = local0;
    for (int q = 0; q < n && popc64(local) < L; ++q) local |= uint64_t(1) << q;
    plocal.push_back(local);
    pchosen.push_back(chosen);
  }
  rebalance_passes(groups, plocal, pchosen);
  for (size_t pi = 0; pi < plocal.size(); ++pi) {
    const uint64_t local = plocal[pi];
    const std::vector<int>& chosen = pchosen[pi];
    if (chosen.empty()) continue;  // (every group moved elsewhere)
    std::vector<int> lpos(64, -1), loc;
    for (int q = 0; q < 64; ++q)
      if (local >> q & 1) {
        lpos[q] = int(loc.size());
        loc.push_back(q);
      }
    ExpPassDev d{};
    d.L = L;
    d.b = b;
    d.nh = L - b;
    for (int i = 0; i < d.nh; ++i) d.hq[i] = loc[b + i];
    d.ng = 0;
    for (int q = 0; q < n; ++q)
      if (!(local >> q & 1)) d.gpos[d.ng++] = q;
    d.grp_begin = int(p->groups.size());
    for (int gi : chosen) {
      const Group& G = groups[gi];
      uint32_t lf = 0;
      for (int q = 0; q < n; ++q)
        if (G.flip >> q & 1) lf |= 1u << lpos[q];
      // a few terms on one flip mask run as that many single-term records
      // (the single-term loop, once per term); more share one record
      const int nrec = G.count <= kExpSplitTerms ? G.count : 1;
      for (int r = 0; r < nrec; ++r) {
        ExpGroupDev gd{};
        gd.lf = lf;
        gd.hbit = lf ? 31 - __builtin_clz(lf) : 0;
        gd.term_begin = int(p->terms.size());
        gd.term_count = nrec > 1 ? 1 : G.count;
        const double im0 = terms[G.begin + (nrec > 1 ? r : 0)].im;
        gd.kind = lf == 0 ? (gd.term_count == 1 ? kExpZ1 : kExpZN)
                          : (gd.term_count > 1 ? kExpFlipN : (im0 == 0.0 ? kExpFlipRe : kExpFlipIm));
        const int k0 = G.begin + (nrec > 1 ? r : 0);
        for (int k = k0; k < k0 + gd.term_count; ++k) {
          ExpTermDev td{};
          td.re = terms[k].re;
          td.im = terms[k].im;
          for (int q = 0; q < n; ++q) {
            if (!(terms[k].z >> q & 1)) continue;
            if (lpos[q] >= 0) td.zl |= 1u << lpos[q];
            else td.zg |= uint64_t(1) << q;
          }
          if (k == k0) {
            gd.re = td.re;
            gd.im = td.im;
            gd.zg = td.zg;
            gd.zl = td.zl;
          }
          p->terms.push_back(td);
        }
        // uniform step parts for kExpThreadsE-thread workgroups
        auto ins0h = [](uint32_t i, int hb) { return ((i >> hb) << (hb + 1)) | (i & ((1u << hb) - 1)); };
        const uint32_t mt = ins0h(kExpThreadsE - 1, gd.hbit);
        gd.hmask = (1u << gd.hbit) - 1;
        gd.lft = lf & mt;
        for (int k = 0; k < kExpSteps; ++k) {
          const uint32_t xs = lf ? ins0h(uint32_t(k) * kExpThreadsE, gd.hbit) : uint32_t(k) * kExpThreadsE;
          if (lf && k < kExpSteps / 2) {
            gd.offx[k] = xs;
            gd.offy[k] = xs ^ (lf & ~mt);
          }
          if (!lf || k < kExpSteps / 2) gd.sgn[k] = uint32_t(__builtin_popcount(xs & gd.zl) & 1) << 31;
          // flip records of complex64 plans: the sign as +-1.0f, applied by
          // one FMA into the running sum (exact: the same result as a sign
          // flip and an add)
          if (lf && k < kExpSteps / 2 && dt == QSV_C64) gd.sgn[k] |= 0x3f800000u;
        }
        p->groups.push_back(gd);
      }
    }
    d.grp_count = int(p->groups.size()) - d.grp_begin;
    d.single_count = int(std::stable_partition(p->groups.begin() + d.grp_begin, p->groups.end(),
                                               [](const ExpGroupDev& g) { return g.term_count == 1; }) -
                         (p->groups.begin() + d.grp_begin));
    p->passes.push_back(d);
  }
  // the kernels read each record's successor ahead of use: one spare record
  // after the last pass keeps that read inside the table
  if (!p->passes.empty()) p->groups.push_back(ExpGroupDev{});
  return p;
}

// The lambda records of a plan of full tiles (built for the first lambda pass).
void ensure_obs_recs(ExpPlan* p, bool c64) {
  if (p->orecs_tried) return;
  p->orecs_tried = true;
  if (p->L != (c64 ? obs_tile_bits<float>() : obs_tile_bits<double>())) return;
  for (const ExpPassDev& d : p->passes)
    if (d.single_count > kSpanRecs) return;
  constexpr int tb = 10;  // 1024 threads
  static_assert(obs_threads<float>() == 1 << tb && obs_threads<double>() == 1 << tb, "thread part of an index");
  p->obs_passes = p->passes;
  for (ExpPassDev& d : p->obs_passes) {
    const ExpGroupDev* g = p->groups.data() + d.grp_begin;
    std::vector<int> order;
    for (int i = 0; i < d.single_count; ++i) order.push_back(i);
    auto gray = [&](int i) {  // neighbours differ in one bit
      uint32_t h = g[i].lf >> tb, k = h;
      for (h >>= 1; h; h >>= 1) k ^= h;
      return k;
    };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
      const bool ia = g[a].kind == kExpFlipIm, ib = g[b].kind == kExpFlipIm;
      return ia != ib ? !ia : gray(a) < gray(b);
    });
    d.obs_begin = int(p->orecs.size());
    d.obs_real = 0;
    uint32_t cur = 0;
    for (int i : order) {
      const ExpGroupDev& G = g[i];
      const bool im = G.kind == kExpFlipIm;
      d.obs_real += im ? 0 : 1;
      const uint32_t hi = G.lf >> tb, zh = G.zl >> tb;
      ObsRecDev r{};
      r.lfb = (G.lf & ((1u << tb) - 1)) * (c64 ? 8u : 16u);
      r.zt = G.zl & ((1u << tb) - 1);
      r.swap = hi ^ cur;
      cur = hi;
      for (int b = 0; b < 3; ++b) r.s[b] = (zh >> b & 1) << 31;
      p->orecs.push_back(r);
      // the sign is that of x = y ^ lf: thread part tid ^ lf (constant lf & zl),
      // upper part j itself
      const double c = im ? G.im : G.re;
      p->ocoef.push_back({__builtin_popcount(G.lf & r.zt) & 1 ? -c : c, G.zg});
    }
    d.obs_last = int(cur);
  }
}

// The spans of a plan of full tiles (built for the first expectation; lambda
// passes have no use for them).
void ensure_spans(ExpPlan* p, bool c64) {
  if (p->spans_tried) return;
  p->spans_tried = true;
  if (p->L != (c64 ? exp_tile_bits<float>() : exp_tile_bits<double>())) return;
  for (const ExpPassDev& d : p->passes)
    if (d.single_count > kSpanRecs) return;
  p->span_passes = p->passes;
  for (ExpPassDev& d : p->span_passes) build_spans(p, d, p->L - 9, c64);
}

constexpr size_t al256(size_t x) { return (x + 255) / 256 * 256; }

// Host tables that go to the device one after the other, each from a multiple of
// 256 bytes.
struct TablePart {
  const void* src;
  size_t bytes;
};

// The device copy c of the parts (one allocation, one transfer), made if `device` has
// none yet.
int upload_parts(ExpPlan::Copy& c, int device, std::initializer_list<TablePart> parts) {
  if (c.p && c.device == device) return QSV_OK;
  if (c.p) (void)hipFree(c.p);
  c.p = nullptr;
  size_t total = 0;
  for (const TablePart& t : parts) total += al256(std::max<size_t>(t.bytes, 1));
  if (hipMalloc(&c.p, total) != hipSuccess) {
    (void)hipGetLastError();
    c.p = nullptr;
    return fail(QSV_ENOMEM, "observable plan allocation failed");
  }
  c.device = -1;  // (until everything is there)
  std::vector<char> stage(total);
  size_t at = 0;
  for (const TablePart& t : parts) {
    if (t.bytes) std::copy_n(static_cast<const char*>(t.src), t.bytes, stage.data() + at);
    at += al256(std::max<size_t>(t.bytes, 1));
  }
  QSV_HIP_CHECK(hipMemcpy(c.p, stage.data(), total, hipMemcpyHostToDevice));
  c.device = device;
  return QSV_OK;
}

template <typename T>
TablePart part_of(const std::vector<T>& v) {
  return {v.data(), v.size() * sizeof(T)};
}
// Offset of the k-th part.
template <typename... V>
size_t part_offset(const V&... before) {
  size_t o = 0;
  ((o += al256(std::max<size_t>(part_of(before).bytes, 1))), ...);
  return o;
}

// The tables as a call uses them.
struct ExpTables {
  const ExpPassDev* passes = nullptr;
  const ExpGroupDev* groups = nullptr;
  const ExpTermDev *terms = nullptr, *wide = nullptr;
  const ExpSpanDev* spans = nullptr;
  const ExpRecDev* recs = nullptr;
  const ObsRecDev* orecs = nullptr;
  const ObsCoefDev* ocoef = nullptr;
};

int upload_exp_plan(ExpPlan* p, int device, ExpTables* t) {
  if (int rc = upload_parts(p->dev, device, {part_of(p->passes), part_of(p->groups), part_of(p->terms), part_of(p->wide_terms)}))
    return rc;
  const char* d = static_cast<const char*>(p->dev.p);
  t->passes = reinterpret_cast<const ExpPassDev*>(d);
  t->groups = reinterpret_cast<const ExpGroupDev*>(d + part_offset(p->passes));
  t->terms = reinterpret_cast<const ExpTermDev*>(d + part_offset(p->passes, p->groups));
  t->wide = reinterpret_cast<const ExpTermDev*>(d + part_offset(p->passes, p->groups, p->terms));
  return QSV_OK;
}
int upload_spans(ExpPlan* p, int device, ExpTables* t) {
  if (int rc = upload_parts(p->dev_spans, device, {part_of(p->span_passes), part_of(p->spans), part_of(p->recs)})) return rc;
  const char* d = static_cast<const char*>(p->dev_spans.p);
  t->passes = reinterpret_cast<const ExpPassDev*>(d);
  t->spans = reinterpret_cast<const ExpSpanDev*>(d + part_offset(p->span_passes));
  t->recs = reinterpret_cast<const ExpRecDev*>(d + part_offset(p->span_passes, p->spans));
  return QSV_OK;
}
int upload_obs_recs(ExpPlan* p, int device, ExpTables* t) {
  if (int rc = upload_parts(p->dev_obs, device, {part_of(p->obs_passes), part_of(p->orecs), part_of(p->ocoef)})) return rc;
  const char* d = static_cast<const char*>(p->dev_obs.p);
  t->passes = reinterpret_cast<const ExpPassDev*>(d);
  t->orecs = reinterpret_cast<const ObsRecDev*>(d + part_offset(p->obs_passes));
  t->ocoef = reinterpret_cast<const ObsCoefDev*>(d + part_offset(p->obs_passes, p->orecs));
  return QSV_OK;
}

// The plan of o for dtype dt (g_plan_mu held).
ExpPlan* exp_plan_of(qsv_observable* o, qsv_dtype dt) {
  ExpPlan*& pl = o->exp_plan[dt];
  if (!pl) pl = build_exp_plan(o, dt);
  return pl;
}

constexpr size_t kNoAllocBytes = size_t(1) << 20;

// Launch shape of an expectation: all passes in one launch (merged, full tiles in
// spans), each split over nz ranges of its spans and groups where the passes' tiles leave the chip idle
// (every range reads its tiles again). The value depends on the shape in its
// last bits, so the no-allocation variant takes the same one: merged only while
// the partials fit its scratch beside the tables (else one launch per pass,
// adding to one partial per workgroup).
// Measured, 250 strings, one launch per pass against merged: complex64 12 qubits
// 175 and 42 us, 16 qubits 171 and 68, 20 qubits 192 and 106, 24 qubits 937 and
// 879, 30 qubits 33.7 and 32.0 ms; complex128 19 qubits 169 and 80 us.
struct ExpShape {
  uint64_t tiles, grid, parts;
  unsigned np, nz;
  bool merged;
};

size_t exp_table_bytes(const ExpPlan* pl) {
  return al256(pl->passes.size() * sizeof(ExpPassDev)) + al256(pl->groups.size() * sizeof(ExpGroupDev)) +
         al256(pl->terms.size() * sizeof(ExpTermDev)) + al256(pl->wide_terms.size() * sizeof(ExpTermDev));
}

size_t exp_span_bytes(const ExpPlan* pl) {
  return al256(pl->spans.size() * sizeof(ExpSpanDev)) + al256(pl->recs.size() * sizeof(ExpRecDev));
}

ExpShape exp_shape(const ExpPlan* pl, int n) {
  ExpShape h{};
  h.tiles = dim(n - pl->L);
  h.grid = std::min<uint64_t>(h.tiles, exp_grid_max());
  h.np = unsigned(pl->passes.size());
  h.nz = 1;
  h.parts = h.grid;
  if (h.np == 0) return h;
  int most = 1;
  const bool spans = !pl->spans.empty();
  for (const ExpPassDev& P : spans ? pl->span_passes : pl->passes)
    most = std::max(most, spans ? P.span_count + P.grp_count - P.single_count : P.grp_count);
  h.nz = unsigned(std::min<uint64_t>(uint64_t(most), std::max<uint64_t>(1, kExpSplitGrid / (h.grid * h.np))));
  const uint64_t parts = h.grid * h.np * h.nz;
  h.merged = al256((size_t(parts) + 1) * sizeof(double)) + exp_table_bytes(pl) + exp_span_bytes(pl) <= kNoAllocBytes;
  if (h.merged) h.parts = parts;
  else h.nz = 1;
  return h;
}

// Enqueues the passes, the wide groups and the sum (into part[h.parts]).
template <typename R>
int exp_launch(const ExpPlan* pl, const ExpShape& h, int n, const R* psi, const ExpTables& t, double* part, hipStream_t st) {
  const size_t lds = (size_t(1) << pl->L) * sizeof(cx<R>);
  // kernel variant: tile of the default size (compile-time trip counts), at
  // least two amplitudes per thread, or any size
  const int mode = pl->L == exp_tile_bits<R>() ? 2 : ((size_t(1) << pl->L) >= size_t(2 * kExpThreadsE) ? 1 : 0);
  const auto kfn = h.merged && !pl->spans.empty() ? &k_expect_tile<R, 3>
                   : mode == 2                    ? &k_expect_tile<R, 2>
                                                  : (mode == 1 ? &k_expect_tile<R, 1> : &k_expect_tile<R, 0>);
  QSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(lds)));
  const unsigned launches = h.merged ? 1u : h.np;
  for (unsigned pi = 0; pi < launches; ++pi) {
    ProfScope ps("expect", double(sizeof(cx<R>)) * double(dim(n)) * (h.merged ? h.np : 1u), st);
    hipLaunchKernelGGL(kfn, dim3(unsigned(h.grid), h.merged ? h.np : 1u, h.nz), dim3(kExpThreadsE), lds, st, psi,
                       t.passes, int(pi), t.groups, t.terms, t.spans, t.recs, part, pi > 0 ? 1 : 0, h.tiles);
    QSV_HIP_CHECK(hipGetLastError());
  }
  for (size_t wi = 0; wi < pl->wide.size(); ++wi) {
    ProfScope ps("expect_wide", double(sizeof(cx<R>)) * double(dim(n)), st);
    const ExpWide& w = pl->wide[wi];
    hipLaunchKernelGGL((k_expect_wide<R>), dim3(unsigned(h.grid)), dim3(kExpThreadsE), 0, st, psi, w.flip, w.hbit,
                       t.wide + w.term_begin, w.term_count, dim(n - 1), part, pl->passes.empty() && wi == 0 ? 0 : 1);
    QSV_HIP_CHECK(hipGetLastError());
  }
  hipLaunchKernelGGL(k_exp_sum, dim3(1), dim3(kExpThreads), 0, st, part, h.parts, part + h.parts);
  QSV_HIP_CHECK(hipGetLastError());
  return QSV_OK;
}

template <typename R>
int expect_tiled_t(qsv_state* s, qsv_observable* o, double* out) {
  ExpPlan* pl = nullptr;
  ExpTables t;
  ExpShape h{};
  int rc = QSV_OK;
  {
    std::lock_guard<std::mutex> lk(g_plan_mu);
    pl = exp_plan_of(o, s->dtype);
    if (pl->passes.empty() && pl->wide.empty()) {
      *out = 0.0;
      return QSV_OK;
    }
    ensure_spans(pl, sizeof(R) == 4);
    h = exp_shape(pl, s->n);
    if ((rc = upload_exp_plan(pl, s->device, &t))) return rc;
    if (h.merged && !pl->spans.empty() && (rc = upload_spans(pl, s->device, &t))) return rc;
  }
  if ((rc = ensure_reduce_scratch(s, size_t(h.parts) + 1))) return rc;
  rc = exp_launch<R>(pl, h, s->n, static_cast<const R*>(s->ptr), t, s->red, s->stream);
  if (rc) return rc;
  QSV_HIP_CHECK(hipMemcpyAsync(s->red_host, s->red + h.parts, sizeof(double), hipMemcpyDeviceToHost, s->stream));
  QSV_HIP_CHECK(hipStreamSynchronize(s->stream));
  *out = s->red_host[0];
  return QSV_OK;
}

template <typename R>
int apply_obs_tiled_t(const qsv_state* in, qsv_observable* o, qsv_state* out) {
  const uint64_t N = dim(in->n);
  ExpPlan* pl = nullptr;
  ExpTables t;
  {
    std::lock_guard<std::mutex> lk(g_plan_mu);
    pl = exp_plan_of(o, in->dtype);
    if (!pl->passes.empty() || !pl->wide.empty()) {
      ensure_obs_recs(pl, sizeof(R) == 4);
      if (int rc = upload_exp_plan(pl, in->device, &t)) return rc;
      if (!pl->orecs.empty())
        if (int rc = upload_obs_recs(pl, in->device, &t)) return rc;
    }
  }
  if (pl->passes.empty() && pl->wide.empty()) {  // no terms: lambda = 0
    const uint64_t blocks = std::min<uint64_t>((N + kExpThreads - 1) / kExpThreads, 65536);
    hipLaunchKernelGGL((k_zero_amps<R>), dim3(unsigned(blocks)), dim3(kExpThreads), 0, in->stream,
                       static_cast<R*>(out->ptr), N);
    QSV_HIP_CHECK(hipGetLastError());
    return QSV_OK;
  }
  const uint64_t tiles = dim(in->n - pl->L);
  const size_t lds = (size_t(1) << pl->L) * sizeof(cx<R>);
  // compile-time output count when every thread has obs_out<R>() outputs
  constexpr int NTo = obs_threads<R>();
  const bool fixed = pl->L == obs_tile_bits<R>() && (size_t(1) << pl->L) == size_t(obs_out<R>()) * NTo;
  const auto kfn = fixed && !pl->orecs.empty() ? &k_apply_obs_tile<R, true, NTo, true>
                   : fixed                     ? &k_apply_obs_tile<R, true, NTo, false>
                                               : &k_apply_obs_tile<R, false, NTo, false>;
  QSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    int(lds)));
  for (size_t pi = 0; pi < pl->passes.size(); ++pi) {
    ProfScope ps("apply_obs", double(sizeof(cx<R>)) * double(N) * (pi > 0 ? 3.0 : 2.0), in->stream);
    hipLaunchKernelGGL(kfn, dim3(unsigned(std::min<uint64_t>(tiles, obs_grid_max()))), dim3(NTo), lds, in->stream,
                       static_cast<const R*>(in->ptr), static_cast<R*>(out->ptr), t.passes, int(pi), t.groups, t.terms,
                       t.orecs, t.ocoef, pi > 0 ? 1 : 0, tiles);
    QSV_HIP_CHECK(hipGetLastError());
  }
  for (size_t wi = 0; wi < pl->wide.size(); ++wi) {
    const bool acc = !pl->passes.empty() || wi > 0;
    ProfScope ps("apply_obs_wide", double(sizeof(cx<R>)) * double(N) * (acc ? 3.0 : 2.0), in->stream);
    const ExpWide& w = pl->wide[wi];
    const unsigned blocks = unsigned(std::min<uint64_t>((N + kExpThreads - 1) / kExpThreads, 8192));
    hipLaunchKernelGGL((k_apply_obs_wide<R>), dim3(blocks), dim3(kExpThreads), 0, in->stream,
                       static_cast<const R*>(in->ptr), static_cast<R*>(out->ptr), w.flip, t.wide + w.term_begin,
                       w.term_count, N, acc ? 1 : 0);
    QSV_HIP_CHECK(hipGetLastError());
  }
  return QSV_OK;
}

// ------------------------------------------------------------------ no-allocation variant
//
// qsv_expectation_noalloc runs the same passes with every device buffer they
// need -- the observable's pass / group / term tables and the per-workgroup
// FP64 partials -- in one file-scope device array of kNoAllocBytes, so the
// call allocates no device or pinned memory (for callers that cannot: code
// under stream capture, serving loops). Each device holds its own copy of the
// array; its address on a device is taken once (hipGetSymbolAddress, with
// that device current) and only that address is used from the host. Calls on
// one device share the array: calls that overlap on one device race.
static __device__ __align__(256) char scratch[kNoAllocBytes];

constexpr int kNoAllocMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kNoAllocMaxDevices] = {};

// Device address of `scratch` on `device` (taken on first use).
int noalloc_scratch(int device, char** out) {
  if (device < 0 || device >= kNoAllocMaxDevices) return fail(QSV_EINVAL, "device index %d out of range", device);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int cur = -1;
    QSV_HIP_CHECK(hipGetDevice(&cur));
    if (cur != device) QSV_HIP_CHECK(hipSetDevice(device));
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr)
      return fail(QSV_EHIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    g_scratch_ptr[device] = static_cast<char*>(ptr);
  }
  *out = g_scratch_ptr[device];
  return QSV_OK;
}

template <typename R>
int expect_noalloc_t(qsv_state* s, qsv_observable* o, double* out) {
  ExpPlan* pl = nullptr;
  ExpShape h{};
  {
    std::lock_guard<std::mutex> lk(g_plan_mu);
    pl = exp_plan_of(o, s->dtype);  // host tables only
    if (pl->passes.empty() && pl->wide.empty()) {
      *out = 0.0;
      return QSV_OK;
    }
    ensure_spans(pl, sizeof(R) == 4);
    h = exp_shape(pl, s->n);
  }
  const bool in_spans = h.merged && !pl->spans.empty();
  // scratch layout: partials[parts + 1] | passes | groups | terms (256-byte aligned)
  const size_t o_pass = al256((size_t(h.parts) + 1) * sizeof(double));
  const size_t o_grp = o_pass + al256(pl->passes.size() * sizeof(ExpPassDev));
  const size_t o_term = o_grp + al256(pl->groups.size() * sizeof(ExpGroupDev));
  const size_t o_wide = o_term + al256(pl->terms.size() * sizeof(ExpTermDev));
  const size_t o_span = o_pass + exp_table_bytes(pl);
  const size_t o_rec = o_span + al256(pl->spans.size() * sizeof(ExpSpanDev));
  const size_t need = h.merged ? o_span + exp_span_bytes(pl) : o_span;
  if (need > kNoAllocBytes)
    return fail(QSV_ERANGE, "observable needs %zu bytes of device scratch; the no-allocation limit is %zu",
                need, kNoAllocBytes);
  char* d = nullptr;
  int rc = noalloc_scratch(s->device, &d);
  if (rc) return rc;
  hipStream_t st = s->stream;
  if (!pl->passes.empty())
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_pass, (in_spans ? pl->span_passes : pl->passes).data(),
                                 pl->passes.size() * sizeof(ExpPassDev), hipMemcpyHostToDevice, st));
  if (!pl->groups.empty())
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_grp, pl->groups.data(), pl->groups.size() * sizeof(ExpGroupDev),
                                 hipMemcpyHostToDevice, st));
  if (!pl->terms.empty())
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_term, pl->terms.data(), pl->terms.size() * sizeof(ExpTermDev),
                                 hipMemcpyHostToDevice, st));
  if (!pl->wide_terms.empty())
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_wide, pl->wide_terms.data(), pl->wide_terms.size() * sizeof(ExpTermDev),
                                 hipMemcpyHostToDevice, st));
  if (in_spans) {
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_span, pl->spans.data(), pl->spans.size() * sizeof(ExpSpanDev),
                                 hipMemcpyHostToDevice, st));
    QSV_HIP_CHECK(hipMemcpyAsync(d + o_rec, pl->recs.data(), pl->recs.size() * sizeof(ExpRecDev),
                                 hipMemcpyHostToDevice, st));
  }
  double* part = reinterpret_cast<double*>(d);
  // (the first launch writes every partial that is summed: nothing left from an
  // earlier call is read)
  ExpTables t;
  t.passes = reinterpret_cast<const ExpPassDev*>(d + o_pass);
  t.groups = reinterpret_cast<const ExpGroupDev*>(d + o_grp);
  t.terms = reinterpret_cast<const ExpTermDev*>(d + o_term);
  t.wide = reinterpret_cast<const ExpTermDev*>(d + o_wide);
  t.spans = reinterpret_cast<const ExpSpanDev*>(d + o_span);
  t.recs = reinterpret_cast<const ExpRecDev*>(d + o_rec);
  rc = exp_launch<R>(pl, h, s->n, static_cast<const R*>(s->ptr), t, part, st);
  if (rc) return rc;
  double v = 0.0;
  QSV_HIP_CHECK(hipMemcpyAsync(&v, part + h.parts, sizeof(double), hipMemcpyDeviceToHost, st));
  QSV_HIP_CHECK(hipStreamSynchronize(st));
  *out = v;
  return QSV_OK;
}

}  // namespace

int expectation_noalloc(qsv_state* s, const qsv_observable* o, double* out) {
  qsv_observable* mo = const_cast<qsv_observable*>(o);  // host plan cache only
  return s->dtype == QSV_C64 ? expect_noalloc_t<float>(s, mo, out) : expect_noalloc_t<double>(s, mo, out);
}

int expectation_tiled(qsv_state* s, const qsv_observable* o, double* out) {
  qsv_observable* mo = const_cast<qsv_observable*>(o);  // plan cache only
  return s->dtype == QSV_C64 ? expect_tiled_t<float>(s, mo, out) : expect_tiled_t<double>(s, mo, out);
}

// lambda = O psi (out must not alias in; both on in's stream).
int apply_observable_tiled(const qsv_state* in, const qsv_observable* o, qsv_state* out) {
  qsv_observable* mo = const_cast<qsv_observable*>(o);  // plan cache only
  return in->dtype == QSV_C64 ? apply_obs_tiled_t<float>(in, mo, out) : apply_obs_tiled_t<double>(in, mo, out);
}

int expectation_passes(const qsv_observable* o, qsv_dtype dt) {
  qsv_observable* mo = const_cast<qsv_observable*>(o);
  std::lock_guard<std::mutex> lk(g_plan_mu);
  const ExpPlan* pl = exp_plan_of(mo, dt);
  return int(pl->passes.size() + pl->wide.size());
}

}  // namespace qsv

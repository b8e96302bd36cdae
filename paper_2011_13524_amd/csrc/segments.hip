// Host side of the register-resident passes: assignment of elementary ops to
// passes, register segments within a pass, and the values they read.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <functional>

#include "plan.h"
#include "tile_reg.h"

namespace qsv {

void rotation_shears(double t, cd* out) {
  // (the sine and cosine of t/2 itself, whatever its size: a reduction by a
  // rounded 2 pi would be off by 4e-17 |t/2|)
  double s = std::sin(0.5 * t), c = std::cos(0.5 * t), sg = 1.0;
  if (c < 0.0) {
    s = -s;
    c = -c;
    sg = -1.0;
  }
  out[0] = {s / (1.0 + c), -s};
  out[1] = {sg, 0.0};
}

bool is_unitary2(const cd* u, double tol) {
  const double n0 = u[0].re * u[0].re + u[0].im * u[0].im + u[2].re * u[2].re + u[2].im * u[2].im;
  const double n1 = u[1].re * u[1].re + u[1].im * u[1].im + u[3].re * u[3].re + u[3].im * u[3].im;
  // (where squares of the entries underflow the test says nothing)
  if (!(n0 >= 1e-250) || !std::isfinite(n0) || !(std::fabs(n0 - n1) <= tol * n0)) return false;
  const double xr = u[0].re * u[1].re + u[0].im * u[1].im + u[2].re * u[3].re + u[2].im * u[3].im;
  const double xi = u[0].re * u[1].im - u[0].im * u[1].re + u[2].re * u[3].im - u[2].im * u[3].re;
  return std::fabs(xr) + std::fabs(xi) <= tol * n0;
}

// Largest difference between an entry of u and what unitary_to_rotation's values
// stand for, relative to a column of u.
static double rotation_error(const cd* u) {
  typedef long double F;
  cd o[6];
  unitary_to_rotation(u, o);
  const F a = o[2].re, b = o[2].im, m[4] = {1 + a * b, a * (2 + a * b), b, 1 + a * b};
  F worst = 0;
  for (int r = 0; r < 2; ++r)
    for (int c = 0; c < 2; ++c) {
      const cd l = o[4 + r], f = o[c];
      const F pr = F(l.re) * f.re - F(l.im) * f.im, pi = F(l.re) * f.im + F(l.im) * f.re;
      const cd z = u[2 * r + c];
      worst = std::max(worst, std::hypot(pr * m[2 * r + c] - z.re, pi * m[2 * r + c] - z.im));
    }
  return double(worst / std::hypot(std::hypot(F(u[0].re), F(u[0].im)), std::hypot(F(u[2].re), F(u[2].im))));
}

bool runs_as_rotation(const cd* u, bool c64) {
  return c64 ? is_unitary2(u, 1e-9) : is_unitary2(u, 2e-15) && rotation_error(u) <= 1.15e-16;
}

void unitary_to_rotation(const cd* u, cd* out) {
  auto mod = [](cd z) { return std::hypot(z.re, z.im); };
  auto unit = [&](cd z) -> cd {
    const double m = mod(z);
    return m > 0.0 ? cd{z.re / m, z.im / m} : cd{1.0, 0.0};
  };
  auto conj = [](cd z) { return cd{z.re, -z.im}; };
  // the scale (1 for a unitary) and the rotation angle h in [0, pi/2]
  const double ca = std::hypot(mod(u[0]), mod(u[3])), sa = std::hypot(mod(u[1]), mod(u[2]));
  const double sc = std::hypot(ca, sa) / std::sqrt(2.0);
  const double c = ca / (sc * std::sqrt(2.0)), s = sa / (sc * std::sqrt(2.0));
  // u00 = mu c, u01 = mu s la, u10 = -nu s, u11 = nu c la (|mu| = |nu| = |la| = 1):
  // the phases from the larger entries, so that they carry no rounding noise
  cd mu, nu, la;
  if (c >= s) {
    mu = unit(u[0]);
    nu = unit(cd{-u[2].re, -u[2].im});
    la = cmul(unit(u[3]), conj(nu));
  } else {
    mu = unit(u[0]);
    nu = unit(cd{-u[2].re, -u[2].im});
    la = cmul(unit(u[1]), conj(mu));
  }
  out[0] = {1.0, 0.0};
  out[1] = la;
  out[2] = {s / (1.0 + c), -s};
  out[3] = {1.0, 0.0};
  out[4] = {sc * mu.re, sc * mu.im};
  out[5] = {sc * nu.re, sc * nu.im};
}

namespace {

// A set of places 0 .. n - 1, as bits.
struct PlaceSet {
  std::vector<uint64_t> w;
  int count = 0;
  void reset(size_t n) {
    w.assign((n + 63) / 64, 0);
    count = 0;
  }
  bool empty() const { return count == 0; }
  void insert(int at) {
    uint64_t& x = w[size_t(at) / 64];
    count += int(~x >> (at & 63) & 1);
    x |= uint64_t(1) << (at & 63);
  }
  void erase(int at) {
    uint64_t& x = w[size_t(at) / 64];
    count -= int(x >> (at & 63) & 1);
    x &= ~(uint64_t(1) << (at & 63));
  }
  int first() const {  // (not empty)
    size_t k = 0;
    while (!w[k]) ++k;
    return int(64 * k) + __builtin_ctzll(w[k]);
  }
  std::vector<int> list() const {
    std::vector<int> v;
    for (size_t k = 0; k < w.size(); ++k)
      for (uint64_t m = w[k]; m; m &= m - 1) v.push_back(int(64 * k) + __builtin_ctzll(m));
    return v;
  }
};

// One pass of the scheduler below: the remaining ops that a pass can take, in
// order. With `grow`, the local set takes the qubits of the ops in order while
// it has room (at most L), else it is fixed.
struct PassTrial {
  uint64_t local = 0;
  int gain = 0;  // ops taken other than phases
};

// lists: also fill take / left (execution order, remaining ops). free_diag: there
// are diagonal ops other than phases, which any pass takes.
PassTrial try_pass(const std::vector<PassOp>& ops, const std::vector<int>& rem, uint64_t local, bool grow, int L,
                   uint64_t all, int max_rows, bool free_diag, std::vector<int>* take, std::vector<int>* left) {
  PassTrial t;
  uint64_t defer_nd = 0, defer_dg = 0;  // qubits of the deferred ops
  int rows = 0;
  std::vector<int> wait;  // phases that nothing taken needs yet
  const bool lists = take != nullptr, count = max_rows < (1 << 29);
  size_t k = 0;
  for (; k < rem.size(); ++k) {
    const int oi = rem[k];
    const PassOp& o = ops[size_t(oi)];
    bool ok = !((o.nd & (defer_nd | defer_dg)) | (o.dg & defer_nd));
    if (ok && o.lazy) {
      if (lists || count) wait.push_back(oi);
      continue;
    }
    if (ok) ok = grow ? __builtin_popcountll(local | o.local) <= L : !(o.local & ~local);
    if (ok && (lists || count)) {
      int r = rows + o.rows;
      for (int w : wait)
        if (ops[size_t(w)].dg & o.nd) r += ops[size_t(w)].rows;
      ok = r <= max_rows;
      if (ok) {
        rows = r;
        size_t j = 0;
        for (int w : wait) {
          if (!(ops[size_t(w)].dg & o.nd)) wait[j++] = w;
          else if (lists) take->push_back(w);
        }
        wait.resize(j);
        if (lists) take->push_back(oi);
      }
    }
    if (ok) {
      local |= o.local;
      t.gain += o.weight;
      continue;
    }
    if (lists) left->push_back(oi);
    defer_nd |= o.nd;
    defer_dg |= o.dg;
    // nothing later can run: every qubit is held back, or every local one is and
    // ops that are not phases act on a local qubit (at the end of a list, phases
    // run for their own sake only in a pass that takes nothing else)
    const uint64_t held = free_diag ? defer_nd : (defer_nd | defer_dg);
    if ((held & (free_diag || grow ? all : local)) == (free_diag || grow ? all : local) && (!lists || !take->empty())) {
      ++k;
      break;
    }
  }
  t.local = local;
  if (lists) {
    left->insert(left->end(), rem.begin() + long(k), rem.end());
    // phases that only later passes need wait for those; at the end of the
    // circuit, or when nothing else can run, they run here
    if (left->empty() || take->empty()) {
      size_t j = 0;
      for (int w : wait) {
        if (rows + ops[size_t(w)].rows <= max_rows) {
          rows += ops[size_t(w)].rows;
          take->push_back(w);
        } else {
          wait[j++] = w;
        }
      }
      wait.resize(j);
    }
    const long mid = long(left->size());
    left->insert(left->end(), wait.begin(), wait.end());
    std::inplace_merge(left->begin(), left->begin() + mid, left->end());
  }
  return t;
}

// The gain of try_pass for a fixed local set, over the ops that bear on it: a phase
// on one qubit without a gradient row holds back nothing that what it waits for does
// not. Phases with rows are on one qubit (plain), so those that wait are counted
// per qubit.
struct GainOps {
  std::vector<PassOp> ops;
  bool plain = true;
  void fill(const std::vector<PassOp>& from, const std::vector<int>& rem) {
    ops.clear();
    for (int oi : rem) {
      const PassOp& o = from[size_t(oi)];
      const bool one = (o.dg & (o.dg - 1)) == 0;
      if (!o.lazy || !one || o.rows) ops.push_back(o);
      plain = plain && (!o.lazy || one || !o.rows);
    }
  }
  template <bool COUNT>
  int gain(uint64_t local, uint64_t all, bool free_diag, int max_rows) const {
    uint64_t defer_nd = 0, defer_dg = 0;
    const uint64_t stop = free_diag ? all : local;
    int g = 0, rows = 0;
    int wait[64];
    if (COUNT) std::fill(wait, wait + 64, 0);
    for (const PassOp& o : ops) {
      bool ok = !((o.nd & (defer_nd | defer_dg)) | (o.dg & defer_nd) | (o.local & ~local));
      if (ok && o.lazy) {
        if (COUNT && o.rows) wait[__builtin_ctzll(o.dg)] += o.rows;
        continue;
      }
      if (COUNT && ok) {
        int r = rows + o.rows;
        for (uint64_t m = o.nd; m; m &= m - 1) r += wait[__builtin_ctzll(m)];
        ok = r <= max_rows;
        if (ok) {
          rows = r;
          for (uint64_t m = o.nd; m; m &= m - 1) wait[__builtin_ctzll(m)] = 0;
        }
      }
      if (ok) {
        g += o.weight;
        continue;
      }
      defer_nd |= o.nd;
      defer_dg |= o.dg;
      if (((free_diag ? defer_nd : (defer_nd | defer_dg)) & stop) == stop) break;
    }
    return g;
  }
};

}  // namespace

int schedule_passes(const std::vector<PassOp>& ops, int n, int L, int b, int max_rows,
                    std::vector<std::vector<int>>& pass_ops, std::vector<uint64_t>& pass_local) {
  pass_ops.clear();
  pass_local.clear();
  std::vector<int> rem(ops.size());
  for (size_t i = 0; i < ops.size(); ++i) rem[i] = int(i);
  const uint64_t all = (n >= 64) ? ~0ull : ((uint64_t(1) << n) - 1);
  const uint64_t low = (b >= 64) ? ~0ull : ((uint64_t(1) << b) - 1);
  const int budget = 100;  // trial exchanges per pass (each scans the ops in reach: under 1 us)
  const bool count = max_rows < (1 << 29);
  bool free_diag = false;
  for (const PassOp& o : ops) free_diag = free_diag || (!o.lazy && o.nd == 0);
  GainOps reach;
  while (!rem.empty()) {
    PassTrial best;
    best.local = all;
    if (n > L) {
      best = try_pass(ops, rem, low, true, L, all, max_rows, free_diag, nullptr, nullptr);
      for (int q = 0; q < n && __builtin_popcountll(best.local) < L; ++q) best.local |= uint64_t(1) << q;
      reach.fill(ops, rem);
      auto consider = [&](uint64_t local) {
        const int gain =
            !count          ? reach.gain<false>(local, all, free_diag, max_rows)
            : reach.plain   ? reach.gain<true>(local, all, free_diag, max_rows)
                            : try_pass(ops, rem, local, false, L, all, max_rows, free_diag, nullptr, nullptr).gain;
        if (gain <= best.gain) return false;
        best.gain = gain;
        best.local = local;
        return true;
      };
      // windows of neighbouring qubits (ladders, rings, bricks)
      for (int q0 = b; q0 < n; ++q0) {
        uint64_t w = low;
        for (int i = 0; __builtin_popcountll(w) < L; ++i) w |= uint64_t(1) << ((q0 + i) % n);
        consider(w);
      }
      // exchanges of one local qubit
      int evals = 0;
      for (bool up = true; up && evals < budget;) {
        up = false;
        for (int out = b; out < n && evals < budget; ++out) {
          if (!(best.local >> out & 1)) continue;
          for (int in = b; in < n && evals < budget; ++in) {
            if (best.local >> in & 1) continue;
            ++evals;
            if (consider((best.local & ~(uint64_t(1) << out)) | (uint64_t(1) << in))) {
              up = true;
              break;
            }
          }
        }
      }
    }
    std::vector<int> take, left;
    try_pass(ops, rem, best.local, false, L, all, max_rows, free_diag, &take, &left);
    if (take.empty()) return fail(QSV_EINVAL, "planner made no progress (tile too small)");
    pass_ops.push_back(std::move(take));
    pass_local.push_back(best.local);
    rem.swap(left);
  }
  return QSV_OK;
}

// Split a pass's ops into register-resident segments.
//
// Scheduling: ops that commute may run in any order. Two ops commute when
// every local qubit they share is acted on diagonally by both (a control, or a
// diagonal target); otherwise the later op depends on the earlier one. A
// segment fixes reg_bits register bits and takes, by list scheduling over
// this dependency order, every ready op whose register needs (the targets of
// one- and two-qubit dense ops; diagonal and LDS ops need none) still fit;
// when no ready op fits, the next segment starts.
//
// Folding: an X gate, or an X with one local control, permutes the tile's
// local indices by an affine map over GF(2) (x_t ^= x_c, or ^= 1). Such an op
// moves no data: it is folded into the next re-map through LDS, whose write
// addresses go through the composed map. Ops that depend on a folded op wait
// for the next segment; ops that commute with it are unaffected.
//
// Layouts: the first segment is the layout the tile is read in and the last
// the one it is written in, so both put the low local bits that form
// contiguous 128-byte runs on lanes 0..2 (and, for complex64, local bit 0 in
// registers: amplitude pairs are 16-byte vectors). A segment's wave bits
// (thread-index bits above the 64 lanes) are chosen so that consecutive
// segments share them where possible: a re-map between two such layouts
// moves data only within each wavefront and needs no workgroup barrier.
void pass_runs(TilePassDev& d) {
  d.nrun = 0;
  for (int j = 0; j < d.ng; ++j) {
    if (j > 0 && d.gpos[j] == d.gpos[j - 1] + 1) {
      ++d.rlen[d.nrun - 1];
      continue;
    }
    d.rsrc[d.nrun] = j;
    d.rdst[d.nrun] = d.gpos[j];
    d.rlen[d.nrun] = 1;
    ++d.nrun;
  }
}

int build_reg_segments(const SegCfg& cfg, std::vector<TileOpDev>& ho, TilePassDev& d, SegBuild& out) {
  const int RB = cfg.reg_bits, TB = cfg.thread_bits, L = d.L;
  const int NW = TB - 6, NR = 1 << RB;
  const bool c64 = cfg.c64;
  const uint32_t full = (1u << L) - 1;
  const uint32_t io_reg = c64 ? 1u : 0u;
  const uint32_t io_lane = c64 ? 0xEu : 0x7u;
  const int nops = d.op_count;
  std::vector<RegSegDev>& out_segs = out.segs;
  std::vector<RegOpDev>& out_rops = out.rops;
  auto pool_take = [&](int nv) {
    const int at = out.pool_elems;
    out.pool_elems += nv;
    return at;
  };

  d.rop_begin = int(out.rops.size());
  d.ent_begin = int(out.ents.size());
  d.pool_begin = out.pool_elems;

  // dependency order
  std::vector<uint32_t> need(nops), nd(nops), dg(nops);
  for (int i = 0; i < nops; ++i) {
    const TileOpDev& o = ho[d.op_begin + i];
    uint32_t tg = 0;
    for (int j = 0; j < o.k && j < 5; ++j)
      if (o.kind != 3 && o.lt[j] >= 0) tg |= 1u << o.lt[j];
    if (o.kind == 4) {
      nd[i] = need[i] = tg;
      dg[i] = 0;
    } else if (o.kind == 5) {
      nd[i] = need[i] = 0;
      dg[i] = tg;
    } else if (o.kind == 3) {  // Pauli-string gradient: X/Y qubits non-diagonal, Z diagonal
      nd[i] = o.off[0];
      dg[i] = o.off[1] & ~o.off[0];
      need[i] = 0;
    } else if (o.kind == 0) {
      nd[i] = tg;
      dg[i] = o.lcm;
      need[i] = o.k <= 2 ? tg : 0u;
    } else {
      nd[i] = 0;
      dg[i] = tg | o.lcm;
      need[i] = 0;
    }
  }
  // Direct predecessors: per local bit, a non-diagonal op follows the diagonal ops
  // since the last non-diagonal one, and that one; a diagonal op follows the last
  // non-diagonal one. Every other op that op i has to follow comes before one of
  // these, and each state below (executed, folded, done) holds for an op only if
  // it holds for all that the op follows: the direct ones tell.
  // preds of op i: pred[pred_at[i] .. pred_at[i + 1]), and the other way round.
  std::vector<int> pred, pred_at(nops + 1, 0), succ, succ_at(nops + 2, 0);
  {
    std::vector<int> last_nd(L, -1);
    std::vector<std::vector<int>> since(L);
    for (int i = 0; i < nops; ++i) {
      const size_t p0 = pred.size();
      for (uint32_t m = nd[i] | dg[i]; m; m &= m - 1) {
        const int q = __builtin_ctz(m);
        if (nd[i] >> q & 1) {
          if (since[q].empty() && last_nd[q] >= 0) pred.push_back(last_nd[q]);
          pred.insert(pred.end(), since[q].begin(), since[q].end());
          since[q].clear();
          last_nd[q] = i;
        } else {
          if (last_nd[q] >= 0) pred.push_back(last_nd[q]);
          since[q].push_back(i);
        }
      }
      std::sort(pred.begin() + long(p0), pred.end());
      pred.erase(std::unique(pred.begin() + long(p0), pred.end()), pred.end());
      pred_at[i + 1] = int(pred.size());
    }
    succ.resize(pred.size());
    for (int q : pred) ++succ_at[q + 2];
    for (int i = 0; i < nops; ++i) succ_at[i + 2] += succ_at[i + 1];
    for (int i = 0; i < nops; ++i)
      for (int k = pred_at[i]; k < pred_at[i + 1]; ++k) succ[size_t(succ_at[pred[size_t(k)] + 1]++)] = i;
  }
  struct Range {
    const int *b, *e;
    const int* begin() const { return b; }
    const int* end() const { return e; }
  };
  auto succs = [&](int i) { return Range{succ.data() + succ_at[i], succ.data() + succ_at[i + 1]}; };
  auto preds = [&](int i) { return Range{pred.data() + pred_at[i], pred.data() + pred_at[i + 1]}; };
  auto npreds = [&](int i) { return pred_at[i + 1] - pred_at[i]; };
  std::vector<char> foldable(nops, 0);
  for (int i = 0; i < nops; ++i) {
    const TileOpDev& o = ho[d.op_begin + i];
    foldable[i] = o.kind == 0 && o.k == 1 && o.xswap && o.gcm == 0 && __builtin_popcount(o.lcm) <= 1;
  }

  // list scheduling into segments: an op executes in a segment when all that it
  // follows was executed, or folded into an earlier re-map; it folds into the
  // re-map after the segment when all that was executed or folded
  struct Seg {
    uint32_t regs = 0;  // register positions the ops need (+ IO constraints)
    bool io = false;
    std::vector<int> ops;
    std::vector<int> fold;  // ops folded into the re-map after this segment
    uint32_t w = 0;         // wave positions
    bool xwave = false;
  };
  std::vector<Seg> segs;
  // predecessors still to come (wait_fold) and those or only just folded (wait_exec)
  std::vector<int> wait_exec(nops), wait_fold(nops);
  std::vector<int> ready, later;  // ops that can be placed, in order
  for (int i = 0; i < nops; ++i) {
    wait_exec[i] = wait_fold[i] = npreds(i);
    if (npreds(i) == 0) ready.push_back(i);
  }
  int left = nops;
  do {
    Seg s;
    const bool first = segs.empty();
    s.io = first;
    s.regs = first ? io_reg : 0u;
    const uint32_t forbid = first ? io_lane : 0u;
    // (one sweep in order: an op that becomes ready comes after the one that made
    // it so, and the registers in use only grow)
    std::make_heap(ready.begin(), ready.end(), std::greater<int>());
    auto next_ready = [&](int j) {
      ready.push_back(j);
      std::push_heap(ready.begin(), ready.end(), std::greater<int>());
    };
    later.clear();
    while (!ready.empty()) {
      std::pop_heap(ready.begin(), ready.end(), std::greater<int>());
      const int i = ready.back();
      ready.pop_back();
      if (foldable[i]) {
        s.fold.push_back(i);
        for (int j : succs(i))
          if (--wait_fold[j] == 0 && foldable[j]) next_ready(j);
      } else {
        const uint32_t u = s.regs | need[i];
        if ((need[i] & forbid) || __builtin_popcount(u) > RB) {
          later.push_back(i);
          continue;
        }
        s.regs = u;
        s.ops.push_back(i);
        for (int j : succs(i)) {
          --wait_exec[j];
          --wait_fold[j];
          if ((foldable[j] ? wait_fold[j] : wait_exec[j]) == 0) next_ready(j);
        }
      }
      --left;
    }
    if (s.ops.empty() && s.fold.empty() && !first) return fail(QSV_EINVAL, "internal: segment scheduling stalled");
    for (int i : s.fold)
      for (int j : succs(i))
        if (--wait_exec[j] == 0 && !foldable[j]) later.push_back(j);
    ready.swap(later);
    segs.push_back(std::move(s));
  } while (left > 0);
  {
    Seg& last = segs.back();
    // ops folded after the last segment need a re-map; when it would be the
    // only reason for one, run them as register exchanges instead
    if (!last.fold.empty() && (last.io || ((last.regs & io_lane) == 0 &&
                                           __builtin_popcount(last.regs | io_reg) <= RB))) {
      uint32_t u = last.regs | io_reg;
      for (int i : last.fold) u |= need[i] | (1u << ho[d.op_begin + i].lt[0]);
      if ((u & io_lane) == 0 && __builtin_popcount(u) <= RB) {
        last.regs = u;
        for (int i : last.fold) last.ops.push_back(i);
        last.fold.clear();
      }
    }
    if (!last.io || !last.fold.empty()) {
      if (last.fold.empty() && (last.regs & io_lane) == 0 && __builtin_popcount(last.regs | io_reg) <= RB) {
        last.regs |= io_reg;
        last.io = true;
      } else {
        Seg s;
        s.regs = io_reg;
        s.io = true;
        segs.push_back(std::move(s));
      }
    }
  }
  // affine map of each re-map (into segment k: the folds of segment k-1):
  // image of local basis vector p, and the constant
  const int K = int(segs.size());
  std::vector<std::vector<uint32_t>> mcol(K, std::vector<uint32_t>(L));
  std::vector<uint32_t> mcst(K, 0), ftarget(K, 0);
  for (int k = 0; k < K; ++k) {
    for (int q = 0; q < L; ++q) mcol[k][q] = 1u << q;
    if (k == 0) continue;
    for (int i : segs[k - 1].fold) {
      const TileOpDev& o = ho[d.op_begin + i];
      const uint32_t t = 1u << o.lt[0];
      ftarget[k] |= t;
      // x_t ^= x_c (control value 1) or x_t ^= x_c ^ 1 (value 0); no control: x_t ^= 1
      auto apply = [&](uint32_t y) -> uint32_t {
        if (o.lcm == 0) return y;
        return (y & o.lcm) ? (y ^ t) : y;
      };
      for (int q = 0; q < L; ++q) mcol[k][q] = apply(mcol[k][q]);
      mcst[k] = apply(mcst[k]);
      if (o.lcm == 0 || (o.lcv & o.lcm) == 0) mcst[k] ^= t;
    }
  }

  // wave bits: maximal runs of segments sharing NW available positions;
  // prefer positions off the low lanes (longer contiguous HBM runs)
  // (a run continues into segment k only if no op folded into the re-map
  // before k targets a wave bit: that re-map would move data across waves)
  std::vector<uint32_t> avail(K);
  for (int k = 0; k < K; ++k) avail[k] = full & ~segs[k].regs & ~(segs[k].io ? (io_lane | io_reg) : 0u);
  for (int k = 0; k < K;) {
    uint32_t I = avail[k];
    int m = k + 1;
    while (m < K && __builtin_popcount(I & avail[m] & ~ftarget[m]) >= NW) {
      I &= avail[m] & ~ftarget[m];
      ++m;
    }
    uint32_t w = 0;
    for (int pass = 0; pass < 2 && __builtin_popcount(w) < NW; ++pass)
      for (int pos = L - 1; pos >= 0 && __builtin_popcount(w) < NW; --pos) {
        const bool low = pos >= 1 && pos <= 6;
        if ((I >> pos & 1) && (pass == 1 || !low)) w |= 1u << pos;
      }
    if (__builtin_popcount(w) != NW) return fail(QSV_EINVAL, "internal: no wave bits");
    for (int t = k; t < m; ++t) {
      segs[t].w = w;
      segs[t].xwave = (t == k && k > 0);
    }
    k = m;
  }
  // A cross-wave re-map writes with the folded map, which may move elements
  // into other wavefronts' regions of the old layout; after a wave-local re-map
  // (no trailing barrier) those wavefronts may still be reading there, so such
  // a re-map also waits for the workgroup before writing.
  // A cross-wave re-map does not close with a barrier: waves go on with the
  // segment's register ops, and the barrier moves to the next LDS write (the
  // next re-map's, or an op through LDS, which always waits first). Until then
  // other waves may still read any region, so the next re-map waits first.
  std::vector<char> pre(K, 0);
  for (int k = 2; k < K; ++k) {
    if (segs[k].xwave && !segs[k - 1].xwave && (ftarget[k] & segs[k - 1].w)) pre[k] = 1;
    if (segs[k - 1].xwave) pre[k] = 1;
  }

  // emission: an op's predecessors not done yet, and those that do not even wait
  // (phases); the current segment's ops that can be emitted, by their place in it
  std::vector<char> done(nops, 0), waiting(nops, 0);
  std::vector<int> undone(nops), unheld(nops), place_of(nops, -1);
  for (int i = 0; i < nops; ++i) undone[i] = unheld[i] = npreds(i);
  PlaceSet can_phase, can_rot, can_other, wanting;
  auto sort_in = [&](int li) {
    const int at = place_of[li], kind = ho[d.op_begin + li].kind;
    if (undone[li] == 0) {
      wanting.erase(at);
      (kind == 5 ? can_phase : kind == 4 ? can_rot : can_other).insert(at);
    } else if (unheld[li] == 0) {
      wanting.insert(at);
    }
  };
  auto set_waiting = [&](int li) {
    waiting[li] = 1;
    for (int j : succs(li))
      if (--unheld[j] == 0 && place_of[j] >= 0) sort_in(j);
  };
  auto set_done = [&](int li) {
    if (done[li]) return;
    done[li] = 1;
    for (int j : succs(li)) {
      if (!waiting[li]) --unheld[j];
      if ((--undone[j] == 0 || unheld[j] == 0) && place_of[j] >= 0) sort_in(j);
    }
  };
  d.general = 0;
  std::vector<int> pend;     // phases waiting for an op that needs them
  std::vector<int> rot_src;  // values of the pass's rotations (their signs)
  int sign_rec = -1;         // first table of the pass: takes the signs
  for (Seg& s : segs) {
    RegSegDev sd{};
    uint32_t regs = s.regs;
    const uint32_t keep_off = s.w | (s.io ? io_lane : 0u);
    for (int pos = L - 1; pos >= 0 && __builtin_popcount(regs) < RB; --pos)
      if (!(keep_off >> pos & 1)) regs |= 1u << pos;
    if (__builtin_popcount(regs) != RB) return fail(QSV_EINVAL, "internal: bad segment layout");
    int nr = 0, nt = 0;
    int regidx[32], thridx[32];
    for (int pos = 0; pos < L; ++pos) {
      regidx[pos] = -1;
      thridx[pos] = -1;
    }
    for (int pos = 0; pos < L; ++pos)
      if (regs >> pos & 1) {
        regidx[pos] = nr;
        sd.reg[nr++] = pos;
      }
    // lanes: the IO lane positions first, then the remaining ascending; then waves
    const uint32_t lanes = full & ~regs & ~s.w;
    if (s.io)
      for (int pos = 0; pos < L; ++pos)
        if (io_lane >> pos & 1) {
          thridx[pos] = nt;
          sd.thr[nt++] = pos;
        }
    for (int pos = 0; pos < L; ++pos)
      if ((lanes >> pos & 1) && thridx[pos] < 0) {
        thridx[pos] = nt;
        sd.thr[nt++] = pos;
      }
    if (nt != 6) return fail(QSV_EINVAL, "internal: bad lane layout");
    for (int pos = 0; pos < L; ++pos)
      if (s.w >> pos & 1) {
        thridx[pos] = nt;
        sd.thr[nt++] = pos;
      }
    if (nr != RB || nt != TB) return fail(QSV_EINVAL, "internal: bad segment layout");
    sd.xwave = (s.xwave ? 1 : 0) | (pre[&s - segs.data()] ? 2 : 0);
    {
      const int k = int(&s - segs.data());
      for (int q = 0; q < L; ++q) sd.mcol[q] = mcol[k][q];
      sd.mcst = mcst[k];
    }
    sd.op_begin = int(out_rops.size());
    uint32_t regmask = 0;
    for (int pos = 0; pos < L; ++pos)
      if (regidx[pos] >= 0) regmask |= 1u << pos;
    // a qubit of a phase: register bit a, or a thread bit / tile base bit in (tm, gm)
    auto place = [&](const TileOpDev& o, int j, int& ra, uint32_t& tm, uint64_t& gm) {
      ra = -1;
      if (o.lt[j] < 0) gm ^= uint64_t(1) << o.gq[j];
      else if (regidx[o.lt[j]] >= 0) ra = regidx[o.lt[j]];
      else tm ^= 1u << thridx[o.lt[j]];
    };
    // one phase op for the given ops (PhaseSub each)
    auto emit_phase = [&](const std::vector<int>& list) {
      RegOpDev r{};
      r.kind = 11;
      std::vector<TabComp> tab;
      struct Acc {  // a merged factor: one-qubit diagonals on one bit, or strings of one pattern
        PhaseEntDev e;
        std::vector<TabComp> comps;
        int odd;
      };
      std::vector<Acc> acc;
      auto merge = [&](const PhaseEntDev& e, const TabComp* c) {
        for (Acc& x : acc)
          if (x.e.kind == e.kind && x.e.rsg == e.rsg && x.e.tm == e.tm && x.e.gm == e.gm && x.e.tm2 == e.tm2 &&
              x.e.gm2 == e.gm2 && e.kind != 4) {
            if (c) x.comps.push_back(*c);
            x.odd ^= 1;
            return;
          }
        Acc x{e, {}, 1};
        if (c) x.comps.push_back(*c);
        acc.push_back(x);
      };
      for (int li : list) {
        const TileOpDev& o = ho[d.op_begin + li];
        PhaseEntDev e{};
        e.ra = -1;
        if (o.sub == PH_DIAG1) {
          int ra;
          place(o, 0, ra, e.tm, e.gm);
          if (o.m) {
            PhaseEntDev gr = e;
            gr.kind = 4;
            gr.moff = o.ins[1];
            gr.ra = ra;
            merge(gr, nullptr);
          }
          const TabComp c{0, o.moff, ra >= 0 ? ra : 0, 0, 0};
          if (ra >= 0) tab.push_back(c);
          else merge(e, &c);
        } else if (o.sub == PH_CZ) {
          int a0, a1;
          uint32_t t0 = 0, t1 = 0;
          uint64_t g0 = 0, g1 = 0;
          place(o, 0, a0, t0, g0);
          place(o, 1, a1, t1, g1);
          if (a0 >= 0 && a1 >= 0) {
            tab.push_back({2, 0, a0, a1, 0});
          } else if (a0 >= 0 || a1 >= 0) {
            const int ra = a0 >= 0 ? a0 : a1;
            r.tm[ra] ^= a0 >= 0 ? t1 : t0;
            r.gm[ra] ^= a0 >= 0 ? g1 : g0;
          } else {
            const bool sw = t0 < t1 || (t0 == t1 && g0 < g1);  // one order per pair
            e.kind = 2;
            e.tm = sw ? t1 : t0;
            e.gm = sw ? g1 : g0;
            e.tm2 = sw ? t0 : t1;
            e.gm2 = sw ? g0 : g1;
            merge(e, nullptr);
          }
        } else {
          uint32_t rm = 0;
          for (int j = 0; j < o.k; ++j) {
            int ra;
            place(o, j, ra, e.tm, e.gm);
            if (ra >= 0) rm |= 1u << ra;
          }
          for (int i = 0; i < NR; ++i)
            if (__builtin_popcount(uint32_t(i) & rm) & 1) e.rsg |= 1u << i;
          const TabComp c{3, o.moff, 0, 0, e.rsg};
          if (e.tm == 0 && e.gm == 0) {
            tab.push_back(c);
          } else {
            e.kind = rm ? 3 : 0;
            TabComp c0 = c;
            c0.rsg = rm ? 0u : 2u;  // (no register bit: the second value is the conjugate)
            if (!rm) e.rsg = 0;
            merge(e, &c0);
          }
        }
      }
      std::stable_sort(acc.begin(), acc.end(), [](const Acc& x, const Acc& y) {
        return x.e.kind != y.e.kind ? x.e.kind < y.e.kind : x.e.rsg < y.e.rsg;
      });
      if (!tab.empty()) {
        r.flags |= 1;
        r.moff = pool_take(NR);
        out.recs.push_back({1, r.moff, 0, NR, tab});
        if (sign_rec < 0) sign_rec = int(out.recs.size()) - 1;
      }
      for (int a = 0; a < RB; ++a)
        if (r.tm[a] || r.gm[a]) r.flags |= 4u | (256u << a);
      r.ent_begin = int(out.ents.size());
      int h = -1;
      for (size_t k = 0; k < acc.size(); ++k) {
        Acc& x = acc[k];
        if (x.e.kind == 2 && !x.odd) continue;  // CZ twice
        int moff = 0;
        if (x.e.kind == 0 || x.e.kind == 3) {
          const int nv = x.e.kind == 0 ? 2 : 1;
          moff = pool_take(nv);
          out.recs.push_back({1, moff, 0, nv, x.comps});
        }
        if (x.e.kind < 3 && (x.e.kind == 0 ? r.ent_count : r.ent_cz) == 0xffff) {  // (the head's fields)
          out_rops.push_back(r);
          r = RegOpDev{};
          r.kind = 11;
          r.ent_begin = int(out.ents.size());
        }
        if (x.e.kind == 0) {
          r.flags |= 2;
          if (r.ent_count++ == 0) r.ent_moff = moff;
        } else if (x.e.kind == 2) {
          r.flags |= 2;
          ++r.ent_cz;
        } else if (x.e.kind == 3) {
          if (h < 0 || r.h_rsg[h] != x.e.rsg) {
            if (h + 1 == kRegMaxH) {  // further patterns: another op
              out_rops.push_back(r);
              r = RegOpDev{};
              r.kind = 11;
              h = -1;
            }
            ++h;
            r.flags |= 16u << h;
            r.h_rsg[h] = x.e.rsg;
            r.h_begin[h] = int(out.ents.size());
            r.h_moff[h] = moff;
          }
          ++r.h_count[h];
        } else {
          if (!(r.flags & 8)) r.row_begin = int(out.ents.size());
          r.flags |= 8;
          ++r.row_count;
        }
        out.ents.push_back(x.e);
      }
      if (r.flags) out_rops.push_back(r);
      for (int li : list) set_done(li);
    };
    // Emission: phases wait (pend) until an op that does not commute with
    // them is due; then every waiting phase that touches a register bit goes
    // into one phase op. Rotations whose predecessors are done form layers.
    // the segment's last op, when a part that runs after its phase (and before
    // its exchange: rotations) can still join it
    auto open_op = [&](bool rots) -> RegOpDev* {
      if (int(out_rops.size()) == sd.op_begin) return nullptr;
      RegOpDev& l = out_rops.back();
      return l.kind == 11 && !l.xch && !(rots && l.rot) ? &l : nullptr;
    };
    auto emit_old = [&](int li) -> int {
      const int oi = d.op_begin + li;
      TileOpDev& o = ho[oi];
      if (o.kind == 0 && o.k == 1 && o.xswap) {  // exchange
        const int p = regidx[o.lt[0]];
        if (p < 0) return fail(QSV_EINVAL, "internal: target not in registers");
        if (!open_op(false)) {
          out_rops.push_back(RegOpDev{});
          out_rops.back().kind = 11;
        }
        RegOpDev& r = out_rops.back();
        uint32_t cm = 0, cv = 0;
        for (int pos = 0; pos < L; ++pos) {
          if (!(o.lcm >> pos & 1)) continue;
          const uint32_t val = (o.lcv >> pos) & 1;
          if (regidx[pos] >= 0) {
            cm |= 1u << regidx[pos];
            cv |= val << regidx[pos];
          } else {
            r.ti_cm |= 1u << thridx[pos];
            r.ti_cv |= val << thridx[pos];
          }
        }
        r.gcm = o.gcm;
        r.gcv = o.gcv;
        r.xch = 1u << p;
        for (int g = 0; g < NR / 2; ++g) {
          const uint32_t i = ((uint32_t(g) >> p) << (p + 1)) | (uint32_t(g) & ((1u << p) - 1));
          if ((i & cm) == cv) r.xch |= 256u << g;
        }
        set_done(li);
        return QSV_OK;
      }
      d.general = 1;
      RegOpDev r{};
      r.lop = oi;
      r.k = o.k;
      r.gcm = o.gcm;
      r.gcv = o.gcv;
      for (int pos = 0; pos < L; ++pos) {
        if (!(o.lcm >> pos & 1)) continue;
        const uint32_t val = (o.lcv >> pos) & 1;
        if (regidx[pos] >= 0) {
          r.ri_cm |= 1u << regidx[pos];
          r.ri_cv |= val << regidx[pos];
        } else {
          r.ti_cm |= 1u << thridx[pos];
          r.ti_cv |= val << thridx[pos];
        }
      }
      if (o.kind != 3) {
        const int nv = o.kind == 1 ? 1 << o.k : 1 << (2 * o.k);
        r.moff = pool_take(nv);
        out.recs.push_back({0, r.moff, o.moff, nv, {}});
      }
      if (o.kind == 3) {
        // Pauli-string gradient through LDS in this segment's layout
        r.kind = 8;
        r.aux[0] = o.ins[1];
        const int SBp = c64 ? 5 : 4;
        const uint32_t msk = (1u << SBp) - 1, fl = o.off[0];
        r.pf_lds = (fl ^ ((fl >> SBp) & msk) ^ ((fl >> (2 * SBp)) & msk)) * (c64 ? 8u : 16u);
        r.pz_reg = r.pz_thr = 0;
        for (int pos = 0; pos < L; ++pos) {
          if (!(o.off[1] >> pos & 1)) continue;
          if (regidx[pos] >= 0) r.pz_reg |= 1u << regidx[pos];
          else r.pz_thr |= 1u << thridx[pos];
        }
        r.pph = int(o.off[2]);
        r.pz_glob = uint64_t(o.off[3]) | (uint64_t(o.off[4]) << 32);
      } else if (o.kind == 0 && o.k <= 2) {
        r.kind = o.k == 1 ? 0 : 1;
        r.p1 = regidx[o.lt[0]];
        r.p2 = o.k == 2 ? regidx[o.lt[1]] : 0;
        if (r.p1 < 0 || (o.k == 2 && r.p2 < 0)) return fail(QSV_EINVAL, "internal: target not in registers");
        r.key = reg_key(r.kind, r.p1, r.p2, r.ri_cm != 0 || r.ti_cm != 0);
      } else if (o.kind == 1 && o.k <= 2) {
        r.kind = 2;
        for (int j = 0; j < o.k; ++j) {
          if (o.lt[j] >= 0) {
            if (regidx[o.lt[j]] >= 0) {
              r.dsrc[j] = 0;
              r.dbit[j] = regidx[o.lt[j]];
            } else {
              r.dsrc[j] = 1;
              r.dbit[j] = thridx[o.lt[j]];
            }
          } else {
            r.dsrc[j] = 2;
            r.dbit[j] = o.gq[j];
          }
        }
        // register-bit targets of the diagonal, ascending (-1: absent)
        int a = -1, b = -1;
        for (int j = 0; j < o.k; ++j) {
          if (r.dsrc[j] != 0) continue;
          if (a < 0) a = r.dbit[j];
          else b = r.dbit[j];
        }
        if (b >= 0 && b < a) std::swap(a, b);
        r.key = reg_key(2, a, b, r.ri_cm != 0 || r.ti_cm != 0);
      } else {
        r.kind = 3;
        o.moff = r.moff;  // the LDS form reads the same pool
      }
      out_rops.push_back(r);
      set_done(li);
      return QSV_OK;
    };
    auto flush = [&](const std::vector<int>& for_ops, bool all) {
      uint32_t t = regmask;
      for (int li : for_ops) t |= nd[li];
      std::vector<int> list, keep;
      for (int w : pend) (all || (dg[w] & t) ? list : keep).push_back(w);
      pend.swap(keep);
      if (!list.empty()) emit_phase(list);
    };
    for (size_t k = 0; k < s.ops.size(); ++k) place_of[s.ops[k]] = int(k);
    for (PlaceSet* x : {&can_phase, &can_rot, &can_other, &wanting}) x->reset(s.ops.size());
    for (int li : s.ops) sort_in(li);
    size_t emitted = 0;  // (phases: once they wait)
    auto take = [&](PlaceSet& from) {
      const int li = s.ops[size_t(from.first())];
      from.erase(from.first());
      place_of[li] = -1;
      ++emitted;
      return li;
    };
    while (emitted < s.ops.size()) {
      if (!can_phase.empty()) {
        const int li = take(can_phase);
        pend.push_back(li);
        set_waiting(li);
      } else if (!can_rot.empty()) {
        // one op per register bit
        if (!open_op(true)) {
          out_rops.push_back(RegOpDev{});
          out_rops.back().kind = 11;
        }
        RegOpDev& r = out_rops.back();
        r.roff = pool_take(RB);
        std::vector<int> rots;
        for (int at : can_rot.list()) rots.push_back(s.ops[size_t(at)]);
        for (int li : rots) {
          const TileOpDev& o = ho[d.op_begin + li];
          const int p = regidx[o.lt[0]];
          if (p < 0) return fail(QSV_EINVAL, "internal: target not in registers");
          if (r.rot >> p & 0x101u) continue;
          r.rot |= 1u << (p + (o.xswap == 1 ? 8 : 0));
          if (o.m) {
            r.rot |= 1u << (16 + p);
            r.aux[p] = o.ins[1];
          }
          out.recs.push_back({0, r.roff + p, o.moff, 1, {}});
          rot_src.push_back(o.moff);
          can_rot.erase(place_of[li]);
          place_of[li] = -1;
          ++emitted;
          set_done(li);
        }
      } else if (!can_other.empty()) {
        const int rc = emit_old(take(can_other));
        if (rc) return rc;
      } else if (!wanting.empty()) {
        std::vector<int> want;
        for (int at : wanting.list()) want.push_back(s.ops[size_t(at)]);
        flush(want, false);
      } else {
        return fail(QSV_EINVAL, "internal: segment emission stalled");
      }
    }
    {
      // ops folded into the next re-map: the phases before them are due here
      bool due = false;
      for (int li : s.fold)
        for (int q : preds(li)) due |= waiting[q] && !done[q];
      if (due) flush(s.fold, false);
      for (int li : s.fold) set_done(li);
    }
    if (&s == &segs.back()) flush({}, true);
    sd.op_count = int(out_rops.size()) - sd.op_begin;
    out_segs.push_back(sd);
    d.seg_count++;
  }
  // the signs that the rotations' angle reductions left (uniform factors)
  d.scale_off = -1;
  if (!rot_src.empty()) {
    std::vector<TabComp> sg;
    for (int src : rot_src) sg.push_back({4, src, 0, 0, 0});
    if (sign_rec >= 0) {
      std::vector<TabComp>& c = out.recs[size_t(sign_rec)].comps;
      c.insert(c.end(), sg.begin(), sg.end());
    } else {
      d.scale_off = pool_take(1);
      out.recs.push_back({1, d.scale_off, 0, 1, sg});
    }
  }
  d.rop_count = int(out.rops.size()) - d.rop_begin;
  d.ent_count = int(out.ents.size()) - d.ent_begin;
  d.pool_count = out.pool_elems - d.pool_begin;
  // LDS address tables of the pass's segments: the tile's LDS index is
  // swizzled by j ^ (j >> SB) ^ (j >> 2 SB) (low SB bits of each), linear over
  // XOR, so the byte offset splits into a per-thread part (XOR of per-bit
  // columns) and a per-element part
  const int SB = c64 ? 5 : 4;
  const uint32_t esz = c64 ? 8u : 16u;
  auto swz = [SB](uint32_t j) {
    const uint32_t m = (1u << SB) - 1;
    return j ^ ((j >> SB) & m) ^ ((j >> (2 * SB)) & m);
  };
  auto gbit = [&](int p) { return uint64_t(1) << (p < d.b ? p : d.hq[p - d.b]); };
  for (int si = d.seg_begin; si < d.seg_begin + d.seg_count; ++si) {
    RegSegDev& S = out_segs[size_t(si)];
    for (int k = 0; k < TB; ++k) S.gcol_t[k] = gbit(S.thr[k]);
    for (int k = 0; k < RB; ++k) S.gcol_r[k] = gbit(S.reg[k]);
    for (int k = 0; k < TB; ++k) S.tcol[k] = (swz(1u << S.thr[k]) * esz) << 16;
    for (int i = 0; i < (1 << RB); ++i) {
      uint32_t x = 0;
      for (int k = 0; k < RB; ++k)
        if (i >> k & 1) x |= 1u << S.reg[k];
      S.get_reg[i] = swz(x) * esz;
    }
    if (si == d.seg_begin) continue;
    const RegSegDev& O = out_segs[size_t(si) - 1];  // written through S's map
    S.tcst = swz(S.mcst) * esz;
    for (int k = 0; k < TB; ++k) S.tcol[k] |= swz(S.mcol[O.thr[k]]) * esz;
    for (int i = 0; i < (1 << RB); ++i) {
      uint32_t x = 0;
      for (int k = 0; k < RB; ++k)
        if (i >> k & 1) x ^= S.mcol[O.reg[k]];
      S.put_reg[i] = swz(x) * esz;
    }
  }
  return QSV_OK;
}

std::vector<RegHeadDev> op_heads(const SegBuild& sb) {
  std::vector<RegHeadDev> heads;
  heads.reserve(sb.rops.size() + 1);
  for (const RegOpDev& r : sb.rops) {
    RegHeadDev h{};
    h.flags = r.flags | uint32_t(r.kind) << 24;
    h.rot = r.rot;
    h.xch = r.xch;
    h.moff = r.moff;
    if (r.kind <= 1 && r.gcm == 0 && r.ti_cm == 0 && r.ri_cm == 0) {
      h.flags |= 1;
      h.xch = uint32_t(r.key);
    }
    h.roff = r.roff;
    h.ent_begin = r.ent_begin;
    h.ent_moff = r.ent_moff;
    h.ent_counts = uint32_t(r.ent_count) | uint32_t(r.ent_cz) << 16;
    h.row_count = r.row_count;
    for (int k = 0; k < kRegMaxH; ++k) h.h_rsg[k] = r.h_rsg[k];
    h.tm01 = r.tm[0] | r.tm[1] << 16;
    h.tm23 = r.tm[2] | r.tm[3] << 16;
    h.tm4 = r.tm[4];
    heads.push_back(h);
  }
  heads.push_back(RegHeadDev{});  // (read ahead past the last op)
  return heads;
}

std::vector<PhaseEntDev> op_entries(const SegBuild& sb) {
  std::vector<PhaseEntDev> e = sb.ents;
  e.resize(e.size() + kEntStep - 1);
  return e;
}

void assemble_pool(const SegBuild& sb, const std::vector<cd>& vals, std::vector<cd>& pool) {
  pool.assign(size_t(sb.pool_elems) + kPoolSpare, cd{0, 0});
  for (const PoolRec& r : sb.recs) {
    if (r.type == 0) {
      for (int i = 0; i < r.n; ++i) pool[size_t(r.dst + i)] = vals[size_t(r.src + i)];
      continue;
    }
    for (int i = 0; i < r.n; ++i) {
      cd z{1, 0};
      for (const TabComp& c : r.comps) {
        switch (c.type) {
          case 0: z = cmul(vals[size_t(c.src + (i >> c.a & 1))], z); break;
          case 1: z = cmul(vals[size_t(c.src + ((i >> c.a & 1) | (i >> c.b & 1) << 1))], z); break;
          case 2:
            if ((i >> c.a & 1) & (i >> c.b & 1)) z = {-z.re, -z.im};
            break;
          case 3: {
            const cd f = vals[size_t(c.src)];
            z = cmul((c.rsg >> i & 1) ? cd{f.re, -f.im} : f, z);
            break;
          }
          default: {
            const double f = vals[size_t(c.src) + 1].re;
            z = {f * z.re, f * z.im};
          }
        }
      }
      pool[size_t(r.dst + i)] = z;
    }
  }
}

}  // namespace qsv

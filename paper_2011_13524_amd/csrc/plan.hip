// Circuit fusion (section 5.4) and tile passes.
//
// Planning, on the host, in three stages:
//  1. Structure: every gate is reduced to its controlled form (section 4.3.2)
//     and marked diagonal or not.
//  2. Merge (section 5.4, merge of two successive gates): a gate joins the
//     block it depends on when that block is the only earlier block sharing
//     its qubits -- so it commutes with every block created in between -- and
//     the merged block stays within max_k qubits. Merges never raise the
//     arithmetic per amplitude: a dense k-qubit block costs 2^k complex
//     multiply-adds per amplitude, a diagonal block one multiply and an
//     exchange (X or controlled X) none. So diagonal gates join diagonal
//     blocks (the product stays diagonal); diagonal and exchange gates join a
//     dense block only on a subset of its qubits, and a dense gate absorbs a
//     diagonal or exchange block only on a subset of its own qubits. Block
//     matrices are products K_later K_earlier on the ascending union of
//     qubits.
//     Heavy mode (section 5.4, the heavy optimization): every gate carries,
//     per qubit it touches, the set of Paulis it commutes with there (a CNOT
//     commutes with Z on its control and X on its target; a diagonal gate
//     with Z on every qubit; RX/RY/RZ with X/Y/Z). A gate may then join an
//     earlier block that is not its immediate predecessor: walking back from
//     the newest block, it moves past every block with which it shares, on
//     each common qubit, a commuting Pauli (such a block and the gate are
//     then both block-diagonal in that Pauli's eigenbasis on every shared
//     qubit, so they commute), and joins the first block sharing a qubit
//     where the merge rules above allow it. On circuits whose gates all
//     commute (diagonal layers) this compresses the depth to a constant.
//  3. Passes: the blocks, broken into rotations, diagonals, exchanges and general
//     products, are scheduled into passes (segments.hip). A pass fixes a set of L
//     local qubits (always including the low b qubits, so that each run of 2^b
//     amplitudes is contiguous in HBM), the one of those tried that lets it take
//     the most ops in order. Diagonal ops and controls may sit on any qubit: for
//     one tile their non-local bits are constants.
//
// Execution: one kernel launch per pass; a tile is the 2^L amplitudes whose
// non-local bits spell its number. Persistent workgroups hold a tile in registers,
// re-mapped through LDS between segments (tile_reg.h); tiles that match no
// register shape (8 qubits and fewer, tile sizes set by hand) go through LDS, a
// barrier between blocks (k_tile). Each pass reads and writes the state once however
// many gates it applies.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "dev_common.h"
#include "plan.h"
#include "prof.h"
#include "tile_reg.h"

namespace qsv {

// LDS-resident tile pass: the whole tile in LDS, every block an LDS sweep.
// Used when the tile does not match the register-resident shape (small
// states, non-default tile sizes).
template <typename R, int KMAX>
__global__ void __launch_bounds__(256)
    k_tile(R* __restrict__ psi, const TilePassDev* __restrict__ passes, int pass_idx,
           const TileOpDev* __restrict__ ops, const cx<R>* __restrict__ pool) {
  extern __shared__ __align__(16) char smem[];
  cx<R>* t = reinterpret_cast<cx<R>*>(smem);
  const TilePassDev& P = passes[pass_idx];
  const int L = P.L, b = P.b, nh = P.nh, ng = P.ng;
  const uint64_t g = blockIdx.x;
  uint64_t base = 0;
  for (int j = 0; j < ng; ++j) base |= ((g >> j) & 1) << P.gpos[j];
  constexpr int V = sizeof(R) == 4 ? 2 : 1;
  const int TS = 1 << L;
  const uint32_t lowmask = (1u << b) - 1;
  for (int e = threadIdx.x; e < TS / V; e += blockDim.x) {
    const uint32_t j = uint32_t(e) * V;
    const uint32_t h = j >> b;
    uint64_t x = base + (j & lowmask);
    for (int i = 0; i < nh; ++i) x |= uint64_t((h >> i) & 1) << P.hq[i];
    AmpIO<R, V>::load(psi, x, &t[j]);
  }
  __syncthreads();
  for (int o = 0; o < P.op_count; ++o) {
    const TileOpDev& op = ops[P.op_begin + o];
    if ((base & op.gcm) != op.gcv) continue;  // non-local controls not met: skip for this tile
    lds_op<R, KMAX>(t, op, pool, L, base, NoSwz());
    __syncthreads();
  }
  for (int e = threadIdx.x; e < TS / V; e += blockDim.x) {
    const uint32_t j = uint32_t(e) * V;
    const uint32_t h = j >> b;
    uint64_t x = base + (j & lowmask);
    for (int i = 0; i < nh; ++i) x |= uint64_t((h >> i) & 1) << P.hq[i];
    AmpIO<R, V>::store(psi, x, &t[j]);
  }
}

// ------------------------------------------------------------------ host: matrices

namespace {

uint64_t qmask(const std::vector<int>& qs) {
  uint64_t m = 0;
  for (int q : qs) m |= uint64_t(1) << q;
  return m;
}

std::vector<int> mask_list(uint64_t m) {
  std::vector<int> v;
  v.reserve(size_t(__builtin_popcountll(m)));
  for (; m; m &= m - 1) v.push_back(__builtin_ctzll(m));
  return v;
}

GateInfo analyse(const Gate& g) {
  GateInfo gi;
  if (g.kind == Gate::ROTATION) {
    gi.targets = g.targets;
    gi.diagonal = (g.pauli == 3);
  } else if (g.kind == Gate::PAULI) {
    gi.targets = g.targets;
    gi.diagonal = std::all_of(g.paulis.begin(), g.paulis.end(), [](int p) { return p == 3; });
  } else {
    std::vector<cd> m = g.mat;
    std::vector<int> tq = g.targets;
    uint64_t cm = 0, cv = 0;
    for (size_t j = 0; j < g.controls.size(); ++j) {
      cm |= uint64_t(1) << g.controls[j];
      if (g.ctrl_vals[j]) cv |= uint64_t(1) << g.controls[j];
    }
    extract_controls(m, tq, cm, cv);
    gi.targets = tq;
    for (int q : mask_list(cm)) {
      gi.controls.push_back(q);
      gi.ctrl_vals.push_back(int(cv >> q & 1));
    }
    const int D = 1 << tq.size();
    bool dg = true;
    for (int r = 0; r < D && dg; ++r)
      for (int c = 0; c < D && dg; ++c)
        if (r != c && !(m[r * D + c].re == 0.0 && m[r * D + c].im == 0.0)) dg = false;
    gi.diagonal = dg;
    gi.exchange = tq.size() == 1 && m[0].re == 0 && m[0].im == 0 && m[1].re == 1 && m[1].im == 0 &&
                  m[2].re == 1 && m[2].im == 0 && m[3].re == 0 && m[3].im == 0;
    gi.mat = m;
  }
  gi.qubits = qmask(gi.targets) | qmask(gi.controls);
  return gi;
}

// Target matrix of a gate in its extracted form, for the given parameters.
void extracted_matrix(const Gate& g, const GateInfo& gi, const double* theta, std::vector<cd>& m) {
  if (g.kind == Gate::ROTATION || g.kind == Gate::PAULI) {
    gate_matrix(g, theta, m);
  } else {
    m = gi.mat;
  }
}

// Full matrix of a gate (targets + controls) embedded in the index space of
// `qs` (bit j <-> qs[j]); result is 2^|qs| square, row-major.
void embed(const std::vector<cd>& gm, const GateInfo& gi, const std::vector<int>& qs,
           std::vector<cd>& out) {
  const int k = int(qs.size());
  const int D = 1 << k;
  out.assign(size_t(D) * D, cd{0, 0});
  std::vector<int> tpos(gi.targets.size()), cpos(gi.controls.size());
  for (size_t j = 0; j < gi.targets.size(); ++j)
    tpos[j] = int(std::find(qs.begin(), qs.end(), gi.targets[j]) - qs.begin());
  for (size_t j = 0; j < gi.controls.size(); ++j)
    cpos[j] = int(std::find(qs.begin(), qs.end(), gi.controls[j]) - qs.begin());
  const int kt = int(tpos.size());
  const int Dt = 1 << kt;
  for (int c = 0; c < D; ++c) {
    bool on = true;
    for (size_t j = 0; j < cpos.size(); ++j)
      if (((c >> cpos[j]) & 1) != gi.ctrl_vals[j]) on = false;
    if (!on) {
      out[size_t(c) * D + c] = {1, 0};
      continue;
    }
    int cc = 0, rest = c;
    for (int j = 0; j < kt; ++j) {
      cc |= ((c >> tpos[j]) & 1) << j;
      rest &= ~(1 << tpos[j]);
    }
    for (int rr = 0; rr < Dt; ++rr) {
      int r = rest;
      for (int j = 0; j < kt; ++j) r |= ((rr >> j) & 1) << tpos[j];
      out[size_t(r) * D + c] = gm[size_t(rr) * Dt + cc];
    }
  }
}

void matmul(const std::vector<cd>& a, const std::vector<cd>& b, int D, std::vector<cd>& out) {
  out.assign(size_t(D) * D, cd{0, 0});
  for (int r = 0; r < D; ++r)
    for (int k = 0; k < D; ++k) {
      const cd x = a[size_t(r) * D + k];
      if (x.re == 0.0 && x.im == 0.0) continue;
      for (int c = 0; c < D; ++c) out[size_t(r) * D + c] = cadd(out[size_t(r) * D + c], cmul(x, b[size_t(k) * D + c]));
    }
}

// Paulis (bit 0: X, bit 1: Y, bit 2: Z) commuting with the gate on each of
// its qubits; 7 on qubits it does not touch. Rotations exp(i t P / 2) commute
// with P on their target(s) for every angle; fixed matrices are tested on
// their full matrix over targets and controls.
std::vector<uint8_t> commute_masks(const Gate& g, const GateInfo& gi, int n) {
  std::vector<uint8_t> m(size_t(n), 7);
  if (g.kind == Gate::ROTATION) {
    m[size_t(g.targets[0])] = uint8_t(1u << (g.pauli - 1));
    return m;
  }
  if (g.kind == Gate::PAULI) {
    for (size_t j = 0; j < g.targets.size(); ++j) m[size_t(g.targets[j])] = uint8_t(1u << (g.paulis[j] - 1));
    return m;
  }
  const std::vector<int> qs = mask_list(gi.qubits);
  std::vector<cd> M;
  embed(gi.mat, gi, qs, M);
  const int D = 1 << qs.size();
  double big = 0.0;
  for (const cd& z : M) big = std::max(big, std::fabs(z.re) + std::fabs(z.im));
  const double tol = 1e-12 * std::max(big, 1.0);
  auto close = [tol](cd a, cd b) { return std::fabs(a.re - b.re) + std::fabs(a.im - b.im) <= tol; };
  for (size_t j = 0; j < qs.size(); ++j) {
    const int bit = 1 << j;
    bool cx = true, cy = true, cz = true;
    for (int r = 0; r < D; ++r)
      for (int c = 0; c < D; ++c) {
        const cd v = M[size_t(r) * D + c];
        // Z_j M = M Z_j: no element between rows and columns whose bit j differs
        if (((r ^ c) & bit) && !close(v, cd{0, 0})) cz = false;
        // X_j M = M X_j: M[r ^ bit][c] = M[r][c ^ bit]
        if (!close(M[size_t(r ^ bit) * D + c], M[size_t(r) * D + (c ^ bit)])) cx = false;
        // Y_j M = M Y_j with Y|0> = i|1>, Y|1> = -i|0>:
        //   (Y M)[r][c] = (bit of r ? i : -i) M[r ^ bit][c]
        //   (M Y)[r][c] = (bit of c ? -i : i) M[r][c ^ bit]
        const cd a = M[size_t(r ^ bit) * D + c], b = M[size_t(r) * D + (c ^ bit)];
        const cd ya = (r & bit) ? cd{-a.im, a.re} : cd{a.im, -a.re};
        const cd yb = (c & bit) ? cd{b.im, -b.re} : cd{-b.im, b.re};
        if (!close(ya, yb)) cy = false;
      }
    m[size_t(qs[j])] = uint8_t((cx ? 1 : 0) | (cy ? 2 : 0) | (cz ? 4 : 0));
  }
  return m;
}

}  // namespace

// ------------------------------------------------------------------ host: planning

static int build_plan(qsv_plan* p) {
  const qsv_circuit& C = p->circ_copy;
  const int n = C.n;
  std::vector<GateInfo>& info = p->info;
  info.resize(C.gates.size());
  for (size_t i = 0; i < C.gates.size(); ++i) info[i] = analyse(C.gates[i]);

  // stage 2: merge
  std::vector<Block>& blocks = p->blocks;
  blocks.clear();
  std::vector<uint64_t> bq;  // qubit masks of blocks
  std::vector<char> bx;      // block is a single exchange gate
  std::vector<int> last(n, -1);
  std::vector<std::vector<uint8_t>> bcm;  // heavy: per block, commuting Paulis per qubit
  // merge rule for gate I joining block j (arithmetic per amplitude never rises)
  auto merge_ok = [&](int j, const GateInfo& I) {
    const Block& B = blocks[size_t(j)];
    const uint64_t uni = bq[size_t(j)] | I.qubits;
    const int ku = __builtin_popcountll(uni);
    const bool cheap_b = B.diagonal || bx[size_t(j)], cheap_i = I.diagonal || I.exchange;
    if (B.diagonal && I.diagonal) return ku <= 2;  // diagonal blocks stay register-friendly
    if (cheap_b && cheap_i) return false;          // the product would be dense: costlier
    if (cheap_i) return (I.qubits & ~bq[size_t(j)]) == 0;
    if (cheap_b) return (bq[size_t(j)] & ~I.qubits) == 0 && ku <= std::max(p->max_k, 1);
    return ku <= p->max_k;
  };
  for (size_t gi = 0; gi < C.gates.size(); ++gi) {
    const GateInfo& I = info[gi];
    std::vector<uint8_t> gcm;
    int target = -1;
    if (p->heavy) {
      gcm = commute_masks(C.gates[gi], I, n);
      for (int j = int(blocks.size()) - 1; j >= 0; --j) {
        const uint64_t shared = bq[size_t(j)] & I.qubits;
        if (!shared) continue;
        if (merge_ok(j, I)) {
          target = j;
          break;
        }
        bool passes = true;  // the gate commutes with block j: move it further back
        for (int q : mask_list(shared))
          if (!(bcm[size_t(j)][size_t(q)] & gcm[size_t(q)])) passes = false;
        if (!passes) break;
      }
    } else {
      int cand = p->nomerge ? -1 : -2;
      for (int q : mask_list(I.qubits)) {
        if (last[q] < 0) continue;
        if (cand == -2) cand = last[q];
        else if (cand != last[q]) cand = -1;
      }
      if (cand >= 0 && merge_ok(cand, I)) target = cand;
    }
    if (target >= 0) {
      Block& B = blocks[size_t(target)];
      B.gates.push_back(int(gi));
      bq[size_t(target)] |= I.qubits;
      bx[size_t(target)] = 0;
      B.diagonal = B.diagonal && I.diagonal;
      for (int q : mask_list(I.qubits)) {
        last[q] = std::max(last[q], target);
        if (p->heavy) bcm[size_t(target)][size_t(q)] &= gcm[size_t(q)];
      }
    } else {
      Block B;
      B.gates = {int(gi)};
      B.diagonal = I.diagonal;
      blocks.push_back(B);
      bq.push_back(I.qubits);
      bx.push_back(I.exchange ? 1 : 0);
      if (p->heavy) bcm.push_back(gcm);
      for (int q : mask_list(I.qubits)) last[q] = int(blocks.size()) - 1;
    }
  }
  for (size_t i = 0; i < blocks.size(); ++i) {
    Block& B = blocks[i];
    B.qubits = mask_list(bq[i]);
    if (B.gates.size() == 1) {
      const GateInfo& I = info[B.gates[0]];
      B.targets = I.targets;
      B.controls = I.controls;
      B.ctrl_vals = I.ctrl_vals;
      B.xswap = I.exchange;
    } else {
      B.targets = B.qubits;
      B.controls.clear();
      B.ctrl_vals.clear();
    }
    if (B.targets.size() > size_t(5)) return fail(QSV_EINVAL, "block wider than 5 qubits");
  }

  return QSV_OK;
}

// ------------------------------------------------------------------ elementary ops

// The plan's blocks as elementary ops. For register-resident passes a
// one-qubit unitary becomes a rotation between diagonals, and diagonal blocks
// fall apart into phases that the segment builder merges again wherever they
// are due together; every other block stays one op.
static void build_lops(qsv_plan* p) {
  const qsv_circuit& C = p->circ_copy;
  p->lops.clear();
  p->nvals = 0;
  auto add = [&](Lop l, int nv) {
    l.voff = p->nvals;
    p->nvals += nv;
    p->lops.push_back(std::move(l));
  };
  const bool c64 = p->dtype == QSV_C64;
  for (size_t bi = 0; bi < p->blocks.size(); ++bi) {
    const Block& B = p->blocks[bi];
    Lop whole;
    whole.kind = B.diagonal ? 1 : 0;
    whole.xswap = B.xswap;
    whole.targets = B.targets;
    whole.controls = B.controls;
    whole.ctrl_vals = B.ctrl_vals;
    whole.block = int(bi);
    const int nv = B.diagonal ? 1 << B.targets.size() : 1 << (2 * B.targets.size());
    if (p->reg_bits == 0) {
      add(whole, nv);
      continue;
    }
    if (B.diagonal) {
      std::vector<std::pair<int, std::vector<int>>> one;               // qubit -> its diagonal gates
      std::vector<std::pair<std::vector<int>, int>> cz;                // pair -> how often
      std::vector<std::pair<std::vector<int>, std::vector<int>>> str;  // qubits -> Z strings
      bool ok = true;
      for (int gi : B.gates) {
        const Gate& g = C.gates[size_t(gi)];
        if (g.kind == Gate::PAULI && g.targets.size() > 1) {
          std::vector<int> t = g.targets;
          std::sort(t.begin(), t.end());
          auto it = std::find_if(str.begin(), str.end(), [&](const auto& x) { return x.first == t; });
          if (it == str.end()) str.push_back({t, {gi}});
          else it->second.push_back(gi);
          continue;
        }
        const GateInfo& I = p->info[size_t(gi)];
        if (I.targets.size() == 1 && I.controls.empty()) {
          auto it = std::find_if(one.begin(), one.end(), [&](const auto& x) { return x.first == I.targets[0]; });
          if (it == one.end()) one.push_back({I.targets[0], {gi}});
          else it->second.push_back(gi);
        } else if (I.targets.size() == 1 && I.controls.size() == 1 && I.ctrl_vals[0] == 1 && I.mat[0].re == 1 &&
                   I.mat[0].im == 0 && I.mat[3].re == -1 && I.mat[3].im == 0) {
          std::vector<int> t = {std::min(I.targets[0], I.controls[0]), std::max(I.targets[0], I.controls[0])};
          auto it = std::find_if(cz.begin(), cz.end(), [&](const auto& x) { return x.first == t; });
          if (it == cz.end()) cz.push_back({t, 1});
          else ++it->second;
        } else {
          ok = false;
        }
      }
      if (ok) {
        for (auto& x : one) {
          Lop l;
          l.kind = 5;
          l.sub = PH_DIAG1;
          l.targets = {x.first};
          l.block = int(bi);
          l.lv = LV_DIAG1;
          l.gates = x.second;
          add(l, 2);
        }
        for (auto& x : cz) {
          if (x.second % 2 == 0) continue;
          Lop l;
          l.kind = 5;
          l.sub = PH_CZ;
          l.targets = x.first;
          l.block = int(bi);
          l.lv = LV_NONE;
          add(l, 0);
        }
        for (auto& x : str) {
          Lop l;
          l.kind = 5;
          l.sub = PH_ZSTR;
          l.targets = x.first;
          l.block = int(bi);
          l.lv = LV_ZSTR;
          l.gates = x.second;
          add(l, 1);
        }
        continue;
      }
    } else if (B.targets.size() == 1 && B.controls.empty() && !B.xswap) {
      // one-qubit block: diagonals around a single RX / RY, or any unitary
      std::vector<int> pre, post;
      int rot = -1, axis = 0;
      bool single = true, unitary = true, fixed = true;
      for (int gi : B.gates) {
        const Gate& g = C.gates[size_t(gi)];
        const GateInfo& I = p->info[size_t(gi)];
        if (I.targets.size() != 1 || !I.controls.empty()) single = unitary = false;
        fixed = fixed && g.slot < 0;
        if (g.kind == Gate::MATRIX && unitary && !runs_as_rotation(I.mat.data(), c64)) unitary = false;
        if (I.diagonal) {
          (rot < 0 ? pre : post).push_back(gi);
        } else if (rot < 0 && g.kind != Gate::MATRIX) {
          rot = gi;
          axis = g.kind == Gate::ROTATION ? g.pauli : g.paulis[0];
        } else {
          single = false;
        }
      }
      Lop l;
      l.targets = B.targets;
      l.block = int(bi);
      if (single && rot >= 0) {
        l.kind = 5;
        l.sub = PH_DIAG1;
        l.lv = LV_DIAG1;
        if (!pre.empty()) {
          l.gates = pre;
          add(l, 2);
        }
        Lop r = l;
        r.kind = 4;
        r.axis = axis;
        r.lv = LV_ROT;
        r.gates = {rot};
        add(r, 2);
        if (!post.empty()) {
          l.gates = post;
          add(l, 2);
        }
        continue;
      }
      if (unitary && fixed && B.gates.size() > 1) {  // (the product itself)
        std::vector<cd> acc = {{1, 0}, {0, 0}, {0, 0}, {1, 0}}, gm, tmp;
        for (int gi : B.gates) {
          extracted_matrix(C.gates[size_t(gi)], p->info[size_t(gi)], nullptr, gm);
          matmul(gm, acc, 2, tmp);
          acc.swap(tmp);
        }
        unitary = runs_as_rotation(acc.data(), c64);
      }
      if (unitary) {
        const int base = p->nvals;
        p->nvals += 6;
        l.kind = 5;
        l.sub = PH_DIAG1;
        l.lv = LV_U_FIRST;
        l.voff = base;
        p->lops.push_back(l);
        Lop r = l;
        r.kind = 4;
        r.axis = 2;
        r.lv = LV_U_ROT;
        r.voff = base + 2;
        p->lops.push_back(r);
        l.lv = LV_U_LAST;
        l.voff = base + 4;
        p->lops.push_back(l);
        continue;
      }
    }
    add(whole, nv);
  }
}

// Passes of the plan's elementary ops.
static int plan_passes(qsv_plan* p) {
  build_lops(p);
  std::vector<PassOp> ops(p->lops.size());
  for (size_t i = 0; i < p->lops.size(); ++i) {
    const Lop& l = p->lops[i];
    PassOp& o = ops[i];
    const uint64_t t = qmask(l.targets), c = qmask(l.controls);
    const bool diag = l.kind == 1 || l.kind == 5;
    o.nd = diag ? 0 : t;
    o.dg = diag ? (t | c) : c;
    o.local = diag ? 0 : t;
    o.lazy = l.kind == 5;
    o.weight = l.kind == 1 || l.xswap ? 1 : 4;
  }
  std::vector<std::vector<int>> po;
  std::vector<uint64_t> pl;
  const int rc = schedule_passes(ops, p->n, p->L, p->b, 1 << 30, po, pl);
  if (rc) return rc;
  p->passes.clear();
  for (size_t i = 0; i < po.size(); ++i) p->passes.push_back({mask_list(pl[i]), po[i]});
  return QSV_OK;
}

// Device tables for the passes and ops (value offsets fixed here; the values
// are uploaded at apply time).
static int upload_tables(qsv_plan* p) {
  const int n = p->n;
  std::vector<TilePassDev> hp;
  std::vector<TileOpDev> ho;
  for (const auto& P : p->passes) {
    TilePassDev d{};
    d.L = int(P.local.size());
    d.b = std::min(p->b, d.L);
    d.nh = d.L - d.b;
    if (d.nh > kTileMaxHigh) return fail(QSV_EINVAL, "too many high local qubits");
    for (int i = 0; i < d.nh; ++i) d.hq[i] = P.local[d.b + i];
    uint64_t lm = qmask(P.local);
    d.ng = 0;
    for (int q = 0; q < n; ++q)
      if (!(lm >> q & 1)) d.gpos[d.ng++] = q;
    pass_runs(d);
    d.scale_off = -1;
    d.op_begin = int(ho.size());
    d.op_count = int(P.ops.size());
    std::vector<int> lpos(64, -1);
    for (size_t i = 0; i < P.local.size(); ++i) lpos[P.local[i]] = int(i);
    for (int bi : P.ops) {
      const Lop& B = p->lops[size_t(bi)];
      TileOpDev o{};
      o.kind = B.kind;
      o.sub = B.sub;
      o.xswap = B.kind == 4 ? B.axis : (B.xswap ? 1 : 0);
      o.k = int(B.targets.size());
      o.moff = B.voff;
      for (size_t j = 0; j < B.controls.size(); ++j) {
        const int q = B.controls[j];
        if (lpos[q] >= 0) {
          o.lcm |= 1u << lpos[q];
          if (B.ctrl_vals[j]) o.lcv |= 1u << lpos[q];
        } else {
          o.gcm |= uint64_t(1) << q;
          if (B.ctrl_vals[j]) o.gcv |= uint64_t(1) << q;
        }
      }
      for (int j = 0; j < 5; ++j) {
        o.lt[j] = -1;
        o.gq[j] = -1;
      }
      for (int j = 0; j < o.k; ++j) {
        const int q = B.targets[j];
        if (lpos[q] >= 0) o.lt[j] = lpos[q];
        else o.gq[j] = q;
      }
      if (o.kind == 0 || o.kind == 4)
        for (int j = 0; j < o.k; ++j)
          if (o.lt[j] < 0) return fail(QSV_EINVAL, "internal: dense target not local");
      if (o.kind == 0) {
        uint32_t ins = o.lcm;
        for (int j = 0; j < o.k; ++j) ins |= 1u << o.lt[j];
        if (__builtin_popcount(ins) > 10) return fail(QSV_EINVAL, "too many local controls on one gate");
        o.m = 0;
        for (int q = 0; q < 32; ++q)
          if (ins >> q & 1) o.ins[o.m++] = q;
        for (int i = 0; i < (1 << o.k); ++i) {
          uint32_t off = 0;
          for (int j = 0; j < o.k; ++j)
            if (i >> j & 1) off |= 1u << o.lt[j];
          o.off[i] = off;
        }
        p->kmax_dense = std::max(p->kmax_dense, o.k);
      }
      ho.push_back(o);
    }
    d.seg_begin = int(p->sb.segs.size());
    d.seg_count = 0;
    if (p->reg_bits > 0) {
      const SegCfg cfg{p->reg_bits, p->thread_bits, p->dtype == QSV_C64};
      int rc = build_reg_segments(cfg, ho, d, p->sb);
      if (rc) return rc;
    }
    hp.push_back(d);
  }
  p->h_pass.swap(hp);
  p->h_ops.swap(ho);
  return QSV_OK;
}

// Host values of the plan's elementary ops for parameters theta (FP64).
static void plan_values(const qsv_plan* p, const double* theta, std::vector<cd>& vals) {
  const qsv_circuit& C = p->circ_copy;
  vals.assign(size_t(p->nvals), cd{0, 0});
  std::vector<cd> gm, full, acc, tmp;
  auto angle = [&](int gi) {
    const Gate& g = C.gates[size_t(gi)];
    return g.slot >= 0 ? theta[g.slot] : g.fixed_angle;
  };
  // matrix of a block's targets (its controls, if any, are apart)
  auto block_matrix = [&](const Block& B) {
    if (B.gates.size() == 1) {
      extracted_matrix(C.gates[size_t(B.gates[0])], p->info[size_t(B.gates[0])], theta, acc);
      return;
    }
    const int D = 1 << B.targets.size();
    acc.assign(size_t(D) * D, cd{0, 0});
    for (int i = 0; i < D; ++i) acc[size_t(i) * D + i] = {1, 0};
    for (int gidx : B.gates) {
      const GateInfo& gi = p->info[size_t(gidx)];
      extracted_matrix(C.gates[size_t(gidx)], gi, theta, gm);
      embed(gm, gi, B.targets, full);
      matmul(full, acc, D, tmp);  // later gate on the left
      acc.swap(tmp);
    }
  };
  for (const Lop& l : p->lops) {
    cd* v = vals.data() + l.voff;
    switch (l.lv) {
      case LV_NONE:
      case LV_U_FIRST:
      case LV_U_LAST:
        break;
      case LV_ROT:
        rotation_shears(angle(l.gates[0]), v);
        break;
      case LV_DIAG1:
        v[0] = v[1] = {1, 0};
        for (int gi : l.gates) {
          const Gate& g = C.gates[size_t(gi)];
          if (g.kind == Gate::MATRIX) extracted_matrix(g, p->info[size_t(gi)], theta, gm);
          else gate_matrix(g, theta, gm);
          v[0] = cmul(gm[0], v[0]);
          v[1] = cmul(gm[3], v[1]);
        }
        break;
      case LV_ZSTR: {
        double t = 0.0;
        if (l.gates.size() == 1) {
          t = angle(l.gates[0]);
          v[0] = {std::cos(t / 2), std::sin(t / 2)};
        } else {
          v[0] = {1, 0};
          for (int gi : l.gates) {
            t = angle(gi);
            v[0] = cmul(cd{std::cos(t / 2), std::sin(t / 2)}, v[0]);
          }
        }
        break;
      }
      case LV_U_ROT:
        block_matrix(p->blocks[size_t(l.block)]);
        unitary_to_rotation(acc.data(), v - 2);
        break;
      default: {
        const Block& B = p->blocks[size_t(l.block)];
        block_matrix(B);
        const int D = 1 << B.targets.size();
        if (B.diagonal)
          for (int i = 0; i < D; ++i) v[i] = acc[size_t(i) * D + i];
        else
          std::copy(acc.begin(), acc.end(), v);
      }
    }
  }
}

// Device pool for parameters theta: the values themselves (LDS-resident
// passes) or the tables of the register segments.
static void plan_pool(const qsv_plan* p, const double* theta, std::vector<cd>& pool) {
  std::vector<cd> vals;
  plan_values(p, theta, vals);
  if (p->reg_bits > 0) assemble_pool(p->sb, vals, pool);
  else pool.swap(vals);
}

// Device copies of the pass and op tables, made on the first apply so that
// planning itself needs no device; a circuit without parameters has its pool
// uploaded here too, once.
template <typename R>
static int ensure_tables(qsv_plan* p, hipStream_t stream) {
  if (p->d_pass) return QSV_OK;
  const size_t pool_n = size_t(std::max(1, p->reg_bits > 0 ? p->sb.pool_elems + kPoolSpare : p->nvals));
  std::vector<cx<R>> pool;
  if (p->circ_copy.nparams == 0) {
    std::vector<cd> vals;
    plan_pool(p, nullptr, vals);
    pool.resize(vals.size());
    for (size_t i = 0; i < vals.size(); ++i) pool[i] = {R(vals[i].re), R(vals[i].im)};
  }
  const std::vector<RegHeadDev> heads = op_heads(p->sb);
  const std::vector<PhaseEntDev> ents = op_entries(p->sb);
  void* buf[7] = {};
  const size_t bytes[7] = {p->h_pass.size() * sizeof(TilePassDev), p->h_ops.size() * sizeof(TileOpDev),
                           p->sb.segs.size() * sizeof(RegSegDev),  p->sb.rops.size() * sizeof(RegOpDev),
                           ents.size() * sizeof(PhaseEntDev), pool_n * sizeof(cx<R>),
                           heads.size() * sizeof(RegHeadDev)};
  const void* src[7] = {p->h_pass.data(), p->h_ops.data(), p->sb.segs.data(), p->sb.rops.data(),
                        ents.data(),       pool.data(),    heads.data()};
  int rc = QSV_OK;
  for (int i = 0; i < 7 && !rc; ++i)
    if (hipMalloc(&buf[i], std::max<size_t>(bytes[i], 16)) != hipSuccess) {
      (void)hipGetLastError();
      buf[i] = nullptr;
      rc = fail(QSV_ENOMEM, "plan table allocation failed");
    }
  for (int i = 0; i < 7 && !rc; ++i) {
    const size_t nb = i == 5 ? pool.size() * sizeof(cx<R>) : bytes[i];
    if (nb && hipMemcpyAsync(buf[i], src[i], nb, hipMemcpyHostToDevice, stream) != hipSuccess)
      rc = fail(QSV_EHIP, "plan table upload failed");
  }
  if (!rc && hipStreamSynchronize(stream) != hipSuccess) rc = fail(QSV_EHIP, "plan table upload failed");
  if (rc) {
    for (void* b : buf)
      if (b) (void)hipFree(b);
    return rc;
  }
  p->d_pass = static_cast<TilePassDev*>(buf[0]);
  p->d_ops = static_cast<TileOpDev*>(buf[1]);
  p->d_segs = static_cast<RegSegDev*>(buf[2]);
  p->d_rops = static_cast<RegOpDev*>(buf[3]);
  p->d_ents = static_cast<PhaseEntDev*>(buf[4]);
  p->d_pool = buf[5];
  p->d_heads = static_cast<RegHeadDev*>(buf[6]);
  p->pool_cap = pool_n;
  p->pass_grid.assign(p->passes.size(), 0);
  return QSV_OK;
}

// Register-resident pass launch for the instantiated shapes (register bits,
// thread bits): complex64 (4, 9), (4, 8), (5, 8), (4, 7); complex128 (4, 8), (4, 7).
template <typename R>
using TileRegFn = void (*)(R*, const TilePassDev*, int, uint32_t, const RegSegDev*, const RegHeadDev*, const RegOpDev*,
                           const TileOpDev*, const PhaseEntDev*, const cx<R>*);

template <typename R, int RB, int TB>
static TileRegFn<R> tile_reg_km(int km) {
  return km == 0   ? &k_tile_reg<R, RB, 0, TB>
         : km == 2 ? &k_tile_reg<R, RB, 2, TB>
         : km == 3 ? &k_tile_reg<R, RB, 3, TB>
                   : &k_tile_reg<R, RB, 5, TB>;
}

template <typename R, int TB>
static TileRegFn<R> tile_reg_small(int km) {
  return km == 0 ? &k_tile_reg<R, 3, 0, TB> : (km <= 3 ? &k_tile_reg<R, 3, 3, TB> : &k_tile_reg<R, 3, 5, TB>);
}
template <typename R>
static TileRegFn<R> tile_reg_fn(int rb, int tb, int km) {
  if (rb == 3) {  // states of one tile
    if (tb == 6) return tile_reg_small<R, 6>(km);
    if (tb == 7) return tile_reg_small<R, 7>(km);
    return tile_reg_small<R, 8>(km);
  }
  if constexpr (sizeof(R) == 4) {
    if (tb == 9) return tile_reg_km<R, 4, 9>(km);
    if (tb == 8 && rb == 5) return tile_reg_km<R, 5, 8>(km);
  }
  if (tb == 7) return tile_reg_km<R, 4, 7>(km);
  return tile_reg_km<R, 4, 8>(km);
}

template <typename R>
static int apply_fused_t(qsv_state* s, qsv_plan* p, const double* theta) {
  int trc = ensure_tables<R>(p, s->stream);
  if (trc) return trc;
  const bool upload = p->circ_copy.nparams > 0;
  if (upload) {
    std::vector<cd> vals;
    plan_pool(p, theta, vals);
    const size_t bytes = vals.size() * sizeof(cx<R>);
    if (p->stage_bytes < bytes) {
      if (p->h_stage) {
        if (p->stage_used) QSV_HIP_CHECK(hipEventSynchronize(p->stage_ev));
        (void)hipHostFree(p->h_stage);
        p->h_stage = nullptr;
        p->stage_bytes = 0;
      }
      if (hipHostMalloc(&p->h_stage, std::max<size_t>(bytes, 16), hipHostMallocDefault) != hipSuccess)
        return fail(QSV_ENOMEM, "plan staging allocation failed");
      p->stage_bytes = bytes;
    }
    if (!p->stage_ev) QSV_HIP_CHECK(hipEventCreateWithFlags(&p->stage_ev, hipEventDisableTiming));
    if (p->stage_used) QSV_HIP_CHECK(hipEventSynchronize(p->stage_ev));
    cx<R>* st = static_cast<cx<R>*>(p->h_stage);
    for (size_t i = 0; i < vals.size(); ++i) st[i] = {R(vals[i].re), R(vals[i].im)};
    if (bytes)
      QSV_HIP_CHECK(hipMemcpyAsync(p->d_pool, p->h_stage, bytes, hipMemcpyHostToDevice, s->stream));
  }
  const int n = s->n;
  for (size_t pi = 0; pi < p->passes.size(); ++pi) {
    const int L = int(p->passes[pi].local.size());
    const uint64_t tiles = dim(n - L);
    size_t lds = (size_t(1) << L) * sizeof(cx<R>);
    const TilePassDev& hp = p->h_pass[pi];
    if (hp.seg_count == 1) {
      // a single register-resident segment never touches LDS unless one of
      // its blocks runs through LDS: launch without it (higher occupancy)
      const RegSegDev& sg = p->sb.segs[size_t(hp.seg_begin)];
      bool needs = false;
      for (int o = sg.op_begin; o < sg.op_begin + sg.op_count; ++o) needs |= p->sb.rops[size_t(o)].kind == 3;
      if (!needs) lds = 0;
    }
    if (lds > 65536) {
      QSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tile<R, 2>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
      QSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tile<R, 3>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
      QSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tile<R, 5>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
    }
    ProfScope ps("tile", 2.0 * sizeof(cx<R>) * double(dim(n)), s->stream);
    R* psi = static_cast<R*>(s->ptr);
    const cx<R>* pool = static_cast<const cx<R>*>(p->d_pool);
    const dim3 grid(static_cast<unsigned>(tiles));
    const int km = p->kmax_dense <= 2 ? 2 : (p->kmax_dense <= 3 ? 3 : 5);
    if (p->h_pass[pi].seg_count > 0) {
      const TileRegFn<R> fn = tile_reg_fn<R>(p->reg_bits, p->thread_bits, hp.general ? km : 0);
      const unsigned nt = 1u << p->thread_bits;
      if (p->pass_grid[pi] == 0) {
        int per = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, int(nt), lds) != hipSuccess || per < 1) per = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, s->device) != hipSuccess || cus < 1)
          cus = 256;
        p->pass_grid[pi] = per * cus * 8;
      }
      const uint64_t wgs = std::min<uint64_t>(tiles, uint64_t(p->pass_grid[pi]));
      hipLaunchKernelGGL(fn, dim3(unsigned(wgs)), dim3(nt), lds, s->stream, psi, p->d_pass, int(pi), uint32_t(tiles), p->d_segs,
                         p->d_heads, p->d_rops, p->d_ops, p->d_ents, pool);
    } else if (km == 2)
      hipLaunchKernelGGL((k_tile<R, 2>), grid, dim3(256), lds, s->stream, psi, p->d_pass, int(pi), p->d_ops, pool);
    else if (km == 3)
      hipLaunchKernelGGL((k_tile<R, 3>), grid, dim3(256), lds, s->stream, psi, p->d_pass, int(pi), p->d_ops, pool);
    else
      hipLaunchKernelGGL((k_tile<R, 5>), grid, dim3(256), lds, s->stream, psi, p->d_pass, int(pi), p->d_ops, pool);
    QSV_HIP_CHECK(hipGetLastError());
  }
  if (upload) {
    QSV_HIP_CHECK(hipEventRecord(p->stage_ev, s->stream));
    p->stage_used = true;
  }
  return QSV_OK;
}

// Releases a plan and its device tables (keeps the error message).
static void plan_release(qsv_plan* p) {
  if (!p) return;
  adjoint_cache_free(p->adj);
  if (p->stage_used) (void)hipEventSynchronize(p->stage_ev);
  if (p->stage_ev) (void)hipEventDestroy(p->stage_ev);
  if (p->h_stage) (void)hipHostFree(p->h_stage);
  if (p->d_pool) (void)hipFree(p->d_pool);
  if (p->d_pass) (void)hipFree(p->d_pass);
  if (p->d_ops) (void)hipFree(p->d_ops);
  if (p->d_segs) (void)hipFree(p->d_segs);
  if (p->d_rops) (void)hipFree(p->d_rops);
  if (p->d_ents) (void)hipFree(p->d_ents);
  if (p->d_heads) (void)hipFree(p->d_heads);
  delete p;
}

// Plan with an explicit register tile shape (thread bits TB); tile_qubits /
// low_qubits 0 select the defaults.
static int plan_create(const qsv_circuit* c, qsv_dtype dtype, int max_k, int tile_qubits, int low_qubits,
                       int TB, qsv_plan** out, bool heavy = false, bool nomerge = false) {
  *out = nullptr;
  const int n = c->n;
  int L = tile_qubits > 0 ? tile_qubits : 12;
  // low qubits always local: 2^b amplitudes form one contiguous run, 128 bytes
  // (one cache line) at the default; fewer fixed low qubits leave more local
  // qubits free for the circuit, so fewer passes
  int b = low_qubits > 0 ? low_qubits : (dtype == QSV_C64 ? 4 : 3);
  if (L > 14 || (dtype == QSV_C128 && L > 13)) return fail(QSV_EINVAL, "tile of %d qubits exceeds LDS", L);
  L = std::min(L, n);
  b = std::min(b, L);
  if (dtype == QSV_C64 && b < 1) b = 1;
  if (L - b < max_k && L < n) return fail(QSV_EINVAL, "tile leaves fewer than max_k free qubits");
  if (L - b > kTileMaxHigh) return fail(QSV_EINVAL, "too many high local qubits");
  qsv_plan* p = new (std::nothrow) qsv_plan();
  if (!p) return fail(QSV_ENOMEM, "host allocation failed");
  p->n = n;
  p->dtype = dtype;
  p->max_k = max_k;
  p->heavy = heavy;
  p->nomerge = nomerge;
  p->L = L;
  p->b = b;
  // (blocks of 4-5 qubits run through LDS with 32-amplitude temporaries: the
  // 512-thread kernel would spill, and complex128 has no 512-thread shape)
  if ((dtype == QSV_C128 || max_k > 3) && TB == 9) TB = kRegThreadBits;
  // register bits: the rest of the tile; instantiated shapes (register bits,
  // thread bits): complex64 (4, 9), (4, 8), (5, 8), (4, 7); complex128 (4, 8), (4, 7);
  // both, for states of one tile, (3, 6), (3, 7), (3, 8)
  // states of 9 to 11 qubits, one tile: three register bits, so that as many
  // wavefronts as the tile allows share its chain of gates (the LDS kernel, which
  // keeps 8 qubits and fewer, takes a barrier per block). Measured, 8-layer
  // ansatz, LDS kernel against registers: complex128 9 qubits 102 and 45 us, 10
  // qubits 149 and 53, 11 qubits 246 and 56; complex64 95 and 43, 139 and 49, 226
  // and 57 us.
  if (n < 12 && L == n && L >= 9 && TB == kRegThreadBits) TB = L - 3;
  const int RB = L - TB;
  const bool rb_ok = RB == 4 || (RB == 3 && L == n && TB >= 6 && TB <= kRegThreadBits) ||
                     (dtype == QSV_C64 && RB == 5 && TB == 8);
  p->thread_bits = TB;
  p->reg_bits = (rb_ok && n >= L) ? RB : 0;
  p->circ_copy = *c;
  int rc = build_plan(p);
  if (!rc) rc = plan_passes(p);
  if (!rc) rc = upload_tables(p);
  if (rc) {
    plan_release(p);
    return rc;
  }
  *out = p;
  return QSV_OK;
}

int plan_unmerged(const qsv_circuit* c, qsv_dtype dtype, qsv_plan** out) {
  return plan_create(c, dtype, 1, 12, 0, kRegThreadBits, out, false, true);
}

void plan_free(qsv_plan* p) { plan_release(p); }

void plan_symbolic(const qsv_plan* p, std::vector<cd>& vals, std::vector<DynVal>& dyn) {
  const qsv_circuit& C = p->circ_copy;
  const std::vector<double> zero(size_t(std::max(1, C.nparams)), 0.0);
  plan_values(p, zero.data(), vals);
  dyn.clear();
  for (const Lop& l : p->lops)
    if (l.lv == LV_ROT || l.lv == LV_DIAG1 || l.lv == LV_ZSTR) {
      const Gate& g = C.gates[size_t(l.gates[0])];  // (unmerged: one gate)
      if (g.kind != Gate::MATRIX && g.slot >= 0)
        dyn.push_back({l.lv == LV_ROT ? 0 : (l.lv == LV_ZSTR ? 2 : 1), l.voff, g.slot, 1.0});
    }
}

}  // namespace qsv

using namespace qsv;

extern "C" {

int qsv_plan_fused(const qsv_circuit* c, qsv_dtype dtype, int max_k, int tile_qubits, int low_qubits,
                   qsv_plan** out) {
  return qsv_plan_fused_ex(c, dtype, max_k, tile_qubits, low_qubits, 0, out);
}

int qsv_plan_fused_ex(const qsv_circuit* c, qsv_dtype dtype, int max_k, int tile_qubits, int low_qubits,
                      int flags, qsv_plan** out) {
  clear_error();
  if (!out) return fail(QSV_EINVAL, "null output handle");
  *out = nullptr;
  if (!c) return fail(QSV_EINVAL, "null circuit");
  if (dtype != QSV_C64 && dtype != QSV_C128) return fail(QSV_EDTYPE, "unknown dtype");
  if (max_k < 1 || max_k > 5) return fail(QSV_EINVAL, "max_k must be in 1..5");
  if (flags & ~QSV_PLAN_HEAVY) return fail(QSV_EINVAL, "unknown plan flags 0x%x", unsigned(flags));
  // default tile: 2^12 amplitudes over 256 threads (TB = 8) x 16 in registers:
  // measured on MI355X, 2^12-amplitude tiles with 256 threads beat 2^13 with
  // 512 threads (6% at 30 qubits complex64, more workgroups in flight per
  // compute unit) despite more passes. QSV_TILE_QUBITS and
  // QSV_TILE_THREAD_BITS (7, 8, 9) override the defaults; qsv_plan_autotune
  // picks by measurement.
  int L = tile_qubits;
  if (const char* e = std::getenv("QSV_TILE_QUBITS"); e && tile_qubits <= 0) L = std::atoi(e);
  int TB = kRegThreadBits;
  if (const char* e = std::getenv("QSV_TILE_THREAD_BITS")) {
    const int v = std::atoi(e);
    TB = v == 9 ? 9 : (v == 7 ? 7 : 8);
  }
  return plan_create(c, dtype, max_k, L, low_qubits, TB, out, (flags & QSV_PLAN_HEAVY) != 0);
}

int qsv_plan_autotune(const qsv_circuit* c, qsv_state* scratch, const double* theta, int reps,
                      qsv_plan** out, int* choice) {
  clear_error();
  if (!out) return fail(QSV_EINVAL, "null output handle");
  *out = nullptr;
  if (!c) return fail(QSV_EINVAL, "null circuit");
  int rc = check_state(scratch);
  if (rc) return rc;
  if (scratch->n != c->n) return fail(QSV_ERANGE, "circuit has %d qubits, state %d", c->n, scratch->n);
  if (c->nparams > 0 && !theta) return fail(QSV_EINVAL, "circuit has parameters but theta is null");
  if (reps < 1 || reps > 100) return fail(QSV_EINVAL, "reps must be in 1..100");
  const qsv_dtype dt = scratch->dtype;
  // candidates: (max_k, tile qubits, thread bits)
  struct Cand { int k, L, TB; };
  std::vector<Cand> cands;
  for (int k : {1, 2, 3}) {
    cands.push_back({k, 12, 8});
    cands.push_back({k, 11, 7});
    if (dt == QSV_C64) {
      cands.push_back({k, 13, 9});
      cands.push_back({k, 13, 8});
    }
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  QSV_HIP_CHECK(hipEventCreate(&e0));
  QSV_HIP_CHECK(hipEventCreate(&e1));
  qsv_plan* best = nullptr;
  float best_ms = 0.f;
  int best_i = -1;
  for (size_t i = 0; i < cands.size(); ++i) {
    qsv_plan* p = nullptr;
    if (plan_create(c, dt, cands[i].k, cands[i].L, 0, cands[i].TB, &p) != QSV_OK) {
      clear_error();  // a shape that does not fit this circuit is skipped
      continue;
    }
    int r = qsv_apply_fused(scratch, p, theta);  // warm-up (uploads tables)
    if (!r) r = hipEventRecord(e0, scratch->stream) == hipSuccess ? QSV_OK : QSV_EHIP;
    for (int k = 0; k < reps && !r; ++k) r = qsv_apply_fused(scratch, p, theta);
    float ms = 0.f;
    if (!r) r = hipEventRecord(e1, scratch->stream) == hipSuccess ? QSV_OK : QSV_EHIP;
    if (!r) r = hipEventSynchronize(e1) == hipSuccess ? QSV_OK : QSV_EHIP;
    if (!r) r = hipEventElapsedTime(&ms, e0, e1) == hipSuccess ? QSV_OK : QSV_EHIP;
    if (r) {
      plan_release(p);
      plan_release(best);
      (void)hipEventDestroy(e0);
      (void)hipEventDestroy(e1);
      return fail(r, "autotune: timing a candidate failed");
    }
    if (!best || ms < best_ms) {
      plan_release(best);
      best = p;
      best_ms = ms;
      best_i = int(i);
    } else {
      plan_release(p);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (!best) return fail(QSV_EINVAL, "autotune: no candidate plan fits this circuit");
  if (choice) {
    choice[0] = cands[best_i].k;
    choice[1] = best->L;
    choice[2] = best->thread_bits;
    choice[3] = best->reg_bits;
  }
  *out = best;
  return QSV_OK;
}

int qsv_circuit_commute(const qsv_circuit* c, int gate, int qubit, int* paulis) {
  clear_error();
  if (!c || !paulis) return fail(QSV_EINVAL, "null argument");
  if (gate < 0 || gate >= int(c->gates.size())) return fail(QSV_ERANGE, "gate index %d out of range", gate);
  if (qubit < 0 || qubit >= c->n) return fail(QSV_ERANGE, "qubit %d out of range", qubit);
  const Gate& g = c->gates[size_t(gate)];
  *paulis = commute_masks(g, analyse(g), c->n)[size_t(qubit)];
  return QSV_OK;
}

int qsv_plan_info(const qsv_plan* p, int* passes, int* blocks, int* gates) {
  clear_error();
  if (!p) return fail(QSV_EINVAL, "null plan");
  if (passes) *passes = int(p->passes.size());
  if (blocks) *blocks = int(p->blocks.size());
  if (gates) *gates = int(p->circ_copy.gates.size());
  return QSV_OK;
}

int qsv_plan_stats(const qsv_plan* p, int* segments, int* lds_ops, int* kmax) {
  clear_error();
  if (!p) return fail(QSV_EINVAL, "null plan");
  int lo = 0;
  for (const RegOpDev& r : p->sb.rops)
    if (r.kind == 3) ++lo;
  if (segments) *segments = int(p->sb.segs.size());
  if (lds_ops) *lds_ops = lo;
  if (kmax) *kmax = p->kmax_dense;
  return QSV_OK;
}

int qsv_plan_free(qsv_plan* p) {
  clear_error();
  plan_release(p);
  return QSV_OK;
}

int qsv_apply_fused(qsv_state* s, qsv_plan* p, const double* theta) {
  clear_error();
  int rc = check_state(s);
  if (rc) return rc;
  if (!p) return fail(QSV_EINVAL, "null plan");
  if (p->n != s->n) return fail(QSV_ERANGE, "plan has %d qubits, state %d", p->n, s->n);
  if (p->dtype != s->dtype) return fail(QSV_EDTYPE, "plan and state dtypes differ");
  if (p->circ_copy.nparams > 0 && !theta) return fail(QSV_EINVAL, "plan has parameters but theta is null");
  return s->dtype == QSV_C64 ? apply_fused_t<float>(s, p, theta) : apply_fused_t<double>(s, p, theta);
}

}  // extern "C"

// Tiled reverse sweep of the adjoint gradient.
//
// The per-gate reverse sweep (psi <- U^dagger psi, lambda <- U^dagger lambda,
// and -Im<lambda|P|psi> before each parametric rotation) reads and writes both
// states once per gate. Here the reversed, daggered gate list is scheduled into
// tile passes exactly like a forward fused plan: a pass keeps L qubits local,
// a workgroup holds the psi and lambda tiles in LDS, applies every op of the
// pass to both and evaluates each gradient term on the tile. Gradient terms go
// into per-workgroup FP64 partials (each workgroup owns a fixed set of tiles
// and adds them in a fixed order), reduced per parameter at the end. Two
// states are streamed once per pass instead of once per gate.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "adj_reg.h"
#include "circuit.h"
#include "dev_common.h"
#include "plan.h"
#include "prof.h"
#include "tile_reg.h"

namespace qsv {

constexpr int kAdjTileThreads = 256;
constexpr int kAdjTileGrid = 2048;
constexpr int kAdjRegMin = 9;  // qubits from which the passes are register-resident

// TileOpDev with kind 2 = parametric rotation exp(i t P/2) seen by the reverse
// sweep: k = Pauli id, lt[0] = local target or -1, gq[0] = global qubit (Z on
// a non-local qubit), moff = pool offset of exp(-i t P/2) (2x2), ins[0] =
// partial row. One LDS sweep adds -Im<lambda|P|psi> of the tile and multiplies
// both states by exp(-i t P/2).

// Dense one-qubit op on both states in one sweep (matrix in registers).
template <typename R>
__device__ __forceinline__ void adj_dense1(cx<R>* __restrict__ ts, cx<R>* __restrict__ tl,
                                           const TileOpDev& op, const cx<R>* __restrict__ mat, int L) {
  const cx<R> m00 = mat[0], m01 = mat[1], m10 = mat[2], m11 = mat[3];
  const int cnt = 1 << (L - op.m);
  const uint32_t o1 = op.off[1];
  for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
    const uint32_t j0 = insert_zeros32(i, op.ins, op.m) | op.lcv;
    const cx<R> a = ts[j0], b = ts[j0 + o1], c = tl[j0], d = tl[j0 + o1];
    ts[j0] = cfma(m00, a, m01 * b);
    ts[j0 + o1] = cfma(m10, a, m11 * b);
    tl[j0] = cfma(m00, c, m01 * d);
    tl[j0 + o1] = cfma(m10, c, m11 * d);
  }
}

// Diagonal op on both states in one sweep.
template <typename R>
__device__ __forceinline__ void adj_diag(cx<R>* __restrict__ ts, cx<R>* __restrict__ tl,
                                         const TileOpDev& op, const cx<R>* __restrict__ d, int L,
                                         uint64_t base) {
  int gidx = 0;
  for (int b = 0; b < op.k; ++b)
    if (op.gq[b] >= 0) gidx |= int((base >> op.gq[b]) & 1) << b;
  const int TS = 1 << L;
  for (int j = threadIdx.x; j < TS; j += blockDim.x) {
    if ((uint32_t(j) & op.lcm) != op.lcv) continue;
    int idx = gidx;
    for (int b = 0; b < op.k; ++b)
      if (op.lt[b] >= 0) idx |= ((j >> op.lt[b]) & 1) << b;
    const cx<R> f = d[idx];
    ts[j] = f * ts[j];
    tl[j] = f * tl[j];
  }
}

// Gradient term of a rotation fused with its uncompute; returns this thread's
// share of -Im<lambda|P|psi> (taken before the uncompute).
template <typename R>
__device__ __forceinline__ double adj_rot(cx<R>* __restrict__ ps, cx<R>* __restrict__ la,
                                          const TileOpDev& op, const cx<R>* __restrict__ u, int L,
                                          uint64_t base) {
  double acc = 0.0;
  const int pauli = op.k;
  const int TS = 1 << L;
  const cx<R> u00 = u[0], u01 = u[1], u10 = u[2], u11 = u[3];
  if (pauli == 3) {
    // Z: sum_x (-1)^{x_q} Im(conj(lambda_x) psi_x); exp(-i t Z/2) is diagonal
    const int p = op.lt[0];
    if (p < 0) {
      const bool one = (base >> op.gq[0]) & 1;
      const double sg = one ? -1.0 : 1.0;
      const cx<R> f = one ? u11 : u00;
      for (int j = threadIdx.x; j < TS; j += blockDim.x) {
        const cx<R> a = ps[j], l = la[j];
        acc -= sg * (double(l.re) * a.im - double(l.im) * a.re);
        ps[j] = f * a;
        la[j] = f * l;
      }
    } else {
      for (int j = threadIdx.x; j < TS; j += blockDim.x) {
        const cx<R> a = ps[j], l = la[j];
        const bool one = (j >> p) & 1;
        const double im = double(l.re) * a.im - double(l.im) * a.re;
        acc -= one ? -im : im;
        const cx<R> f = one ? u11 : u00;
        ps[j] = f * a;
        la[j] = f * l;
      }
    }
  } else {
    const int p = op.lt[0];
    const uint32_t bit = 1u << p;
    for (int i = threadIdx.x; i < TS / 2; i += blockDim.x) {
      const uint32_t x0 = ((uint32_t(i) >> p) << (p + 1)) | (uint32_t(i) & (bit - 1));
      const uint32_t x1 = x0 | bit;
      const cx<R> a0 = ps[x0], a1 = ps[x1], l0 = la[x0], l1 = la[x1];
      const double a0r = a0.re, a0i = a0.im, a1r = a1.re, a1i = a1.im;
      const double l0r = l0.re, l0i = l0.im, l1r = l1.re, l1i = l1.im;
      double im;
      if (pauli == 1) im = (l0r * a1i - l0i * a1r) + (l1r * a0i - l1i * a0r);
      else im = -(l0r * a1r + l0i * a1i) + (l1r * a0r + l1i * a0i);
      acc -= im;
      ps[x0] = cfma(u00, a0, u01 * a1);
      ps[x1] = cfma(u10, a0, u11 * a1);
      la[x0] = cfma(u00, l0, u01 * l1);
      la[x1] = cfma(u10, l0, u11 * l1);
    }
  }
  return acc;
}

// Gradient term of a multi-qubit Pauli rotation exp(i t P/2) (TileOpDev kind
// 3): this thread's share of -Im<lambda|P|psi> over the tile, with
// (P psi)_x = i^ph (-1)^{|x & zy|} psi_{x ^ f} (the constant part of the sign
// folded into ph on the host; Z/Y factors on non-local qubits give the tile's
// sign). The states are not changed.
template <typename R>
__device__ __forceinline__ double adj_pauli_grad(const cx<R>* __restrict__ ps, const cx<R>* __restrict__ la,
                                                 const TileOpDev& op, int L, uint64_t base) {
  const uint32_t lf = op.off[0], zl = op.off[1];
  const uint64_t zg = uint64_t(op.off[3]) | (uint64_t(op.off[4]) << 32);
  const uint32_t gs = uint32_t(__popcll(base & zg) & 1);
  const int TS = 1 << L;
  double sr = 0.0, si = 0.0;
  for (int j = threadIdx.x; j < TS; j += blockDim.x) {
    const cx<R> a = ps[uint32_t(j) ^ lf], l = la[j];
    const double wr = double(l.re) * a.re + double(l.im) * a.im;
    const double wi = double(l.re) * a.im - double(l.im) * a.re;
    const bool neg = ((__popc(uint32_t(j) & zl) & 1) ^ gs) != 0;
    sr += neg ? -wr : wr;
    si += neg ? -wi : wi;
  }
  return neg_im_phase(sr, si, int(op.off[2]));
}

template <typename R, int KMAX>
__global__ void __launch_bounds__(kAdjTileThreads)
    k_tile_adj(R* __restrict__ psi, R* __restrict__ lam, const TilePassDev* __restrict__ passes,
               int pass_idx, const TileOpDev* __restrict__ ops, const cx<R>* __restrict__ pool,
               double* __restrict__ partial, uint64_t tiles) {
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[kAdjTileThreads / 64];
  const TilePassDev& P = passes[pass_idx];
  const int L = P.L, b = P.b, nh = P.nh;
  const int TS = 1 << L;
  cx<R>* ts = reinterpret_cast<cx<R>*>(smem);
  cx<R>* tl = ts + TS;
  constexpr int V = sizeof(R) == 4 ? 2 : 1;
  const uint32_t lowmask = (1u << b) - 1;
  for (uint64_t g = blockIdx.x; g < tiles; g += gridDim.x) {
    uint64_t base = 0;
    for (int j = 0; j < P.ng; ++j) base |= ((g >> j) & 1) << P.gpos[j];
    __syncthreads();  // previous tile's stores have read the LDS tiles
    for (int e = threadIdx.x; e < TS / V; e += blockDim.x) {
      const uint32_t j = uint32_t(e) * V;
      const uint32_t h = j >> b;
      uint64_t x = base + (j & lowmask);
      for (int i = 0; i < nh; ++i) x |= uint64_t((h >> i) & 1) << P.hq[i];
      AmpIO<R, V>::load(psi, x, &ts[j]);
      AmpIO<R, V>::load(lam, x, &tl[j]);
    }
    __syncthreads();
    for (int o = 0; o < P.op_count; ++o) {
      const TileOpDev& op = ops[P.op_begin + o];
      if ((base & op.gcm) != op.gcv) continue;
      if (op.kind == 2 || op.kind == 3) {
        double acc = op.kind == 2 ? adj_rot<R>(ts, tl, op, pool + op.moff, L, base)
                                  : adj_pauli_grad<R>(ts, tl, op, L, base);
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) acc += __shfl_xor(acc, s, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
          double r = 0.0;
          for (int w = 0; w < kAdjTileThreads / 64; ++w) r += red[w];
          partial[size_t(op.ins[0]) * gridDim.x + blockIdx.x] += r;
        }
      } else if (op.kind == 1) {
        adj_diag<R>(ts, tl, op, pool + op.moff, L, base);
      } else if (op.k == 1) {
        adj_dense1<R>(ts, tl, op, pool + op.moff, L);
      } else {
        lds_op<R, KMAX>(ts, op, pool, L, base, NoSwz());
        lds_op<R, KMAX>(tl, op, pool, L, base, NoSwz());
      }
      __syncthreads();
    }
    for (int e = threadIdx.x; e < TS / V; e += blockDim.x) {
      const uint32_t j = uint32_t(e) * V;
      const uint32_t h = j >> b;
      uint64_t x = base + (j & lowmask);
      for (int i = 0; i < nh; ++i) x |= uint64_t((h >> i) & 1) << P.hq[i];
      AmpIO<R, V>::store(psi, x, &ts[j]);
      AmpIO<R, V>::store(lam, x, &tl[j]);
    }
  }
}


// rows[r] = sum of the cols partials of row r (fixed order)
__global__ void __launch_bounds__(kAdjTileThreads)
    k_rows_sum(const double* __restrict__ partial, int cols, double* __restrict__ rows) {
  __shared__ double red[kAdjTileThreads / 64];
  double acc = 0.0;
  const double* p = partial + size_t(blockIdx.x) * cols;
  for (int i = threadIdx.x; i < cols; i += blockDim.x) acc += p[i];
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) acc += __shfl_xor(acc, s, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < kAdjTileThreads / 64; ++w) r += red[w];
    rows[blockIdx.x] = r;
  }
}

__global__ void k_zero_doubles(double* __restrict__ p, uint64_t n) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0;
}

// ------------------------------------------------------------------ host

namespace {

struct BOp {
  int kind;  // 0 dense, 1 diagonal, 2 gradient, 3 gradient of a Pauli string;
             // register-resident sweep: 4 rotation, 5 phase (TileOpDev)
  std::vector<int> targets, controls, ctrl_vals;
  std::vector<cd> val;  // dense: matrix; diagonal: diagonal entries; 4, 5: as TileOpDev
  int pauli = 0, row = -1;  // (row >= 0: with a gradient)
  int sub = 0;              // kind 5
  bool xswap = false;       // kind 0: Pauli X on the target
  int slot = -1;            // kinds 4, 5: the value is that of theta[slot]
  std::vector<int> paulis;  // kind 3: Pauli ids (1..3) of the string on targets
};

void dagger_inplace(std::vector<cd>& m, int D) {
  std::vector<cd> t(m.size());
  for (int r = 0; r < D; ++r)
    for (int c = 0; c < D; ++c) t[size_t(c) * D + r] = {m[size_t(r) * D + c].re, -m[size_t(r) * D + c].im};
  m.swap(t);
}

uint64_t qmask_of(const std::vector<int>& qs) {
  uint64_t m = 0;
  for (int q : qs) m |= uint64_t(1) << q;
  return m;
}

}  // namespace

template <typename R>
int adjoint_tables(const qsv_circuit* c, const double* theta, AdjTables& T) {
  const int n = c->n;
  // complex64 states of at least one 2^12 tile (complex128: 2^11) run
  // register-resident: 256 threads x 16 (8) amplitudes per state; smaller ones
  // down to 9 qubits are one tile of 8 amplitudes per thread
  const int Lc = sizeof(R) == 4 ? 12 : 11;
  const int L = T.L = std::min(n, Lc);
  const bool reg = T.reg = n >= kAdjRegMin;
  const int RB = n >= Lc && sizeof(R) == 4 ? 4 : 3;
  T.thread_bits = L - RB;
  const SegCfg cfg{RB, T.thread_bits, sizeof(R) == 4};
  const int b = std::min(L, sizeof(R) == 4 ? 4 : 3);  // 128-byte contiguous runs
  // reversed, daggered op list with gradient terms
  std::vector<BOp> ops;
  std::vector<int>& row_slot = T.row_slot;
  std::vector<cd> m;
  for (int gi = int(c->gates.size()) - 1; gi >= 0; --gi) {
    const Gate& g = c->gates[gi];
    // (without theta: only values that the parameters fill in later, as DynVals)
    const bool zstr = reg && g.kind == Gate::PAULI && g.targets.size() > 1 &&
                      std::all_of(g.paulis.begin(), g.paulis.end(), [](int p) { return p == 3; });
    if (!theta && g.kind != Gate::MATRIX && g.slot >= 0 && !zstr && !(reg && g.kind == Gate::ROTATION))
      return fail(QSV_EINVAL, "sweep tables of this circuit need its parameters");
    const double t = g.kind == Gate::MATRIX ? 0.0 : (g.slot >= 0 ? (theta ? theta[g.slot] : 0.0) : g.fixed_angle);
    if (g.kind == Gate::PAULI && g.slot >= 0) {
      // gradient term -Im<lambda|P|psi> of exp(i t P/2) (its own op), then the
      // uncompute exp(-i t P/2) as an ordinary gate below
      BOp gr;
      gr.kind = 3;
      gr.targets = g.targets;
      gr.paulis = g.paulis;
      gr.row = int(row_slot.size());
      row_slot.push_back(g.slot);
      ops.push_back(gr);
    }
    if (g.kind == Gate::ROTATION && (reg || g.slot >= 0)) {
      // gradient term (parametric) fused with the uncompute exp(-i t P/2)
      BOp gr;
      gr.pauli = g.pauli;
      gr.targets = g.targets;
      if (g.slot >= 0) {
        gr.row = int(row_slot.size());
        gr.slot = g.slot;
        row_slot.push_back(g.slot);
      }
      gr.val.resize(4);
      if (!reg) {
        gr.kind = 2;
        rotation_matrix(g.pauli, -t, gr.val.data());
      } else if (g.pauli == 3) {
        gr.kind = 5;
        gr.sub = PH_DIAG1;
        rotation_matrix(3, -t, gr.val.data());
        gr.val[1] = gr.val[3];
        gr.val.resize(2);
      } else {
        gr.kind = 4;
        rotation_shears(-t, gr.val.data());
        gr.val.resize(2);
      }
      ops.push_back(gr);
      continue;
    }
    if (zstr) {
      BOp z;
      z.kind = 5;
      z.sub = PH_ZSTR;
      z.targets = g.targets;
      z.slot = g.slot;
      z.val = {{std::cos(t / 2), -std::sin(t / 2)}};
      ops.push_back(z);
      continue;
    }
    gate_matrix(g, theta, m);
    std::vector<int> tq = g.targets;
    dagger_inplace(m, 1 << tq.size());
    uint64_t cm = 0, cv = 0;
    for (size_t j = 0; j < g.controls.size(); ++j) {
      cm |= uint64_t(1) << g.controls[j];
      if (g.ctrl_vals[j]) cv |= uint64_t(1) << g.controls[j];
    }
    extract_controls(m, tq, cm, cv);
    const int D = 1 << tq.size();
    bool diag = true;
    for (int r = 0; r < D && diag; ++r)
      for (int cc = 0; cc < D && diag; ++cc)
        if (r != cc && !(m[size_t(r) * D + cc].re == 0 && m[size_t(r) * D + cc].im == 0)) diag = false;
    BOp op;
    op.kind = diag ? 1 : 0;
    op.targets = tq;
    for (int q = 0; q < 64; ++q)
      if (cm >> q & 1) {
        op.controls.push_back(q);
        op.ctrl_vals.push_back(int(cv >> q & 1));
      }
    const bool exch = tq.size() == 1 && m[0].re == 0 && m[0].im == 0 && m[1].re == 1 && m[1].im == 0 &&
                      m[2].re == 1 && m[2].im == 0 && m[3].re == 0 && m[3].im == 0;
    if (diag) {
      if (tq.size() > 5) return fail(QSV_EINVAL, "diagonal gate too wide for the tiled sweep");
      for (int i = 0; i < D; ++i) op.val.push_back(m[size_t(i) * D + i]);
      if (reg && tq.size() == 1 && cm == 0) {
        op.kind = 5;
        op.sub = PH_DIAG1;
      } else if (reg && tq.size() == 1 && op.controls.size() == 1 && cv == cm && m[0].re == 1 && m[0].im == 0 &&
                 m[3].re == -1 && m[3].im == 0) {
        op.kind = 5;
        op.sub = PH_CZ;
        op.targets.push_back(op.controls[0]);
        op.controls.clear();
        op.ctrl_vals.clear();
        op.val.clear();
      }
    } else if (reg && tq.size() == 1 && cm == 0 && !exch && runs_as_rotation(m.data(), sizeof(R) == 4)) {
      // diagonal, rotation, diagonal
      cd u[6];
      unitary_to_rotation(m.data(), u);
      op.kind = 5;
      op.sub = PH_DIAG1;
      op.val = {u[0], u[1]};
      ops.push_back(op);
      op.kind = 4;
      op.pauli = 2;
      op.val = {u[2], u[3]};
      ops.push_back(op);
      op.kind = 5;
      op.val = {u[4], u[5]};
    } else {
      op.val = m;
      op.xswap = exch;
    }
    ops.push_back(op);
  }
  // passes (as in the forward planner): dense targets must be local, at most
  // kAdjMaxRows gradient rows per register-resident pass
  std::vector<std::vector<int>> pass_ops;
  std::vector<uint64_t> pass_local;
  {
    std::vector<PassOp> po(ops.size());
    for (size_t i = 0; i < ops.size(); ++i) {
      const BOp& o = ops[i];
      const uint64_t t = qmask_of(o.targets), cq = qmask_of(o.controls);
      uint64_t flip = t;  // qubits acted on non-diagonally
      if (o.kind == 1 || o.kind == 5 || (o.kind == 2 && o.pauli == 3)) flip = 0;
      if (o.kind == 3)  // the X/Y qubits of the string: pairs x, x ^ f in one tile
        for (size_t j = 0; j < o.targets.size(); ++j)
          if (o.paulis[j] == 3) flip &= ~(uint64_t(1) << o.targets[j]);
      po[i].nd = po[i].local = flip;
      po[i].dg = (t & ~flip) | cq;
      po[i].lazy = o.kind == 5;
      po[i].rows = o.row >= 0 ? 1 : 0;
    }
    const int rc = schedule_passes(po, n, L, b, reg ? kAdjMaxRows : 1 << 30, pass_ops, pass_local);
    if (rc) return rc;
  }
  // device tables
  std::vector<TilePassDev>& hp = T.hp;
  std::vector<TileOpDev>& ho = T.ho;
  std::vector<cd>& vals = T.vals;
  std::vector<int>& prow = T.prow;
  SegBuild& sb = T.sb;
  int& kmax = T.kmax;
  for (size_t pi = 0; pi < pass_ops.size(); ++pi) {
    const uint64_t local = pass_local[pi];
    std::vector<int> lpos(64, -1), loc;
    for (int q = 0; q < n; ++q)
      if (local >> q & 1) {
        lpos[q] = int(loc.size());
        loc.push_back(q);
      }
    TilePassDev d{};
    d.L = L;
    d.b = b;
    d.nh = L - b;
    for (int i = 0; i < d.nh; ++i) d.hq[i] = loc[b + i];
    d.ng = 0;
    for (int q = 0; q < n; ++q)
      if (!(local >> q & 1)) d.gpos[d.ng++] = q;
    pass_runs(d);
    d.scale_off = -1;
    d.op_begin = int(ho.size());
    d.op_count = int(pass_ops[pi].size());
    d.row_begin = int(prow.size());
    d.row_count = 0;
    for (int oi : pass_ops[pi]) {
      const BOp& o = ops[oi];
      TileOpDev t{};
      for (int j = 0; j < 5; ++j) t.lt[j] = t.gq[j] = -1;
      if (o.kind == 3) {
        t.kind = 3;
        t.k = int(o.targets.size());
        t.ins[0] = o.row;
        t.ins[1] = d.row_count++;
        prow.push_back(o.row);
        uint32_t lf = 0, zl = 0;
        uint64_t zg = 0;
        int ny = 0;
        for (size_t j = 0; j < o.targets.size(); ++j) {
          const int q = o.targets[j], pid = o.paulis[j];
          if (pid == 2) ++ny;
          if (pid != 3) lf |= 1u << lpos[q];  // (X/Y qubits are local)
          if (pid != 1) {
            if (lpos[q] >= 0) zl |= 1u << lpos[q];
            else zg |= uint64_t(1) << q;
          }
        }
        t.off[0] = lf;
        t.off[1] = zl;
        // (P psi)_x = i^nY (-1)^{|(x ^ f) & zy|} psi_{x ^ f}; the part of the
        // sign from f & zy is a constant: two more quarter turns when odd
        t.off[2] = uint32_t((ny + 2 * (__builtin_popcount(lf & zl) & 1)) & 3);
        t.off[3] = uint32_t(zg);
        t.off[4] = uint32_t(zg >> 32);
        ho.push_back(t);
        continue;
      }
      if (o.kind == 2) {
        t.kind = 2;
        t.k = o.pauli;
        t.ins[0] = o.row;
        t.ins[1] = d.row_count++;
        prow.push_back(o.row);
        t.moff = int(vals.size());
        vals.insert(vals.end(), o.val.begin(), o.val.end());
        const int q = o.targets[0];
        if (lpos[q] >= 0) t.lt[0] = lpos[q];
        else t.gq[0] = q;
        ho.push_back(t);
        continue;
      }
      t.kind = o.kind;
      t.sub = o.sub;
      t.k = int(o.targets.size());
      t.moff = int(vals.size());
      vals.insert(vals.end(), o.val.begin(), o.val.end());
      if (o.slot >= 0) T.dyn.push_back({o.kind == 4 ? 0 : (o.sub == PH_ZSTR ? 2 : 1), t.moff, o.slot, -1.0});
      t.xswap = o.kind == 4 ? o.pauli : (o.xswap ? 1 : 0);
      if (o.kind >= 4 && o.row >= 0) {
        t.m = 1;
        t.ins[0] = o.row;
        t.ins[1] = d.row_count++;
        prow.push_back(o.row);
      }
      for (size_t j = 0; j < o.controls.size(); ++j) {
        const int q = o.controls[j];
        if (lpos[q] >= 0) {
          t.lcm |= 1u << lpos[q];
          if (o.ctrl_vals[j]) t.lcv |= 1u << lpos[q];
        } else {
          t.gcm |= uint64_t(1) << q;
          if (o.ctrl_vals[j]) t.gcv |= uint64_t(1) << q;
        }
      }
      for (int j = 0; j < t.k; ++j) {
        const int q = o.targets[j];
        if (lpos[q] >= 0) t.lt[j] = lpos[q];
        else t.gq[j] = q;
      }
      if (t.kind == 0) {
        kmax = std::max(kmax, t.k);
        uint32_t ins = t.lcm;
        for (int j = 0; j < t.k; ++j) ins |= 1u << t.lt[j];
        if (__builtin_popcount(ins) > 10) return fail(QSV_EINVAL, "too many local controls on one gate");
        t.m = 0;
        for (int q = 0; q < 32; ++q)
          if (ins >> q & 1) t.ins[t.m++] = q;
        for (int i = 0; i < (1 << t.k); ++i) {
          uint32_t off = 0;
          for (int j = 0; j < t.k; ++j)
            if (i >> j & 1) off |= 1u << t.lt[j];
          t.off[i] = off;
        }
      }
      ho.push_back(t);
    }
    if (reg) {
      d.seg_begin = int(sb.segs.size());
      d.seg_count = 0;
      const int rc = build_reg_segments(cfg, ho, d, sb);
      if (rc) return rc;
    }
    hp.push_back(d);
  }
  return QSV_OK;
}
template int adjoint_tables<float>(const qsv_circuit*, const double*, AdjTables&);
template int adjoint_tables<double>(const qsv_circuit*, const double*, AdjTables&);

// The tables of a sweep that do not depend on theta, one after the other.
struct AdjLayout {
  size_t pass, ops, segs, rops, ents, heads, prow, bytes;
};

static AdjLayout adj_pack(const AdjTables& T, std::vector<char>* out) {
  const std::vector<RegHeadDev> heads = op_heads(T.sb);
  const std::vector<PhaseEntDev> ents = op_entries(T.sb);
  AdjLayout o{};
  size_t at = 0;
  auto put = [&](size_t& off, const void* p, size_t bytes) {
    off = at;
    at += (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    if (!out) return;
    out->resize(at);
    if (bytes) std::copy_n(static_cast<const char*>(p), bytes, out->data() + off);
  };
  put(o.pass, T.hp.data(), T.hp.size() * sizeof(TilePassDev));
  put(o.ops, T.ho.data(), T.ho.size() * sizeof(TileOpDev));
  put(o.segs, T.sb.segs.data(), T.sb.segs.size() * sizeof(RegSegDev));
  put(o.rops, T.sb.rops.data(), T.sb.rops.size() * sizeof(RegOpDev));
  put(o.ents, ents.data(), ents.size() * sizeof(PhaseEntDev));
  put(o.heads, heads.data(), heads.size() * sizeof(RegHeadDev));
  put(o.prow, T.prow.data(), T.prow.size() * sizeof(int));
  o.bytes = at;
  return o;
}

void adjoint_values(const AdjTables& T, const double* theta, std::vector<cd>& vals) {
  vals = T.vals;
  for (const DynVal& d : T.dyn) {
    const double t = d.sgn * theta[d.slot];
    cd* v = &vals[size_t(d.voff)];
    if (d.type == 0) {
      rotation_shears(t, v);
    } else if (d.type == 1) {
      cd m[4];
      rotation_matrix(3, t, m);
      v[0] = m[0];
      v[1] = m[3];
    } else {
      v[0] = {std::cos(t / 2), std::sin(t / 2)};
    }
  }
}

template <typename R>
AdjCache* adjoint_cache(qsv_plan* plan, const qsv_circuit* c) {
  if (c->n < kAdjRegMin || !same_circuit(*c, plan->circ_copy)) return nullptr;
  if (!plan->adj) {
    plan->adj = new AdjCache();
    if (adjoint_tables<R>(c, nullptr, plan->adj->T) != QSV_OK) clear_error();
    else plan->adj->usable = true;
  }
  return plan->adj->usable ? plan->adj : nullptr;
}
template AdjCache* adjoint_cache<float>(qsv_plan*, const qsv_circuit*);
template AdjCache* adjoint_cache<double>(qsv_plan*, const qsv_circuit*);

void adjoint_cache_free(AdjCache* a) {
  if (!a) return;
  if (a->dev) (void)hipFree(a->dev);
  delete a;
}

template <typename R>
using AdjRegFn = void (*)(R*, R*, const TilePassDev*, int, const RegSegDev*, const RegHeadDev*, const RegOpDev*,
                          const TileOpDev*, const PhaseEntDev*, const cx<R>*, const int*, double*, uint64_t, R, R);

template <typename R, int TB>
static AdjRegFn<R> adj_reg_small(int km) {
  return km == 0   ? &k_adj_reg<R, double, 3, 0, TB>
         : km <= 3 ? &k_adj_reg<R, double, 3, 3, TB>
                   : &k_adj_reg<R, double, 3, 5, TB>;
}
template <typename R, typename G>
static AdjRegFn<R> adj_reg_full(int km) {
  constexpr int RB = sizeof(R) == 4 ? 4 : 3;
  return km == 0   ? &k_adj_reg<R, G, RB, 0, 8>
         : km <= 2 ? &k_adj_reg<R, G, RB, 2, 8>
         : km <= 3 ? &k_adj_reg<R, G, RB, 3, 8>
                   : &k_adj_reg<R, G, RB, 5, 8>;
}

// Qubits from which complex64 gradients form their products in FP32 (grad_xy).
constexpr int kAdjFp32Min = 20;

// The sweep's kernel for n qubits, register bits rb, thread bits tb and the widest
// dense op (0: no general products).
template <typename R>
static AdjRegFn<R> adj_reg_fn(int n, int rb, int tb, int km) {
  if (tb == 6) return adj_reg_small<R, 6>(km);
  if (tb == 7) return adj_reg_small<R, 7>(km);
  if (rb < (sizeof(R) == 4 ? 4 : 3)) return adj_reg_small<R, 8>(km);
  return n >= kAdjFp32Min ? adj_reg_full<R, R>(km) : adj_reg_full<R, double>(km);
}

// Reverse sweep by tile passes. On entry psi = psi_L, lam = H psi_L and energy =
// <psi|lam>; on return both are uncomputed and rows[r] holds the gradient term of the r-th
// parametric rotation counted from the end (T.row_slot maps rows to slots). vals:
// the host values; cache: T's, if it is kept with a plan (else null).
template <typename R>
int adjoint_backward_tiled(const AdjTables& T, std::vector<cd>& vals, AdjCache* cache, int n, double energy,
                           qsv_state* psi, qsv_state* lam, std::vector<double>& rows) {
  const std::vector<int>& row_slot = T.row_slot;
  const int L = T.L, kmax = T.kmax;
  const bool reg = T.reg;
  const std::vector<TilePassDev>& hp = T.hp;
  std::vector<cx<R>> pool;
  {
    std::vector<cd> pv;
    if (reg) assemble_pool(T.sb, vals, pv);
    else pv.swap(vals);
    pool.resize(pv.size());
    for (size_t i = 0; i < pv.size(); ++i) pool[i] = {R(pv[i].re), R(pv[i].im)};
  }
  const int nrows = int(row_slot.size());
  const uint64_t tiles = dim(n - L);
  // register-resident passes: tile + gradient slots in LDS
  const int nt = 1 << T.thread_bits;
  const size_t reg_lds = (size_t(1) << L) * sizeof(cx<R>) + size_t(kAdjMaxRows) * (nt / 64) * sizeof(double);
  bool general = false;
  for (const TilePassDev& p : hp) general |= p.general != 0;
  // persistent grid: for the register sweep, eight rounds of the workgroups
  // the device holds at once (the variant's occupancy times the compute
  // units), so no round runs part-full and the last one is short (measured:
  // 24 qubits complex64 27.7 ms with a fixed 1024, 25.1 ms with 4 x 768, 24.7
  // ms with 8 x 768; 32 qubits 8.10, 7.14 and 6.98 s); QSV_ADJOINT_GRID
  // overrides it (tuning, and tests that give every workgroup a ragged range
  // of several tiles at small sizes)
  uint64_t gmax = kAdjTileGrid;
  if (reg) {
    int per_cu = 0, cus = 0;
    const AdjRegFn<R> fn = adj_reg_fn<R>(n, L - T.thread_bits, T.thread_bits, general ? kmax : 0);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, nt, reg_lds) != hipSuccess || per_cu < 1)
      per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, psi->device) != hipSuccess || cus < 1)
      cus = 256;
    gmax = uint64_t(per_cu) * uint64_t(cus) * 8;
  }
  if (const char* e = std::getenv("QSV_ADJOINT_GRID")) gmax = uint64_t(std::max(1, std::atoi(e)));
  const int G = int(std::min<uint64_t>(tiles, gmax));
  // psi's work buffer (kept for the next gradient; the sweep synchronises before
  // returning): pool | partial[nrows x G] | rows[nrows], and the tables unless they
  // are kept with a plan, each uploaded in one copy
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  std::vector<char> stage;
  const bool kept = cache && cache->dev && cache->device == psi->device;
  const AdjLayout lo = adj_pack(T, kept ? nullptr : &stage);
  const size_t o_part = al(std::max<size_t>(1, pool.size()) * sizeof(cx<R>));
  const size_t o_rows = o_part + al(std::max<size_t>(1, size_t(nrows) * G) * sizeof(double));
  const size_t o_tab = o_rows + al(std::max(1, nrows) * sizeof(double));
  void* wb = nullptr;
  if (int e = state_work(psi, cache ? o_tab : o_tab + lo.bytes, &wb)) return e;
  char* d = static_cast<char*>(wb);
  char* tab = cache ? static_cast<char*>(cache->dev) : d + o_tab;
  hipStream_t st = psi->stream;
  int rc = QSV_OK;
  auto fin = [&](int r) {
    (void)hipStreamSynchronize(st);
    return r;
  };
  if (cache && !kept) {
    if (cache->dev) (void)hipFree(cache->dev);
    cache->dev = nullptr;
    if (hipMalloc(&cache->dev, lo.bytes) != hipSuccess) {
      (void)hipGetLastError();
      cache->dev = nullptr;
      return fail(QSV_ENOMEM, "sweep table allocation failed");
    }
    cache->device = -1;  // (until they are uploaded)
    tab = static_cast<char*>(cache->dev);
  }
  if ((!kept && hipMemcpyAsync(tab, stage.data(), lo.bytes, hipMemcpyHostToDevice, st) != hipSuccess) ||
      (!pool.empty() &&
       hipMemcpyAsync(d, pool.data(), pool.size() * sizeof(cx<R>), hipMemcpyHostToDevice, st) != hipSuccess))
    return fin(fail(QSV_EHIP, "tiled sweep table upload failed"));
  if (cache && !kept) cache->device = psi->device;
  double* part = reinterpret_cast<double*>(d + o_part);
  hipLaunchKernelGGL(k_zero_doubles, dim3(256), dim3(256), 0, st, part, uint64_t(nrows) * G);
  {
    if (reg) {
      for (size_t pi = 0; pi < hp.size(); ++pi) {
        ProfScope ps("adjoint", 4.0 * sizeof(cx<R>) * double(dim(n)), st);
        hipLaunchKernelGGL((adj_reg_fn<R>(n, L - T.thread_bits, T.thread_bits, hp[pi].general ? kmax : 0)), dim3(G),
                           dim3(nt), reg_lds, st, static_cast<R*>(psi->ptr), static_cast<R*>(lam->ptr),
                           reinterpret_cast<const TilePassDev*>(tab + lo.pass), int(pi),
                           reinterpret_cast<const RegSegDev*>(tab + lo.segs),
                           reinterpret_cast<const RegHeadDev*>(tab + lo.heads),
                           reinterpret_cast<const RegOpDev*>(tab + lo.rops),
                           reinterpret_cast<const TileOpDev*>(tab + lo.ops),
                           reinterpret_cast<const PhaseEntDev*>(tab + lo.ents), reinterpret_cast<const cx<R>*>(d),
                           reinterpret_cast<const int*>(tab + lo.prow), part, tiles, R(pi == 0 ? energy : 0.0),
                           R(pi + 1 == hp.size() ? energy : 0.0));
        if (hipGetLastError() != hipSuccess) return fin(fail(QSV_EHIP, "register sweep launch failed"));
      }
    }
  }
  if (!reg) {
    const size_t lds = 2 * (size_t(1) << L) * sizeof(cx<R>);
    for (const void* k : {reinterpret_cast<const void*>(&k_tile_adj<R, 2>),
                          reinterpret_cast<const void*>(&k_tile_adj<R, 3>),
                          reinterpret_cast<const void*>(&k_tile_adj<R, 5>)})
      if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
        return fin(fail(QSV_EHIP, "cannot raise LDS limit of the tiled sweep"));
    for (size_t pi = 0; pi < hp.size(); ++pi) {
      ProfScope ps("adjoint", 4.0 * sizeof(cx<R>) * double(dim(n)), st);
#define QSV_ADJ_LAUNCH(KM)                                                                       \
    hipLaunchKernelGGL((k_tile_adj<R, KM>), dim3(G), dim3(kAdjTileThreads), lds, st,               \
                       static_cast<R*>(psi->ptr), static_cast<R*>(lam->ptr),                      \
                       reinterpret_cast<const TilePassDev*>(tab + lo.pass), int(pi),                          \
                       reinterpret_cast<const TileOpDev*>(tab + lo.ops),                             \
                       reinterpret_cast<const cx<R>*>(d), part, tiles)
      if (kmax <= 2) QSV_ADJ_LAUNCH(2);
      else if (kmax <= 3) QSV_ADJ_LAUNCH(3);
      else QSV_ADJ_LAUNCH(5);
#undef QSV_ADJ_LAUNCH
      if (hipGetLastError() != hipSuccess) return fin(fail(QSV_EHIP, "tiled sweep launch failed"));
    }
  }
  rows.assign(nrows, 0.0);
  if (nrows > 0) {
    hipLaunchKernelGGL(k_rows_sum, dim3(nrows), dim3(kAdjTileThreads), 0, st, part, G,
                       reinterpret_cast<double*>(d + o_rows));
    if (hipMemcpyAsync(rows.data(), d + o_rows, nrows * sizeof(double), hipMemcpyDeviceToHost, st) !=
        hipSuccess)
      return fin(fail(QSV_EHIP, "gradient download failed"));
  }
  return fin(rc);
}

template int adjoint_backward_tiled<float>(const AdjTables&, std::vector<cd>&, AdjCache*, int, double, qsv_state*,
                                           qsv_state*, std::vector<double>&);
template int adjoint_backward_tiled<double>(const AdjTables&, std::vector<cd>&, AdjCache*, int, double, qsv_state*,
                                            qsv_state*, std::vector<double>&);

}  // namespace qsv

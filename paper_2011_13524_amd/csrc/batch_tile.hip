// Batch items of at least 12 qubits as register tile passes over all items at
// once. Round k of a sweep is one launch that runs the k-th pass of every item,
// one workgroup per tile: the largest items no longer wait on one workgroup
// each, and the tiles of small and large items fill the chip together. The
// parameters reach the kernels as each item's pool of pass tables, which two
// small kernels form on the device from the uploaded theta. 256 items of 12 to
// 18 qubits, 8 layers, complex64: 92 ms with one workgroup per item (the
// 18-qubit items' serial chain), 3.05 ms here, of which the reverse passes 2.2
// ms, the forward passes 0.63 ms and H psi 0.32 ms.
#include <algorithm>
#include <cmath>

#include "adj_reg.h"
#include "batch_tile.h"
#include "plan.h"
#include "tile_reg.h"
#include "wave_sum.h"

namespace qsv {

// Workgroups of one item's pass, at most (a full chip of them): beyond, each
// takes several tiles and the partials stay few.
constexpr uint32_t kItemWgs = 1024;
constexpr int kLamThreads = 256;
constexpr int kLamAmps = 4096;  // amplitudes per workgroup of the H psi kernel

struct MItem {
  uint64_t psi, lam;      // amplitude offsets of the item's states
  uint64_t pool[2];       // pool offsets, forward and reverse
  uint64_t part;          // partials of the reverse sweep: rows x cols
  int n, circ;
  int val[2];             // host-value offsets
  uint32_t ntiles[2], cols[2];
  int theta, grad, nparams;
  int grp_begin, grp_count;
  int index;
  int chunk0, nchunk;     // partials of the energy and the norm
  int unitary;            // the norm that rounding left is divided out
};

// A distinct circuit of the batch: where its tables start.
struct MCirc {
  int pass[2];
  int elem[2], nelem[2];  // pool elements
  int dyn[2], ndyn[2];
  int slot;               // slot_begin entries (nparams + 1)
};

struct MWork {
  int item;
  uint32_t g;
};

struct MRec {
  int type, dst, src;
  int comp, ncomp;
};

struct MGroup {
  uint64_t flip;
  int begin, count;
};

struct MArgs {
  const MItem* items;
  const MCirc* circs;
  const TilePassDev* passes;
  const TileOpDev* ops;
  const RegSegDev* segs;
  const RegOpDev* rops;
  const RegHeadDev* heads;
  const PhaseEntDev* ents;
  const int* prow;
  const MRec* recs;
  const TabComp* comps;
  const int* elem_rec;    // pool element -> record (-1: spare)
  const DynVal* dyn;
  const int* slot_begin;  // rows of each parameter slot
  const int* slot_rows;
  const int* param_item;  // item of each gradient entry (of this path's items)
  const int* param_slot;
  const MGroup* groups;
  const GTerm* terms;
};

// ------------------------------------------------------------------ values

// Host values that follow the parameters, as the host forms them for a single
// circuit. One thread per value.
__global__ void __launch_bounds__(256) k_item_vals(MArgs a, const double* __restrict__ theta, cx<double>* __restrict__ vals) {
  const MItem& I = a.items[blockIdx.y >> 1];
  const int dir = int(blockIdx.y & 1);
  const MCirc& C = a.circs[I.circ];
  const int i = int(blockIdx.x * 256 + threadIdx.x);
  if (i >= C.ndyn[dir]) return;
  const DynVal d = a.dyn[C.dyn[dir] + i];
  cx<double>* v = vals + I.val[dir] + d.voff;
  const double t = d.sgn * theta[I.theta + d.slot];
  if (d.type == 0) {
    double s, c, sg = 1.0;
    sincos(0.5 * t, &s, &c);
    if (c < 0.0) {
      s = -s;
      c = -c;
      sg = -1.0;
    }
    v[0] = {s / (1.0 + c), -s};
    v[1] = {sg, 0.0};
  } else {
    double s, c;
    sincos(0.5 * t, &s, &c);
    v[0] = {c, s};
    if (d.type == 1) v[1] = {c, -s};
  }
}

__device__ __forceinline__ cx<double> zmul(cx<double> a, cx<double> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

// The pools (assemble_pool on the device): one thread per element, so that a run
// uploads theta (0.3 MB for 256 items of 12 to 18 qubits) and not the pools (44
// us for that batch).
template <typename R>
__global__ void __launch_bounds__(256) k_item_pool(MArgs a, const cx<double>* __restrict__ vals, cx<R>* __restrict__ pool) {
  const MItem& I = a.items[blockIdx.y >> 1];
  const int dir = int(blockIdx.y & 1);
  const MCirc& C = a.circs[I.circ];
  const int e = int(blockIdx.x * 256 + threadIdx.x);
  if (e >= C.nelem[dir]) return;
  const int ri = a.elem_rec[C.elem[dir] + e];
  const cx<double>* v = vals + I.val[dir];
  cx<double> z{0, 0};
  if (ri >= 0) {
    const MRec r = a.recs[ri];
    const int i = e - r.dst;
    if (r.type == 0) {
      z = v[r.src + i];
    } else {
      z = {1, 0};
      for (int k = r.comp; k < r.comp + r.ncomp; ++k) {
        const TabComp c = a.comps[k];
        if (c.type == 0) {
          z = zmul(v[c.src + (i >> c.a & 1)], z);
        } else if (c.type == 1) {
          z = zmul(v[c.src + ((i >> c.a & 1) | (i >> c.b & 1) << 1)], z);
        } else if (c.type == 2) {
          if ((i >> c.a & 1) & (i >> c.b & 1)) z = {-z.re, -z.im};
        } else if (c.type == 3) {
          cx<double> f = v[c.src];
          if (c.rsg >> i & 1) f.im = -f.im;
          z = zmul(f, z);
        } else {
          const double f = v[c.src + 1].re;
          z = {f * z.re, f * z.im};
        }
      }
    }
  }
  pool[I.pool[dir] + uint64_t(e)] = {R(z.re), R(z.im)};
}

// ------------------------------------------------------------------ states

// |0...0> of every item (the items' psi are contiguous, in order).
template <typename R>
__global__ void __launch_bounds__(256) k_item_zero(cx<R>* __restrict__ states, uint64_t total) {
  float4* p = reinterpret_cast<float4*>(states);
  const uint64_t nv = total * sizeof(cx<R>) / sizeof(float4);
  for (uint64_t i = uint64_t(blockIdx.x) * 256 + threadIdx.x; i < nv; i += uint64_t(gridDim.x) * 256)
    p[i] = {0, 0, 0, 0};
}

template <typename R>
__global__ void __launch_bounds__(256) k_item_one(MArgs a, int nitems, cx<R>* __restrict__ states) {
  const int i = int(blockIdx.x * 256 + threadIdx.x);
  if (i < nitems) states[a.items[i].psi] = {R(1), R(0)};
}

// The tables come as pointers of their own that nothing else aliases, so that they
// are read through the scalar cache.
#define QSV_ITEM_TABLES                                                                                       \
  const MItem *__restrict__ items, const MCirc *__restrict__ circs, const TilePassDev *__restrict__ passes,   \
      const RegSegDev *__restrict__ segs, const RegHeadDev *__restrict__ heads, const RegOpDev *__restrict__ rops, \
      const TileOpDev *__restrict__ ops, const PhaseEntDev *__restrict__ ents, const MWork *__restrict__ work, int round
template <typename R, int KMAX>
__global__ void __launch_bounds__(1 << kRegThreadBits, (tile_waves_per_simd<R, 4>()))
    k_item_tile(QSV_ITEM_TABLES, cx<R>* __restrict__ states, const cx<R>* __restrict__ pool) {
  extern __shared__ __align__(16) char smem[];
  const MWork w = work[blockIdx.x];
  const MItem& I = items[w.item];
  tile_pass<R, 4, KMAX, kRegThreadBits>(reinterpret_cast<R*>(states + I.psi), passes[circs[I.circ].pass[0] + round], w.g,
                                        I.cols[0], I.ntiles[0], 0u, segs, heads, rops, ops, ents, pool + I.pool[0], smem);
}

template <typename R, int KMAX>
__global__ void __launch_bounds__(1 << kRegThreadBits)
    k_item_adj(QSV_ITEM_TABLES, cx<R>* __restrict__ states, const cx<R>* __restrict__ pool, const int* __restrict__ prow,
               double* __restrict__ part, const double* __restrict__ energies) {
  extern __shared__ __align__(16) char smem[];
  const MWork w = work[blockIdx.x];
  const MItem& I = items[w.item];
  const uint64_t per = I.ntiles[1] / I.cols[1];  // (both powers of two)
  adj_pass<R, double, sizeof(R) == 4 ? 4 : 3, KMAX, kRegThreadBits>(
      reinterpret_cast<R*>(states + I.psi), reinterpret_cast<R*>(states + I.lam), passes[circs[I.circ].pass[1] + round],
      w.g * per, (w.g + 1) * per, segs, heads, rops, ops, ents, pool + I.pool[1], prow, part + I.part, I.cols[1], w.g,
      round == 0 ? R(energies[I.index]) : R(0), R(0), smem);
}
#undef QSV_ITEM_TABLES

// lambda = H psi on kLamAmps amplitudes per workgroup, with the energy's
// partial. Per group of equal flip mask, a term's sign is the parity of (x & z):
// the thread's part is formed once per term, the part of a thread's 16
// amplitudes (256 apart) is uniform. FP64 throughout. The partners come from the
// caches: bound by their rate (19 groups at 18 qubits, 319 us for 19 M amplitudes).
template <typename R>
__global__ void __launch_bounds__(kLamThreads) k_item_lam(MArgs a, const MWork* __restrict__ work, cx<R>* __restrict__ states,
                                                          double* __restrict__ epart) {
  __shared__ double red[2][kLamThreads / 64];
  constexpr int J = 8;
  const MWork w = work[blockIdx.x];
  const MItem& I = a.items[w.item];
  const cx<R>* __restrict__ psi = states + I.psi;
  cx<R>* __restrict__ lam = states + I.lam;
  double e = 0.0, nn = 0.0;
  for (int h = 0; h < kLamAmps / (J * kLamThreads); ++h) {
    const uint32_t base = w.g * kLamAmps + uint32_t(h) * (J * kLamThreads);
    const uint32_t y = base | threadIdx.x;
    double ar[J] = {}, ai[J] = {};
    for (int gi = I.grp_begin; gi < I.grp_begin + I.grp_count; ++gi) {
      const MGroup G = a.groups[gi];
      const uint32_t flip = uint32_t(G.flip);
      cx<R> v[J];
#pragma unroll
      for (int j = 0; j < J; ++j) v[j] = psi[(y + j * kLamThreads) ^ flip];
      double cr[J] = {}, ci[J] = {};
      for (int k = G.begin; k < G.begin + G.count; ++k) {
        const GTerm t = a.terms[k];
        const uint32_t z = uint32_t(t.z);
        const uint32_t s0 = uint32_t(__popc((y ^ flip) & z)) << 31;
        const uint32_t zj = z / kLamThreads;  // bits of j
        if (t.im == 0.0) {
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const uint32_t s = s0 ^ (uint32_t(__popc(zj & j)) << 31);
            cr[j] += __hiloint2double(__double2hiint(t.re) ^ int(s), __double2loint(t.re));
          }
        } else {
#pragma unroll
          for (int j = 0; j < J; ++j) {
            const uint32_t s = s0 ^ (uint32_t(__popc(zj & j)) << 31);
            cr[j] += __hiloint2double(__double2hiint(t.re) ^ int(s), __double2loint(t.re));
            ci[j] += __hiloint2double(__double2hiint(t.im) ^ int(s), __double2loint(t.im));
          }
        }
      }
#pragma unroll
      for (int j = 0; j < J; ++j) {
        ar[j] += cr[j] * double(v[j].re) - ci[j] * double(v[j].im);
        ai[j] += cr[j] * double(v[j].im) + ci[j] * double(v[j].re);
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const cx<R> p = psi[y + j * kLamThreads], l{R(ar[j]), R(ai[j])};
      lam[y + j * kLamThreads] = l;
      e += double(p.re) * double(l.re) + double(p.im) * double(l.im);
      nn += double(p.re) * double(p.re) + double(p.im) * double(p.im);
    }
  }
  e = wave_sum_to_last(e);
  nn = wave_sum_to_last(nn);
  if ((threadIdx.x & 63) == 63) {
    red[0][threadIdx.x >> 6] = e;
    red[1][threadIdx.x >> 6] = nn;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
    for (int i = 0; i < kLamThreads / 64; ++i) s += red[threadIdx.x][i];
    epart[2 * (I.chunk0 + int(w.g)) + int(threadIdx.x)] = s;
  }
}

// One wavefront per sum, in a fixed order: the energy, and the norm that the
// gradients are divided by.
__global__ void __launch_bounds__(64) k_item_energy(MArgs a, const double* __restrict__ epart, double* __restrict__ energies,
                                                    double* __restrict__ norms) {
  const MItem& I = a.items[blockIdx.x];
  double s = 0.0, nn = 0.0;
  for (int i = int(threadIdx.x); i < I.nchunk; i += 64) {
    s += epart[2 * (I.chunk0 + i)];
    nn += epart[2 * (I.chunk0 + i) + 1];
  }
  s = wave_sum_to_last(s);
  nn = wave_sum_to_last(nn);
  if (threadIdx.x == 63) {
    const double d = I.unitary && nn > 0.0 && isfinite(nn) ? nn : 1.0;
    energies[I.index] = s / d;
    norms[blockIdx.x] = d;
  }
}

__global__ void __launch_bounds__(256) k_item_grads(MArgs a, int nparams, const double* __restrict__ part,
                                                    const double* __restrict__ norms, double* __restrict__ grads) {
  const int p = int(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (p >= nparams) return;
  const MItem& I = a.items[a.param_item[p]];
  const int slot = a.param_slot[p];
  const int* sb = a.slot_begin + a.circs[I.circ].slot + slot;
  const uint32_t cols = I.cols[1], lane = threadIdx.x & 63;
  double s = 0.0;
  for (int k = sb[0]; k < sb[1]; ++k) {
    const double* row = part + I.part + uint64_t(a.slot_rows[k]) * cols;
    for (uint32_t c = lane; c < cols; c += 64) s += row[c];
  }
  s = wave_sum_to_last(s);
  if (lane == 63) grads[I.grad + slot] = s / norms[a.param_item[p]];
}

// ------------------------------------------------------------------ host

struct BatchTiles {
  struct Launch {
    int dir, round;  // dir 2: H psi
    bool general;
    size_t work;
    unsigned count;
  };
  std::vector<Launch> launches;
  int nitems = 0, nparams = 0;
  unsigned val_blocks = 0, pool_blocks = 0;
  uint64_t psi_total = 0;
  MArgs args{};
  void* d_tables = nullptr;
  void* d_data = nullptr;  // states | pools | partials
  cx<double>* d_vals = nullptr;
  const MWork* d_work = nullptr;
  void *d_states = nullptr, *d_pool = nullptr;
  double *d_part = nullptr, *d_epart = nullptr, *d_norms = nullptr;
};

namespace {

// Host tables of all distinct circuits, one after the other.
struct Tables {
  std::vector<MCirc> circs;
  std::vector<TilePassDev> passes;
  std::vector<TileOpDev> ops;
  SegBuild sb;  // (recs unused)
  std::vector<int> prow;
  std::vector<MRec> recs;
  std::vector<TabComp> comps;
  std::vector<int> elem_rec;
  std::vector<DynVal> dyn;
  std::vector<int> slot_begin, slot_rows;
  // per circuit and direction
  struct Host {
    const qsv_circuit* c;
    int npass[2];
    std::vector<char> general[2];
    std::vector<cd> vals[2];
    int rows;
    int unitary;
  };
  std::vector<Host> host;

  void append(int dir, MCirc& C, Host& H, const std::vector<TilePassDev>& hp, const std::vector<TileOpDev>& ho,
              const SegBuild& b, const std::vector<int>& rows, const std::vector<DynVal>& dv) {
    C.pass[dir] = int(passes.size());
    H.npass[dir] = int(hp.size());
    const int op0 = int(ops.size()), seg0 = int(sb.segs.size()), rop0 = int(sb.rops.size()), ent0 = int(sb.ents.size()),
              row0 = int(prow.size()), rec0 = int(recs.size());
    for (TilePassDev p : hp) {
      H.general[dir].push_back(char(p.general != 0));
      p.op_begin += op0;
      p.seg_begin += seg0;
      p.rop_begin += rop0;
      p.ent_begin += ent0;
      p.row_begin += row0;
      passes.push_back(p);
    }
    ops.insert(ops.end(), ho.begin(), ho.end());
    for (RegSegDev s : b.segs) {
      s.op_begin += rop0;
      sb.segs.push_back(s);
    }
    for (RegOpDev r : b.rops) {
      r.ent_begin += ent0;
      r.row_begin += ent0;
      for (int h = 0; h < kRegMaxH; ++h) r.h_begin[h] += ent0;
      r.lop += op0;
      sb.rops.push_back(r);
    }
    sb.ents.insert(sb.ents.end(), b.ents.begin(), b.ents.end());
    prow.insert(prow.end(), rows.begin(), rows.end());
    C.elem[dir] = int(elem_rec.size());
    C.nelem[dir] = b.pool_elems + kPoolSpare;
    elem_rec.resize(elem_rec.size() + size_t(C.nelem[dir]), -1);
    for (size_t i = 0; i < b.recs.size(); ++i) {
      const PoolRec& r = b.recs[i];
      recs.push_back({r.type, r.dst, r.src, int(comps.size()), int(r.comps.size())});
      comps.insert(comps.end(), r.comps.begin(), r.comps.end());
      for (int k = 0; k < r.n; ++k) elem_rec[size_t(C.elem[dir] + r.dst + k)] = rec0 + int(i);
    }
    C.dyn[dir] = int(dyn.size());
    C.ndyn[dir] = int(dv.size());
    dyn.insert(dyn.end(), dv.begin(), dv.end());
  }
};

// Plans circuit c and appends it; false (nothing appended) if it has to be left.
template <typename R>
bool add_circuit(Tables& T, const qsv_circuit* c) {
  qsv_plan* p = nullptr;
  if (plan_unmerged(c, sizeof(R) == 4 ? QSV_C64 : QSV_C128, &p) != QSV_OK) {
    clear_error();
    return false;
  }
  AdjTables A;
  bool ok = p->reg_bits == 4 && p->kmax_dense <= 2 && !p->h_pass.empty();
  for (const TilePassDev& d : p->h_pass) ok = ok && d.seg_count > 0;
  if (ok && adjoint_tables<R>(c, nullptr, A) != QSV_OK) {
    clear_error();
    ok = false;
  }
  ok = ok && A.reg && A.thread_bits == kRegThreadBits && A.kmax <= 2;
  for (const TilePassDev& d : A.hp) ok = ok && d.seg_count > 0;
  if (ok) {
    MCirc C{};
    Tables::Host H{};
    H.c = c;
    H.unitary = circuit_unitary(c) ? 1 : 0;
    std::vector<DynVal> dv;
    plan_symbolic(p, H.vals[0], dv);
    T.append(0, C, H, p->h_pass, p->h_ops, p->sb, {}, dv);
    H.vals[1] = A.vals;
    T.append(1, C, H, A.hp, A.ho, A.sb, A.prow, A.dyn);
    H.rows = int(A.row_slot.size());
    C.slot = int(T.slot_begin.size());
    std::vector<std::vector<int>> rows(static_cast<size_t>(c->nparams));
    for (int r = 0; r < H.rows; ++r) rows[size_t(A.row_slot[size_t(r)])].push_back(r);
    T.slot_begin.push_back(int(T.slot_rows.size()));
    for (const auto& r : rows) {
      T.slot_rows.insert(T.slot_rows.end(), r.begin(), r.end());
      T.slot_begin.push_back(int(T.slot_rows.size()));
    }
    T.circs.push_back(C);
    T.host.push_back(std::move(H));
  }
  plan_free(p);
  return ok;
}

}  // namespace

bool batch_tiles_take(const qsv_circuit& c) {
  if (c.n < 12 || c.gates.empty()) return false;
  // a Pauli rotation with X or Y factors is a dense block, whose matrix the
  // pool kernel does not form
  for (const Gate& g : c.gates)
    if (g.kind == Gate::PAULI &&
        (g.targets.size() < 2 || std::any_of(g.paulis.begin(), g.paulis.end(), [](int p) { return p != 3; })))
      return false;
  return true;
}

template <typename R>
int batch_tiles_build(const std::vector<BatchTileItem>& all, BatchTiles** out, std::vector<BatchTileItem>& left) {
  *out = nullptr;
  Tables T;
  std::vector<BatchTileItem> its;
  std::vector<int> circ_of;
  for (const BatchTileItem& it : all) {
    int ci = -1;
    for (size_t k = 0; k < T.host.size() && ci < 0; ++k)
      if (same_circuit(*T.host[k].c, *it.c)) ci = int(k);
    if (ci < 0 && add_circuit<R>(T, it.c)) ci = int(T.host.size()) - 1;
    if (ci < 0) {
      left.push_back(it);
      continue;
    }
    its.push_back(it);
    circ_of.push_back(ci);
  }
  if (its.empty()) return QSV_OK;
  std::vector<MItem> items;
  std::vector<MGroup> groups;
  std::vector<GTerm> terms;
  std::vector<cd> vals;
  std::vector<int> param_item, param_slot;
  uint64_t psi_total = 0, pool_total = 0, part_total = 0;
  int chunks = 0;
  BatchTiles* t = new (std::nothrow) BatchTiles();
  if (!t) return fail(QSV_ENOMEM, "host allocation failed");
  for (size_t i = 0; i < its.size(); ++i) psi_total += dim(its[i].c->n);
  uint64_t off = 0;
  for (size_t i = 0; i < its.size(); ++i) {
    const BatchTileItem& it = its[i];
    const MCirc& C = T.circs[size_t(circ_of[i])];
    const Tables::Host& H = T.host[size_t(circ_of[i])];
    MItem I{};
    I.n = it.c->n;
    I.circ = circ_of[i];
    I.psi = off;
    I.lam = psi_total + off;
    off += dim(I.n);
    for (int dir = 0; dir < 2; ++dir) {
      I.pool[dir] = pool_total;
      pool_total += uint64_t(C.nelem[dir]);
      I.val[dir] = int(vals.size());
      vals.insert(vals.end(), H.vals[dir].begin(), H.vals[dir].end());
      const int L = dir == 1 && sizeof(R) == 8 ? 11 : 12;
      I.ntiles[dir] = uint32_t(dim(I.n - L));
      I.cols[dir] = std::min(I.ntiles[dir], kItemWgs);
      t->val_blocks = std::max(t->val_blocks, unsigned(C.ndyn[dir] + 255) / 256);
      t->pool_blocks = std::max(t->pool_blocks, unsigned(C.nelem[dir] + 255) / 256);
    }
    I.part = part_total;
    part_total += uint64_t(H.rows) * I.cols[1];
    I.theta = it.theta_off;
    I.grad = it.grad_off;
    I.nparams = it.c->nparams;
    for (int s = 0; s < I.nparams; ++s) {
      param_item.push_back(int(i));
      param_slot.push_back(s);
    }
    std::vector<Group> gs;
    std::vector<GTerm> ts;
    build_groups(it.o, gs, ts);
    I.grp_begin = int(groups.size());
    I.grp_count = int(gs.size());
    for (const Group& g : gs) groups.push_back({g.flip, g.begin + int(terms.size()), g.count});
    terms.insert(terms.end(), ts.begin(), ts.end());
    I.index = it.index;
    I.unitary = H.unitary;
    I.chunk0 = chunks;
    I.nchunk = int(dim(I.n) / kLamAmps);
    chunks += I.nchunk;
    items.push_back(I);
  }
  // launches: one per round of each direction and kernel variant
  std::vector<MWork> work;
  auto launch = [&](int dir, int round, bool general) {
    const size_t w0 = work.size();
    for (size_t i = 0; i < its.size(); ++i) {
      if (dir < 2) {
        const Tables::Host& H = T.host[size_t(circ_of[i])];
        if (round >= H.npass[dir] || (H.general[dir][size_t(round)] != 0) != general) continue;
      }
      const uint32_t n = dir < 2 ? items[i].cols[dir] : uint32_t(items[i].nchunk);
      for (uint32_t g = 0; g < n; ++g) work.push_back({int(i), g});
    }
    if (work.size() > w0) t->launches.push_back({dir, round, general, w0, unsigned(work.size() - w0)});
  };
  for (int dir = 0; dir < 2; ++dir) {
    int rounds = 0;
    for (const Tables::Host& H : T.host) rounds = std::max(rounds, H.npass[dir]);
    for (int k = 0; k < rounds; ++k)
      for (int g = 0; g < 2; ++g) launch(dir, k, g != 0);
    if (dir == 0) launch(2, 0, false);
  }
  const std::vector<RegHeadDev> heads = op_heads(T.sb);
  const std::vector<PhaseEntDev> ents = op_entries(T.sb);
  t->nitems = int(items.size());
  t->nparams = int(param_item.size());
  t->psi_total = psi_total;
  // one allocation for the tables, one for what the kernels write
  struct Part {
    const void* src;
    size_t bytes;
    const void** dst;
  };
  MArgs& a = t->args;
  const void* vals_p = nullptr;
#define QSV_PART(v, m) {(v).data(), (v).size() * sizeof((v)[0]), reinterpret_cast<const void**>(&(m))}
  const Part parts[] = {QSV_PART(items, a.items),         QSV_PART(T.circs, a.circs),
                        QSV_PART(T.passes, a.passes),     QSV_PART(T.ops, a.ops),
                        QSV_PART(T.sb.segs, a.segs),      QSV_PART(T.sb.rops, a.rops),
                        QSV_PART(heads, a.heads),         QSV_PART(ents, a.ents),
                        QSV_PART(T.prow, a.prow),         QSV_PART(T.recs, a.recs),
                        QSV_PART(T.comps, a.comps),       QSV_PART(T.elem_rec, a.elem_rec),
                        QSV_PART(T.dyn, a.dyn),           QSV_PART(T.slot_begin, a.slot_begin),
                        QSV_PART(T.slot_rows, a.slot_rows), QSV_PART(param_item, a.param_item),
                        QSV_PART(param_slot, a.param_slot), QSV_PART(groups, a.groups),
                        QSV_PART(terms, a.terms),         QSV_PART(work, t->d_work),
                        QSV_PART(vals, vals_p)};
#undef QSV_PART
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t total = 0;
  for (const Part& p : parts) total += al(p.bytes + 16);
  if (hipMalloc(&t->d_tables, total) != hipSuccess) {
    (void)hipGetLastError();
    t->d_tables = nullptr;
    batch_tiles_free(t);
    return fail(QSV_ENOMEM, "batch table allocation failed (%zu bytes)", total);
  }
  {
    std::vector<char> stage(total, 0);
    size_t o = 0;
    for (const Part& p : parts) {
      if (p.bytes) std::copy_n(static_cast<const char*>(p.src), p.bytes, stage.data() + o);
      *p.dst = static_cast<char*>(t->d_tables) + o;
      o += al(p.bytes + 16);
    }
    if (hipMemcpy(t->d_tables, stage.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
      batch_tiles_free(t);
      return fail(QSV_EHIP, "batch table upload failed");
    }
  }
  t->d_vals = static_cast<cx<double>*>(const_cast<void*>(vals_p));
  const size_t b_states = al(2 * psi_total * sizeof(cx<R>)), b_pool = al(pool_total * sizeof(cx<R>)),
               b_part = al((part_total + 1) * sizeof(double)), b_epart = al(2 * size_t(chunks) * sizeof(double)),
               b_norms = al(its.size() * sizeof(double));
  const size_t bytes = b_states + b_pool + b_part + b_epart + b_norms;
  if (hipMalloc(&t->d_data, bytes) != hipSuccess) {
    (void)hipGetLastError();
    t->d_data = nullptr;
    batch_tiles_free(t);
    return fail(QSV_ENOMEM, "batch state allocation failed (%zu bytes)", bytes);
  }
  char* d = static_cast<char*>(t->d_data);
  t->d_states = d;
  t->d_pool = d + b_states;
  t->d_part = reinterpret_cast<double*>(d + b_states + b_pool);
  t->d_epart = reinterpret_cast<double*>(d + b_states + b_pool + b_part);
  t->d_norms = reinterpret_cast<double*>(d + b_states + b_pool + b_part + b_epart);
  *out = t;
  return QSV_OK;
}

template <typename R>
int batch_tiles_launch(const BatchTiles* t, const double* theta, double* energies, double* grads, hipStream_t st) {
  const unsigned ni = unsigned(t->nitems);
  cx<R>* states = static_cast<cx<R>*>(t->d_states);
  cx<R>* pool = static_cast<cx<R>*>(t->d_pool);
  const unsigned nt = 1u << kRegThreadBits;
  const size_t lds_f = size_t(4096) * sizeof(cx<R>);
  const size_t lds_r = size_t(sizeof(R) == 4 ? 4096 : 2048) * sizeof(cx<R>) + size_t(kAdjMaxRows) * (nt / 64) * sizeof(double);
  // (grid y: 2 x items, at most 65535 -- larger batches in slices)
  for (unsigned i0 = 0; i0 < ni; i0 += 32767) {
    MArgs a = t->args;
    a.items += i0;
    const unsigned y = 2 * std::min(32767u, ni - i0);
    if (t->val_blocks)
      hipLaunchKernelGGL(k_item_vals, dim3(t->val_blocks, y), dim3(256), 0, st, a, theta, t->d_vals);
    hipLaunchKernelGGL((k_item_pool<R>), dim3(t->pool_blocks, y), dim3(256), 0, st, a, t->d_vals, pool);
  }
  hipLaunchKernelGGL((k_item_zero<R>), dim3(2048), dim3(256), 0, st, states, t->psi_total);
  hipLaunchKernelGGL((k_item_one<R>), dim3((ni + 255) / 256), dim3(256), 0, st, t->args, t->nitems, states);
  const MArgs& a = t->args;
  for (const BatchTiles::Launch& l : t->launches) {
    const MWork* w = t->d_work + l.work;
    const dim3 g(l.count);
    if (l.dir == 2) {
      hipLaunchKernelGGL((k_item_lam<R>), g, dim3(kLamThreads), 0, st, a, w, states, t->d_epart);
      hipLaunchKernelGGL(k_item_energy, dim3(ni), dim3(64), 0, st, a, t->d_epart, energies, t->d_norms);
    } else if (l.dir == 0) {
      const auto fn = l.general ? &k_item_tile<R, 2> : &k_item_tile<R, 0>;
      hipLaunchKernelGGL(fn, g, dim3(nt), lds_f, st, a.items, a.circs, a.passes, a.segs, a.heads, a.rops, a.ops, a.ents, w,
                         l.round, states, pool);
    } else {
      const auto fn = l.general ? &k_item_adj<R, 2> : &k_item_adj<R, 0>;
      hipLaunchKernelGGL(fn, g, dim3(nt), lds_r, st, a.items, a.circs, a.passes, a.segs, a.heads, a.rops, a.ops, a.ents, w,
                         l.round, states, pool, a.prow, t->d_part, energies);
    }
  }
  if (t->nparams)
    hipLaunchKernelGGL(k_item_grads, dim3(unsigned(t->nparams + 3) / 4), dim3(256), 0, st, t->args, t->nparams, t->d_part,
                       t->d_norms, grads);
  QSV_HIP_CHECK(hipGetLastError());
  return QSV_OK;
}

void batch_tiles_free(BatchTiles* t) {
  if (!t) return;
  if (t->d_tables) (void)hipFree(t->d_tables);
  if (t->d_data) (void)hipFree(t->d_data);
  delete t;
}

template int batch_tiles_build<float>(const std::vector<BatchTileItem>&, BatchTiles**, std::vector<BatchTileItem>&);
template int batch_tiles_build<double>(const std::vector<BatchTileItem>&, BatchTiles**, std::vector<BatchTileItem>&);
template int batch_tiles_launch<float>(const BatchTiles*, const double*, double*, double*, hipStream_t);
template int batch_tiles_launch<double>(const BatchTiles*, const double*, double*, double*, hipStream_t);

}  // namespace qsv

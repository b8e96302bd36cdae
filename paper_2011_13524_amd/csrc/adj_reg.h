// Register-resident reverse sweep (device code): shared by the single-circuit
// sweep and the batch.
#pragma once

#include "dev_common.h"
#include "plan.h"
#include "tile_reg.h"
#include "wave_sum.h"

namespace qsv {

// -Im of i^ph (sr + i si).
__device__ __forceinline__ double neg_im_phase(double sr, double si, int ph) {
  switch (ph & 3) {
    case 0: return -si;
    case 1: return -sr;
    case 2: return si;
    default: return sr;
  }
}

// ------------------------------------------------------------------ register-resident sweep
//
// The reverse sweep with both tiles (psi and lambda) register-resident, using
// the segment layouts of the forward tile passes: ops on register bits run on
// both states from registers, X / CNOT ops fold into the LDS re-maps (a
// permutation of indices, applied to both states), and a rotation's gradient
// term -Im<lambda|P|psi> is evaluated on the register pairs just before its
// uncompute. Per gradient op, each wavefront sums its share (fixed order) into
// its own LDS slot; workgroups are persistent over a contiguous range of tiles
// and write one FP64 partial per (row, workgroup) at the end of the pass.

// This thread's share of -Im<lambda|P|psi> for P = Y (YAX) or X on register bit
// P: v[0] is psi, v[1] lambda. Products and the thread's sum in G; the caller sums in
// FP64. G is FP64, but for complex64 states of at least 20 qubits alone (FP32
// products and 8-term sums, relative error <= 11 x 2^-24 of sum |lambda_x||psi_y|
// <= |lambda||psi|), where the passes are bound by their vector instructions.
template <typename R, typename G, int NR, int P, bool YAX>
__device__ __forceinline__ G grad_xy(const cx<R> (&v)[2][NR]) {
  G acc = G(0);
  if constexpr ((1 << P) < NR) {
#pragma unroll
    for (int g = 0; g < NR / 2; ++g) {
      const int i = ins1<P>(g), j = i | (1 << P);
      const cx<R> a0 = v[0][i], a1 = v[0][j], l0 = v[1][i], l1 = v[1][j];
      if constexpr (YAX)
        acc += fma(G(l0.re), G(a1.re), G(l0.im) * G(a1.im)) - fma(G(l1.re), G(a0.re), G(l1.im) * G(a0.im));
      else
        acc += fma(G(l0.im), G(a1.re), -(G(l0.re) * G(a1.im))) + fma(G(l1.im), G(a0.re), -(G(l1.re) * G(a0.im)));
    }
  }
  return acc;
}

// Adds the wavefront's sum of `acc` to the wavefront's slot of a gradient row.
template <int TB>
__device__ __forceinline__ void add_row(double acc, double* wslot, int row, uint32_t tau) {
  const double w = wave_sum_to_last(acc);
  if ((tau & 63) == 63) wslot[row * (1 << (TB - 6))] += w;
}

// The rotations of a kind-11 op with their gradients: per register bit, the
// gradient's share from both states, then the uncompute exp(-i t P/2) of both.
template <typename R, typename G, int RB, int TB, int P = 0>
__device__ __forceinline__ void grad_layer(cx<R> (&v)[2][1 << RB], uint32_t rot, const RegOpDev& op,
                                           const cx<R>* __restrict__ coef, double* wslot, uint32_t tau) {
  if constexpr (P < RB) {
    if (rot >> (16 + P) & 1u) {
      double acc;
      if (rot >> P & 1u) acc = double(grad_xy<R, G, 1 << RB, P, true>(v));
      else acc = double(grad_xy<R, G, 1 << RB, P, false>(v));
      add_row<TB>(acc, wslot, op.aux[P], tau);
    }
    const cx<R> c = coef[P];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if constexpr (RB == 3) rot8_bit<P>(v[s], c, rot);
      else rot16_bit<P>(v[s], c, rot);
    }
    grad_layer<R, G, RB, TB, P + 1>(v, rot, op, coef, wslot, tau);
  }
}

// Gradient rows of the Z rotations of a phase op: -Im<lambda|Z_q|psi> =
// -sum_x (-1)^(x_q) w_x, w_x = Im(conj(lambda_x) psi_x). Diagonal factors of
// modulus one leave w alone, so the rows of every rotation that waits in the
// op share one evaluation of w: its sums with the sign of each register bit
// (s[0..RB-1]) and without (s[RB]) come from one tree of additions (in G, as in
// grad_xy), and a row
// on a thread bit or a non-local qubit takes the plain sum with its sign.
template <typename R, typename G, int RB, int TB>
__device__ __forceinline__ void phase_rows(const cx<R> (&v)[2][1 << RB], const RegHeadDev& hd,
                                           const RegOpDev& op, const PhaseEntDev* __restrict__ ents, double* wslot, uint32_t tau,
                                           uint64_t base) {
  constexpr int NR = 1 << RB;
  G w[NR], s[RB + 1];
#pragma unroll
  for (int r = 0; r < NR; ++r) w[r] = fma(G(v[1][r].im), G(v[0][r].re), -(G(v[1][r].re) * G(v[0][r].im)));
#pragma unroll
  for (int b = RB - 1; b >= 0; --b) {
    G d = w[0] - w[1 << b];
#pragma unroll
    for (int r = 1; r < (1 << b); ++r) d += w[r] - w[r | (1 << b)];
    s[b] = d;
#pragma unroll
    for (int r = 0; r < (1 << b); ++r) w[r] += w[r | (1 << b)];
  }
  s[RB] = w[0];
  for (int e = op.row_begin; e < op.row_begin + hd.row_count; ++e) {
    const PhaseEntDev E = ents[e];
    G x = s[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) x = E.ra == b ? s[b] : x;
    add_row<TB>(double(sgn_xor(x, ph_par(tau, E.tm, base, E.gm) << 31)), wslot, E.moff, tau);
  }
}

// Re-map of one state's registers through LDS (write in the old layout with
// the folded map, read in the new one).
// close: a cross-wave re-map ends with a workgroup barrier (another state's
// re-map writes next); otherwise that barrier is left to the next LDS write.
template <typename R, int RB, int TB>
__device__ __forceinline__ void adj_remap(cx<R> (&v)[1 << RB], const LdsMap<R, RB>& mo,
                                          const LdsMap<R, RB>& mn, bool xw, bool close, char* smem) {
#pragma unroll
  for (int i = 0; i < (1 << RB); ++i) mo.put(smem, i, v[i]);
  if (xw) __syncthreads();
  else wave_sync();
#pragma unroll
  for (int i = 0; i < (1 << RB); ++i) v[i] = mn.get(smem, i);
  if (!xw) wave_sync();
  else if (close) __syncthreads();
}

// A block applied through LDS to one state held in registers.
template <typename R, int RB, int TB, int KMAX, typename SW>
__device__ __forceinline__ void adj_lds_op(cx<R>* v, const LdsMap<R, RB>& ms, char* smem, const TileOpDev& op,
                                           const cx<R>* pool, int L, uint64_t base, SW sw) {
#pragma unroll
  for (int i = 0; i < (1 << RB); ++i) ms.put(smem, i, v[i]);
  __syncthreads();
  lds_op<R, KMAX>(reinterpret_cast<cx<R>*>(smem), op, pool, L, base, sw);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < (1 << RB); ++i) v[i] = ms.get(smem, i);
  __syncthreads();
}

// An op of the reverse sweep on both states, in place; gradient ops add this
// wavefront's share to its slot. Kind 11:
template <typename R, typename G, int RB, int TB>
__device__ __forceinline__ void adj_super(const RegHeadDev& hd, const RegOpDev& op, cx<R> (&v)[2][1 << RB],
                                          uint32_t tau, uint64_t base, const PhaseEntDev* __restrict__ ents,
                                          const cx<R>* __restrict__ pool, double* wslot) {
  if (hd.flags & 8u) phase_rows<R, G, RB, TB>(v, hd, op, ents, wslot, tau, base);
  phase_apply<R, RB, 2>(v, hd, op, ents, pool, tau, base);
  grad_layer<R, G, RB, TB>(v, su(hd.rot), op, pool + hd.roff, wslot, tau);
  const uint64_t xm = exchange_mask(hd.xch, op, tau, base);
  exchange<R, RB>(v[0], su(hd.xch), xm);
  exchange<R, RB>(v[1], su(hd.xch), xm);
}

// and the others.
template <typename R, int RB, int KMAX, int TB>
__device__ __forceinline__ void adj_general(const RegHeadDev& hd, const RegOpDev& op, cx<R> (&v)[2][1 << RB], const RegSegDev& S,
                                            const ThrMask<TB>& tm, uint32_t tau, uint64_t base, Swz<sizeof(R) == 4 ? 5 : 4> sw, char* smem,
                                            const TileOpDev* __restrict__ lops, const cx<R>* __restrict__ pool, int L,
                                            double* wslot) {
  constexpr int NR = 1 << RB;
  const cx<R>* m = pool + hd.moff;
  int key = int(hd.xch);  // (dense products without controls need the head alone, see reg_general)
  uint32_t cm = 0, cv = 0;
  bool lane = true;
  cx<R> gtab[4];
  if (!(hd.flags & 1u)) {
    if ((base & op.gcm) != op.gcv) return;  // non-local controls: uniform per tile
    if (op.kind == 8) {
      // Pauli-string gradient: psi staged in LDS in this segment's layout; the
      // partner x ^ f of element i is at its address XOR pf_lds (the swizzle is
      // linear over XOR and the tile starts at LDS address 0)
      const LdsMap<R, RB> ms(S.get_reg, tm.map(0u, S.tcol) >> 16);
      __syncthreads();  // (a preceding cross-wave re-map's reads are done)
#pragma unroll
      for (int i = 0; i < NR; ++i) ms.put(smem, i, v[0][i]);
      __syncthreads();
      typedef R R2 __attribute__((ext_vector_type(2)));
      typedef __attribute__((address_space(3))) R2 lds_r2;
      const uint32_t tpar = uint32_t(__popc(tau & op.pz_thr) + __popcll(base & op.pz_glob)) & 1u;
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const R2 av = *reinterpret_cast<lds_r2*>(uintptr_t(reinterpret_cast<uintptr_t>(ms.at(smem, i)) ^ op.pf_lds));
        const cx<R> c = v[1][i];
        const double wr = double(c.re) * av.x + double(c.im) * av.y;
        const double wi = double(c.re) * av.y - double(c.im) * av.x;
        const bool neg = ((uint32_t(__popc(uint32_t(i) & op.pz_reg)) ^ tpar) & 1u) != 0;
        sr += neg ? -wr : wr;
        si += neg ? -wi : wi;
      }
      __syncthreads();  // every read done before the LDS tile is written again
      add_row<TB>(neg_im_phase(sr, si, op.pph), wslot, op.aux[0], tau);
      return;
    }
    if (op.kind == 3) {
      const LdsMap<R, RB> ms(S.get_reg, tm.map(0u, S.tcol) >> 16);
      __syncthreads();  // (a preceding cross-wave re-map's reads are done)
      adj_lds_op<R, RB, TB, KMAX>(v[0], ms, smem, lops[op.lop], pool, L, base, sw);
      adj_lds_op<R, RB, TB, KMAX>(v[1], ms, smem, lops[op.lop], pool, L, base, sw);
      return;
    }
    int a = op.p1, b = op.p2;
    if (op.kind == 2) diag_table<R>(op, m, tau, base, gtab, a, b);
    key = op.key;
    cm = op.ri_cm;
    cv = op.ri_cv;
    lane = (tau & op.ti_cm) == op.ti_cv;
  }
  reg_apply<R, NR>(v[0], key, m, gtab, cm, cv, lane);
  reg_apply<R, NR>(v[1], key, m, gtab, cm, cv, lane);
}

// One pass over the tiles [g0, gend) of one workgroup; its partial of row r goes
// to partial[row * cols + col]. KMAX 0: passes of kind-11 ops only.
// The sweep runs on lambda - E psi (e_in = E in the first pass, else 0; e_out = E
// in the last, else 0, puts it back): Im <psi|P|psi> = 0, so the gradient is the
// same, but a rounding drift phi of the phase between the two states no longer
// enters it as phi E <P>. Measured against FP64, 24 qubits, 960 rotations,
// complex64, four sets of angles: relative error of the gradient 0.7e-5 to 4.5e-5
// on lambda itself, 0.3e-5 to 0.5e-5 here.
template <typename R, typename G, int RB, int KMAX, int TB>
__device__ __forceinline__ void adj_pass(R* __restrict__ psi, R* __restrict__ lam, const TilePassDev& P, uint64_t g0,
                                         uint64_t gend, const RegSegDev* __restrict__ segs,
                                         const RegHeadDev* __restrict__ heads, const RegOpDev* __restrict__ rops,
                                         const TileOpDev* __restrict__ lops, const PhaseEntDev* __restrict__ ents,
                                         const cx<R>* __restrict__ pool, const int* __restrict__ prow,
                                         double* __restrict__ partial, uint64_t cols, uint64_t col, R e_in, R e_out, char* smem) {
  constexpr int NR = 1 << RB;
  constexpr int NW = 1 << (TB - 6);  // wavefronts per workgroup
  constexpr int SB = sizeof(R) == 4 ? 5 : 4;
  const Swz<SB> sw;
  // one dynamic LDS block: the tile (first, at LDS address 0, as the re-map
  // addressing requires) then the gradient slots [row][wave]
  const int L = P.L;
  double(*slot)[NW] = reinterpret_cast<double(*)[NW]>(smem + (size_t(1) << L) * sizeof(cx<R>));
  const uint32_t tau = threadIdx.x;
  const ThrMask<TB> tm(tau);
  const int wave = int(tau >> 6);
  for (int i = int(tau); i < kAdjMaxRows * NW; i += blockDim.x) slot[i / NW][i % NW] = 0.0;
  // tiles of this workgroup: a contiguous range (fixed order of its partial sums)
  uint64_t gmask = 0;
  for (int r = 0; r < P.nrun; ++r) gmask |= ((uint64_t(1) << P.rlen[r]) - 1) << P.rdst[r];
  uint64_t base = 0;
  for (int r = 0; r < P.nrun; ++r) base |= ((g0 >> P.rsrc[r]) & ((uint64_t(1) << P.rlen[r]) - 1)) << P.rdst[r];
  const RegSegDev* S0 = &segs[P.seg_begin];
  const RegSegDev* SL = &segs[P.seg_begin + P.seg_count - 1];
  // HBM address parts of the first and last layouts: per thread (fixed for
  // the kernel) and per register element (uniform columns)
  uint64_t th0 = 0, thL = 0;
#pragma unroll
  for (int k = 0; k < TB; ++k) {
    const uint64_t on = uint64_t(0) - ((tau >> k) & 1);
    th0 |= S0->gcol_t[k] & on;
    thL |= SL->gcol_t[k] & on;
  }
  auto addr = [&](const RegSegDev& s, uint64_t th, uint64_t bs, int i) -> uint64_t {
    uint64_t x = bs | th;
#pragma unroll
    for (int k = 0; k < RB; ++k)
      if ((i >> k) & 1) x |= s.gcol_r[k];
    return x;
  };
  cx<R> v[2][NR];  // psi, lambda
  for (uint64_t g = g0; g < gend; ++g) {
    if (g > g0) base = ((base | ~gmask) + 1) & gmask;
    // HBM -> registers in the first segment's layout
    if (sizeof(R) == 4 && S0->reg[0] == 0) {
#pragma unroll
      for (int i = 0; i < NR; i += 2) {
        const uint64_t x = addr(*S0, th0, base, i);
        AmpIO<R, 2>::load(psi, x, &v[0][i]);
        AmpIO<R, 2>::load(lam, x, &v[1][i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const uint64_t x = addr(*S0, th0, base, i);
        AmpIO<R, 1>::load(psi, x, &v[0][i]);
        AmpIO<R, 1>::load(lam, x, &v[1][i]);
      }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
      v[1][i] = {fma(-e_in, v[0][i].re, v[1][i].re), fma(-e_in, v[0][i].im, v[1][i].im)};
    __syncthreads();  // the previous tile's last LDS reads are done (and the slots cleared)
    const RegSegDev* S = S0;
    int oi = S0->op_begin;
    RegHeadDev next = heads[oi];  // the next op's head, read one op ahead
    for (int sgi = 0; sgi < P.seg_count; ++sgi) {
      const RegSegDev* Sn = &segs[P.seg_begin + sgi];
      if (sgi > 0) {
        // re-map both states through LDS (folded X / CNOT ops applied to both)
        const bool xw = (Sn->xwave & 1) != 0;
        const bool xpre = (Sn->xwave & 2) != 0;
        const uint32_t j = tm.map(Sn->tcst, Sn->tcol);
        const LdsMap<R, RB> mo(Sn->put_reg, j & 0xffffu);
        const LdsMap<R, RB> mn(Sn->get_reg, j >> 16);
        if (xpre) __syncthreads();
        adj_remap<R, RB, TB>(v[0], mo, mn, xw, true, smem);
        adj_remap<R, RB, TB>(v[1], mo, mn, xw, false, smem);
      }
      S = Sn;
      for (const int oe = S->op_begin + S->op_count; oi < oe;) {
        const RegHeadDev hd = next;
        const RegOpDev& op = rops[oi];
        next = heads[++oi];
        if constexpr (KMAX > 0) {
          if ((hd.flags >> 24) != 11) {
            adj_general<R, RB, KMAX, TB>(hd, op, v, *S, tm, tau, base, sw, smem, lops, pool, L, &slot[0][wave]);
            continue;
          }
        }
        adj_super<R, G, RB, TB>(hd, op, v, tau, base, ents, pool, &slot[0][wave]);
      }
    }
    if (P.scale_off >= 0) {  // the sign left by the pass's rotations, when no phase op took it
      const R f = pool[P.scale_off].re;
      if (f != R(1)) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int i = 0; i < NR; ++i) v[s][i] = {f * v[s][i].re, f * v[s][i].im};
      }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
      v[1][i] = {fma(e_out, v[0][i].re, v[1][i].re), fma(e_out, v[0][i].im, v[1][i].im)};
    // registers -> HBM in the last segment's layout
    if (sizeof(R) == 4 && SL->reg[0] == 0) {
#pragma unroll
      for (int i = 0; i < NR; i += 2) {
        const uint64_t x = addr(*SL, thL, base, i);
        AmpIO<R, 2>::store(psi, x, &v[0][i]);
        AmpIO<R, 2>::store(lam, x, &v[1][i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const uint64_t x = addr(*SL, thL, base, i);
        AmpIO<R, 1>::store(psi, x, &v[0][i]);
        AmpIO<R, 1>::store(lam, x, &v[1][i]);
      }
    }
  }
  __syncthreads();
  for (int r = int(tau); r < P.row_count; r += blockDim.x) {
    double sum = 0.0;
    for (int w = 0; w < NW; ++w) sum += slot[r][w];
    partial[size_t(prow[P.row_begin + r]) * cols + col] = sum;
  }
}

template <typename R, typename G, int RB, int KMAX, int TB>
__global__ void __launch_bounds__(1 << TB)
    k_adj_reg(R* __restrict__ psi, R* __restrict__ lam, const TilePassDev* __restrict__ passes, int pass_idx,
              const RegSegDev* __restrict__ segs, const RegHeadDev* __restrict__ heads,
              const RegOpDev* __restrict__ rops, const TileOpDev* __restrict__ lops,
              const PhaseEntDev* __restrict__ ents, const cx<R>* __restrict__ pool, const int* __restrict__ prow,
              double* __restrict__ partial, uint64_t ntiles, R e_in, R e_out) {
  extern __shared__ __align__(16) char smem[];
  const uint64_t per = (ntiles + gridDim.x - 1) / gridDim.x;
  const uint64_t g0 = uint64_t(blockIdx.x) * per;
  const uint64_t gend = g0 + per < ntiles ? g0 + per : ntiles;
  adj_pass<R, G, RB, KMAX, TB>(psi, lam, passes[pass_idx], g0, gend, segs, heads, rops, lops, ents, pool, prow, partial,
                            gridDim.x, blockIdx.x, e_in, e_out, smem);
}

}  // namespace qsv

// Register-resident tile pass (device code, included by plan.hip).
//
// The 2^L amplitudes of a tile are spread over 2^TB threads, 2^RB per thread
// in VGPRs (RB = L - TB). A segment's layout says which local bits index a
// thread's registers (reg[0..RB-1]) and which index the thread (thr[0..TB-1]).
// Ops of a segment act on register bits. One-qubit unitaries come as rotations
// between diagonals, and every diagonal that is due at one point of the pass
// as one phase (phase_apply), wherever its qubits are; other blocks run as
// general products (reg_general). Between segments the tile is re-mapped through LDS
// (write in the old layout, barrier, read in the new one). LDS addresses are
// XOR-swizzled so that lanes whose local indices differ only in high bits do
// not collide on a bank. The first and last segments keep local bit 0 in
// registers (complex64), so HBM is read and written with 16-byte vectors and
// the low local bits index consecutive lanes (contiguous runs).
#pragma once

#include "dev_common.h"
#include "plan.h"

namespace qsv {

// LDS index swizzle: XOR the low SB bits with two higher SB-bit fields.
template <int SB>
struct Swz {
  __device__ __forceinline__ uint32_t operator()(uint32_t j) const {
    constexpr uint32_t m = (1u << SB) - 1;
    return j ^ ((j >> SB) & m) ^ ((j >> (2 * SB)) & m);
  }
};

struct NoSwz {
  __device__ __forceinline__ uint32_t operator()(uint32_t j) const { return j; }
};

__device__ __forceinline__ uint32_t insert_zeros32(uint32_t i, const int* pos, int m) {
  for (int j = 0; j < m; ++j) {
    const uint32_t lo = i & ((1u << pos[j]) - 1);
    i = ((i >> pos[j]) << (pos[j] + 1)) | lo;
  }
  return i;
}

// Dense block on local targets, whole tile in LDS (addresses through sw).
template <typename R, int K, typename SW>
__device__ __forceinline__ void lds_dense(cx<R>* __restrict__ t, const TileOpDev& op,
                                          const cx<R>* __restrict__ mat, int L, SW sw) {
  constexpr int D = 1 << K;
  const int cnt = 1 << (L - op.m);
  for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
    const uint32_t j0 = insert_zeros32(i, op.ins, op.m) | op.lcv;
    cx<R> v[D];
#pragma unroll
    for (int c = 0; c < D; ++c) v[c] = t[sw(j0 + op.off[c])];
#pragma unroll
    for (int r = 0; r < D; ++r) {
      cx<R> acc = {R(0), R(0)};
#pragma unroll
      for (int c = 0; c < D; ++c) acc = cfma(mat[r * D + c], v[c], acc);
      t[sw(j0 + op.off[r])] = acc;
    }
  }
}

template <typename R, typename SW>
__device__ __forceinline__ void lds_diag(cx<R>* __restrict__ t, const TileOpDev& op,
                                         const cx<R>* __restrict__ d, int L, uint64_t base, SW sw) {
  int gidx = 0;
  for (int b = 0; b < op.k; ++b)
    if (op.gq[b] >= 0) gidx |= int((base >> op.gq[b]) & 1) << b;
  const int TS = 1 << L;
  for (int j = threadIdx.x; j < TS; j += blockDim.x) {
    if ((uint32_t(j) & op.lcm) != op.lcv) continue;
    int idx = gidx;
    for (int b = 0; b < op.k; ++b)
      if (op.lt[b] >= 0) idx |= ((j >> op.lt[b]) & 1) << b;
    const uint32_t a = sw(uint32_t(j));
    t[a] = d[idx] * t[a];
  }
}

// KMAX bounds the widest dense block compiled in: a kernel instantiated for
// small blocks does not pay the register cost of 32-amplitude temporaries.
template <typename R, int KMAX, typename SW>
__device__ __forceinline__ void lds_op(cx<R>* t, const TileOpDev& op, const cx<R>* pool, int L,
                                       uint64_t base, SW sw) {
  const cx<R>* mat = pool + op.moff;
  if (op.kind == 1) {
    lds_diag<R>(t, op, mat, L, base, sw);
  } else {
    switch (op.k) {
      case 1: lds_dense<R, 1>(t, op, mat, L, sw); break;
      case 2: if constexpr (KMAX >= 2) lds_dense<R, 2>(t, op, mat, L, sw); break;
      case 3: if constexpr (KMAX >= 3) lds_dense<R, 3>(t, op, mat, L, sw); break;
      case 4: if constexpr (KMAX >= 4) lds_dense<R, 4>(t, op, mat, L, sw); break;
      default: if constexpr (KMAX >= 5) lds_dense<R, 5>(t, op, mat, L, sw); break;
    }
  }
}

// ------------------------------------------------------------------ register ops
//
// Register element indices are compile-time constants in every loop below
// (loops run over the compressed index g and insert the target bits), so the
// per-thread amplitude array stays in VGPRs.

// Component-wise select: a conditional choice between two complex values
// written on the scalars keeps both in registers (a select of whole structs
// can become a select of their addresses, which pins the arrays in memory).
template <typename R>
__device__ __forceinline__ cx<R> csel(bool c, const cx<R>& a, const cx<R>& b) {
  return {c ? a.re : b.re, c ? a.im : b.im};
}

template <int P>
__device__ __forceinline__ constexpr int ins1(int g) {
  return ((g >> P) << (P + 1)) | (g & ((1 << P) - 1));
}

template <int A, int B>
__device__ __forceinline__ constexpr int ins2(int g) {
  constexpr int lo = A < B ? A : B, hi = A < B ? B : A;
  return ins1<hi>(ins1<lo>(g));
}

// General products, in place (kernels of passes that hold such ops only).
// Variants for a register bit that does not exist for NR elements do nothing
// (never selected). Controlled variants (HASC) take the per-element
// register-bit control (i & cm) == cv and the per-lane thread-bit control
// `lane`.
template <typename R, int NR, int P, bool HASC>
__device__ __forceinline__ void reg_dense1(cx<R>* v, const cx<R>* __restrict__ m, uint32_t cm, uint32_t cv,
                                           bool lane) {
  if constexpr ((1 << P) < NR) {
    const cx<R> m00 = m[0], m01 = m[1], m10 = m[2], m11 = m[3];
#pragma unroll
    for (int g = 0; g < NR / 2; ++g) {
      const int i = ins1<P>(g), j = i | (1 << P);
      const cx<R> a = v[i], b = v[j];
      const cx<R> na = cfma(m00, a, m01 * b), nb = cfma(m10, a, m11 * b);
      if constexpr (HASC) {
        const bool on = lane && (uint32_t(i) & cm) == cv;
        v[i] = csel(on, na, a);
        v[j] = csel(on, nb, b);
      } else {
        v[i] = na;
        v[j] = nb;
      }
    }
  }
}

// Matrix index bit 0 <-> register bit A, bit 1 <-> register bit B.
template <typename R, int NR, int A, int B, bool HASC>
__device__ __forceinline__ void reg_dense2(cx<R>* v, const cx<R>* __restrict__ m, uint32_t cm, uint32_t cv,
                                           bool lane) {
  if constexpr ((1 << A) < NR && (1 << B) < NR) {
    const cx<R> k0 = m[0], k1 = m[1], k2 = m[2], k3 = m[3], k4 = m[4], k5 = m[5], k6 = m[6],
                k7 = m[7], k8 = m[8], k9 = m[9], k10 = m[10], k11 = m[11], k12 = m[12],
                k13 = m[13], k14 = m[14], k15 = m[15];
#pragma unroll
    for (int g = 0; g < NR / 4; ++g) {
      const int i0 = ins2<A, B>(g);
      const int i1 = i0 | (1 << A), i2 = i0 | (1 << B), i3 = i0 | (1 << A) | (1 << B);
      const bool on = !HASC || (lane && (uint32_t(i0) & cm) == cv);
      const cx<R> x0 = v[i0], x1 = v[i1], x2 = v[i2], x3 = v[i3];
      const cx<R> y0 = cfma(k3, x3, cfma(k2, x2, cfma(k1, x1, k0 * x0)));
      const cx<R> y1 = cfma(k7, x3, cfma(k6, x2, cfma(k5, x1, k4 * x0)));
      const cx<R> y2 = cfma(k11, x3, cfma(k10, x2, cfma(k9, x1, k8 * x0)));
      const cx<R> y3 = cfma(k15, x3, cfma(k14, x2, cfma(k13, x1, k12 * x0)));
      v[i0] = csel(on, y0, x0);
      v[i1] = csel(on, y1, x1);
      v[i2] = csel(on, y2, x2);
      v[i3] = csel(on, y3, x3);
    }
  }
}

// Diagonal factor on up to two register bits (A < B; -1: absent): the factor
// of element i is g[(bit A of i) | (bit B of i) << 1], picked at compile time.
template <typename R, int NR, int A, int B, bool HASC>
__device__ __forceinline__ void reg_diag(cx<R>* v, const cx<R>* g, uint32_t cm, uint32_t cv, bool lane) {
  if constexpr ((A < 0 || (1 << A) < NR) && (B < 0 || (1 << B) < NR)) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int idx = (A >= 0 ? (i >> A) & 1 : 0) | (B >= 0 ? ((i >> B) & 1) << 1 : 0);
      const bool on = !HASC || (lane && (uint32_t(i) & cm) == cv);
      v[i] = csel(on, g[idx] * v[i], v[i]);
    }
  }
}

// One flat switch over (op type, control presence, register bits). Keys:
// reg_key().
#define QSV_C1(HC, P)                                                            \
  case (HC) * 8 + (P):                                                           \
    reg_dense1<R, NR, P, HC>(v, m, cm, cv, lane);                                \
    break;
#define QSV_C1P(HC) QSV_C1(HC, 0) QSV_C1(HC, 1) QSV_C1(HC, 2) QSV_C1(HC, 3)
#define QSV_C2(HC, A, B)                                                         \
  case 32 + (HC) * 64 + (A) * 8 + (B):                                           \
    reg_dense2<R, NR, A, B, HC>(v, m, cm, cv, lane);                             \
    break;
#define QSV_C2P4(HC)                                                             \
  QSV_C2(HC, 0, 1) QSV_C2(HC, 0, 2) QSV_C2(HC, 0, 3) QSV_C2(HC, 1, 0) QSV_C2(HC, 1, 2) \
  QSV_C2(HC, 1, 3) QSV_C2(HC, 2, 0) QSV_C2(HC, 2, 1) QSV_C2(HC, 2, 3) QSV_C2(HC, 3, 0) \
  QSV_C2(HC, 3, 1) QSV_C2(HC, 3, 2)
#define QSV_C2P5(HC)                                                             \
  QSV_C2(HC, 0, 4) QSV_C2(HC, 1, 4) QSV_C2(HC, 2, 4) QSV_C2(HC, 3, 4) QSV_C2(HC, 4, 0) \
  QSV_C2(HC, 4, 1) QSV_C2(HC, 4, 2) QSV_C2(HC, 4, 3)
#define QSV_CD(HC, A, B)                                                         \
  case 160 + (HC) * 64 + ((A) + 1) * 8 + ((B) + 1):                              \
    reg_diag<R, NR, A, B, HC>(v, g, cm, cv, lane);                               \
    break;
#define QSV_CDP4(HC)                                                             \
  QSV_CD(HC, -1, -1) QSV_CD(HC, 0, -1) QSV_CD(HC, 1, -1) QSV_CD(HC, 2, -1)         \
  QSV_CD(HC, 3, -1) QSV_CD(HC, 0, 1) QSV_CD(HC, 0, 2) QSV_CD(HC, 0, 3)             \
  QSV_CD(HC, 1, 2) QSV_CD(HC, 1, 3) QSV_CD(HC, 2, 3)
#define QSV_CDP5(HC)                                                             \
  QSV_CD(HC, 4, -1) QSV_CD(HC, 0, 4) QSV_CD(HC, 1, 4) QSV_CD(HC, 2, 4) QSV_CD(HC, 3, 4)

// kind 0 dense one-qubit, 1 dense two-qubit, 2 diagonal; a, b: register bits (diagonal: -1 when absent, a < b)
__host__ __device__ __forceinline__ int reg_key(int kind, int a, int b, bool hc) {
  const int h = hc ? 1 : 0;
  if (kind == 1) return 32 + h * 64 + a * 8 + b;
  if (kind == 2) return 160 + h * 64 + (a + 1) * 8 + (b + 1);
  return h * 8 + a;
}

template <typename R, int NR>
__device__ __forceinline__ void reg_apply(cx<R>* v, int key, const cx<R>* m, const cx<R>* g, uint32_t cm,
                                          uint32_t cv, bool lane) {
  switch (key) {
    QSV_C1P(0) QSV_C1P(1)
    QSV_C2P4(0) QSV_C2P4(1)
    QSV_CDP4(0) QSV_CDP4(1)
    default:
      if constexpr (NR > 16) {
        switch (key) {
          QSV_C1(0, 4) QSV_C1(1, 4)
          QSV_C2P5(0) QSV_C2P5(1)
          QSV_CDP5(0) QSV_CDP5(1)
          default:
            __builtin_unreachable();  // the planner emits only the keys above
        }
      } else {
        __builtin_unreachable();
      }
      break;
  }
}
#undef QSV_C1
#undef QSV_C1P
#undef QSV_C2
#undef QSV_C2P4
#undef QSV_C2P5
#undef QSV_CD
#undef QSV_CDP4
#undef QSV_CDP5

// ------------------------------------------------------------------ phases, rotations, exchanges
//
// The parts of a kind-11 op run on the register array in place, as blocks of
// assembly with tied operands that branch over what the op does not have. So
// the op loop is straight-line code to the compiler: with branches between the
// parts in the source, or results in fresh registers, the compiler keeps the
// array in two places and copies it at the joins (32 to 64 moves per op beside
// the 48 FMAs of a rotation and the 64 products of a table). Few, large blocks:
// a taken branch costs a wavefront more than the instructions it skips; a block
// first tests whether there is anything to do in it.
// Uniform factors sit in scalar registers, one per instruction.
//
// Operands: the components of elements 0 .. 15 (or 0 .. 7) are %0 .. %31, the
// rest are named. Lists of the components of the first and second members of
// register bit P's pairs, 8 at a time (elements 0 .. 7 in QSV_A<P>, QSV_B<P>
// for P < 3):
#define QSV_A0 0, 1, 4, 5, 8, 9, 12, 13
#define QSV_B0 2, 3, 6, 7, 10, 11, 14, 15
#define QSV_C0 16, 17, 20, 21, 24, 25, 28, 29
#define QSV_D0 18, 19, 22, 23, 26, 27, 30, 31
#define QSV_A1 0, 1, 2, 3, 8, 9, 10, 11
#define QSV_B1 4, 5, 6, 7, 12, 13, 14, 15
#define QSV_C1 16, 17, 18, 19, 24, 25, 26, 27
#define QSV_D1 20, 21, 22, 23, 28, 29, 30, 31
#define QSV_A2 0, 1, 2, 3, 4, 5, 6, 7
#define QSV_B2 8, 9, 10, 11, 12, 13, 14, 15
#define QSV_C2 16, 17, 18, 19, 20, 21, 22, 23
#define QSV_D2 24, 25, 26, 27, 28, 29, 30, 31
#define QSV_A3 0, 1, 2, 3, 4, 5, 6, 7
#define QSV_B3 16, 17, 18, 19, 20, 21, 22, 23
#define QSV_C3 8, 9, 10, 11, 12, 13, 14, 15
#define QSV_D3 24, 25, 26, 27, 28, 29, 30, 31
#define QSV_X(K, ...) K(__VA_ARGS__)
#define QSV_E1(x) "+v"((x).re), "+v"((x).im)
#define QSV_E8(v) \
  QSV_E1(v[0]), QSV_E1(v[1]), QSV_E1(v[2]), QSV_E1(v[3]), QSV_E1(v[4]), QSV_E1(v[5]), QSV_E1(v[6]), QSV_E1(v[7])
#define QSV_E16(v) QSV_E8(v), QSV_E8((v + 8))
// skip to label L unless bit B of the uniform M is set
#define QSV_UNLESS(M, B, L) "s_bitcmp0_b32 %[" M "], " B "\n\ts_cbranch_scc1 " L "f\n\t"

// skip to label L if the uniform M is 0, or has none of the bits B (overwrites vcc_lo)
#define QSV_NONE(M, L) "s_cmp_eq_u32 %[" M "], 0\n\ts_cbranch_scc1 " L "f\n\t"
#define QSV_WITHOUT(M, B, L) "s_and_b32 vcc_lo, %[" M "], " B "\n\ts_cbranch_scc0 " L "f\n\t"

// Rotation by t/2 of two real components (x, y) as three shears, x += al y,
// y += be x, x += al y with al = tan(t/4), be = -sin(t/2) (|t/2| <= pi/2: both
// factors at most 1 in magnitude): three FMAs in place instead of two
// multiplies and two FMAs, and of determinant 1 however al and be are rounded.
// RY turns (Re a, Re b) and (Im a, Im b) of a pair of amplitudes, RX turns
// (Im a, Re b) and, the other way, (Re a, Im b): 6 FMAs per pair, where the
// general complex 2x2 product takes 16.
#define QSV_F32(D, A, B) "v_fmac_f32 %" #D ", %[" A "], %" #B "\n\t"
#define QSV_N32(D, A, B) "v_fma_f32 %" #D ", -%[" A "], %" #B ", %" #D "\n\t"
#define QSV_F64(D, A, B) "v_fma_f64 %" #D ", %[" A "], %" #B ", %" #D "\n\t"
#define QSV_N64(D, A, B) "v_fma_f64 %" #D ", -%[" A "], %" #B ", %" #D "\n\t"
// one shear of four pairs: Y, X onto the first members, X onto the second
#define QSV_SY(F, N, A, a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7) \
  F(a0, A, b0) F(a1, A, b1) F(a2, A, b2) F(a3, A, b3) F(a4, A, b4) F(a5, A, b5) F(a6, A, b6) F(a7, A, b7)
#define QSV_SX(F, N, A, a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7) \
  N(a0, A, b1) F(a1, A, b0) N(a2, A, b3) F(a3, A, b2) N(a4, A, b5) F(a5, A, b4) N(a6, A, b7) F(a7, A, b6)
#define QSV_SZ(F, N, A, a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7) \
  F(a0, A, b1) N(a1, A, b0) F(a2, A, b3) N(a3, A, b2) F(a4, A, b5) N(a5, A, b4) F(a6, A, b7) N(a7, A, b6)
#define QSV_ROT16(F, N, P, L1, L2)                                                                         \
  QSV_UNLESS("m", #P, L1)                                                                                  \
  QSV_X(QSV_SY, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SY, F, N, "al" #P, QSV_C##P, QSV_D##P)         \
  QSV_X(QSV_SY, F, N, "be" #P, QSV_B##P, QSV_A##P) QSV_X(QSV_SY, F, N, "be" #P, QSV_D##P, QSV_C##P)         \
  QSV_X(QSV_SY, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SY, F, N, "al" #P, QSV_C##P, QSV_D##P)         \
  "s_branch " L2 "f\n" L1 ":\n\t" QSV_UNLESS("m", "8+" #P, L2)                                             \
  QSV_X(QSV_SX, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SX, F, N, "al" #P, QSV_C##P, QSV_D##P)         \
  QSV_X(QSV_SZ, F, N, "be" #P, QSV_B##P, QSV_A##P) QSV_X(QSV_SZ, F, N, "be" #P, QSV_D##P, QSV_C##P)         \
  QSV_X(QSV_SX, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SX, F, N, "al" #P, QSV_C##P, QSV_D##P)         \
  L2 ":\n\t"
#define QSV_ROT8(F, N, P, L1, L2)                                                                          \
  QSV_UNLESS("m", #P, L1)                                                                                  \
  QSV_X(QSV_SY, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SY, F, N, "be" #P, QSV_B##P, QSV_A##P)         \
  QSV_X(QSV_SY, F, N, "al" #P, QSV_A##P, QSV_B##P)                                                         \
  "s_branch " L2 "f\n" L1 ":\n\t" QSV_UNLESS("m", "8+" #P, L2)                                             \
  QSV_X(QSV_SX, F, N, "al" #P, QSV_A##P, QSV_B##P) QSV_X(QSV_SZ, F, N, "be" #P, QSV_B##P, QSV_A##P)         \
  QSV_X(QSV_SX, F, N, "al" #P, QSV_A##P, QSV_B##P)                                                         \
  L2 ":\n\t"
#define QSV_AB(c, P) [al##P] "s"(c[P].re), [be##P] "s"(c[P].im)
#define QSV_ROTS(T, F, N)                                                                                  \
  /* rotations on bits 0 .. 3 of 16 elements: bit P of rot about Y, 8 + P about X, shears c[P] */          \
  __device__ __forceinline__ void rot16(cx<T>* v, const cx<T>* c, uint32_t rot) {                          \
    asm(QSV_NONE("m", "9") QSV_ROT16(F, N, 0, "1", "2") QSV_ROT16(F, N, 1, "3", "4")                        \
            QSV_ROT16(F, N, 2, "5", "6") QSV_ROT16(F, N, 3, "7", "8") "9:"                                 \
        : QSV_E16(v)                                                                                       \
        : QSV_AB(c, 0), QSV_AB(c, 1), QSV_AB(c, 2), QSV_AB(c, 3), [m] "s"(rot)                             \
        : "scc");                                                                                          \
  }                                                                                                        \
  /* bits 0 .. 2 of 8 elements */                                                                          \
  __device__ __forceinline__ void rot8(cx<T>* v, const cx<T>* c, uint32_t rot) {                           \
    asm(QSV_NONE("m", "9") QSV_ROT8(F, N, 0, "1", "2") QSV_ROT8(F, N, 1, "3", "4")                          \
            QSV_ROT8(F, N, 2, "5", "6") "9:"                                                               \
        : QSV_E8(v)                                                                                        \
        : QSV_AB(c, 0), QSV_AB(c, 1), QSV_AB(c, 2), [m] "s"(rot)                                           \
        : "scc");                                                                                          \
  }                                                                                                        \
  /* one bit of a 16- or 8-element array (the reverse sweep evaluates gradients between them) */           \
  template <int P>                                                                                         \
  __device__ __forceinline__ void rot16_bit(cx<T>* v, cx<T> f, uint32_t rot) {                             \
    const cx<T> c[4] = {f, f, f, f};                                                                       \
    if constexpr (P == 0) asm(QSV_ROT16(F, N, 0, "1", "2") : QSV_E16(v) : QSV_AB(c, 0), [m] "s"(rot) : "scc"); \
    if constexpr (P == 1) asm(QSV_ROT16(F, N, 1, "1", "2") : QSV_E16(v) : QSV_AB(c, 1), [m] "s"(rot) : "scc"); \
    if constexpr (P == 2) asm(QSV_ROT16(F, N, 2, "1", "2") : QSV_E16(v) : QSV_AB(c, 2), [m] "s"(rot) : "scc"); \
    if constexpr (P == 3) asm(QSV_ROT16(F, N, 3, "1", "2") : QSV_E16(v) : QSV_AB(c, 3), [m] "s"(rot) : "scc"); \
  }                                                                                                        \
  template <int P>                                                                                         \
  __device__ __forceinline__ void rot8_bit(cx<T>* v, cx<T> f, uint32_t rot) {                              \
    const cx<T> c[4] = {f, f, f, f};                                                                       \
    if constexpr (P == 0) asm(QSV_ROT8(F, N, 0, "1", "2") : QSV_E8(v) : QSV_AB(c, 0), [m] "s"(rot) : "scc"); \
    if constexpr (P == 1) asm(QSV_ROT8(F, N, 1, "1", "2") : QSV_E8(v) : QSV_AB(c, 1), [m] "s"(rot) : "scc"); \
    if constexpr (P == 2) asm(QSV_ROT8(F, N, 2, "1", "2") : QSV_E8(v) : QSV_AB(c, 2), [m] "s"(rot) : "scc"); \
  }                                                                                                        \
  /* pairs (a[k], b[k]), k = 0 .. 7: register bit 4 of 32 elements, half of them */                        \
  __device__ __forceinline__ void rot_pairs8(cx<T>* a, cx<T>* b, cx<T> f, uint32_t rot) {                  \
    const cx<T> c[4] = {f, f, f, f};                                                                       \
    asm(QSV_ROT16(F, N, 3, "1", "2")                                                                       \
        : QSV_E8(a), QSV_E8(b)                                                                             \
        : QSV_AB(c, 3), [m] "s"(rot)                                                                       \
        : "scc");                                                                                          \
  }
QSV_ROTS(float, QSV_F32, QSV_N32)
QSV_ROTS(double, QSV_F64, QSV_N64)

// x <- f x with one temporary: re' = fr re - fi im, im' = fr im + fi re; or by
// the conjugate of f.
#define QSV_CM(O, R_, I_, T_, FR, FI)                                                                       \
  "v_mul_" O " " T_ ", " FI ", %" R_ "\n\tv_mul_" O " %" R_ ", " FR ", %" R_ "\n\tv_fma_" O " %" R_ ", -" FI \
  ", %" I_ ", %" R_ "\n\tv_fma_" O " %" I_ ", " FR ", %" I_ ", " T_ "\n\t"
#define QSV_CJ(O, R_, I_, T_, FR, FI)                                                                       \
  "v_mul_" O " " T_ ", " FI ", %" R_ "\n\tv_mul_" O " %" R_ ", " FR ", %" R_ "\n\tv_fma_" O " %" R_ ", " FI  \
  ", %" I_ ", %" R_ "\n\tv_fma_" O " %" I_ ", " FR ", %" I_ ", -" T_ "\n\t"
// the factor of the thread
#define QSV_FC(O, R_, I_, T_) QSV_CM(O, R_, I_, T_, "%[cr]", "%[ci]")
#define QSV_FAC8(O, a0, a1, a2, a3, a4, a5, a6, a7, a8, a9, b0, b1, b2, b3, b4, b5)                          \
  QSV_FC(O, a0, a1, "%[t]") QSV_FC(O, a2, a3, "%[u]") QSV_FC(O, a4, a5, "%[t]") QSV_FC(O, a6, a7, "%[u]")     \
  QSV_FC(O, a8, a9, "%[t]") QSV_FC(O, b0, b1, "%[u]") QSV_FC(O, b2, b3, "%[t]") QSV_FC(O, b4, b5, "%[u]")
#define QSV_N8A "0", "1", "2", "3", "4", "5", "6", "7", "8", "9", "10", "11", "12", "13", "14", "15"
#define QSV_N8B "16", "17", "18", "19", "20", "21", "22", "23", "24", "25", "26", "27", "28", "29", "30", "31"
// a string pattern's factor, conjugated where the element's bit of the pattern is set
#define QSV_ST(O, H, K, R_, I_)                                                                             \
  "s_bitcmp1_b32 %[g" H "], " K "\n\ts_cbranch_scc1 8f\n\t" QSV_CM(O, R_, I_, "%[t]", "%[hr" H "]", "%[hi" H "]") \
  "s_branch 9f\n8:\n\t" QSV_CJ(O, R_, I_, "%[t]", "%[hr" H "]", "%[hi" H "]") "9:\n\t"
#define QSV_STR8(O, H)                                                                                      \
  QSV_ST(O, H, "0", "0", "1") QSV_ST(O, H, "1", "2", "3") QSV_ST(O, H, "2", "4", "5")                        \
  QSV_ST(O, H, "3", "6", "7") QSV_ST(O, H, "4", "8", "9") QSV_ST(O, H, "5", "10", "11")                      \
  QSV_ST(O, H, "6", "12", "13") QSV_ST(O, H, "7", "14", "15")
#define QSV_STR16(O, H)                                                                                     \
  QSV_STR8(O, H) QSV_ST(O, H, "8", "16", "17") QSV_ST(O, H, "9", "18", "19") QSV_ST(O, H, "10", "20", "21")  \
  QSV_ST(O, H, "11", "22", "23") QSV_ST(O, H, "12", "24", "25") QSV_ST(O, H, "13", "26", "27")               \
  QSV_ST(O, H, "14", "28", "29") QSV_ST(O, H, "15", "30", "31")
// the signs of register bit P's set elements
#define QSV_FL(OP, P, a0, a1, a2, a3, a4, a5, a6, a7)                                                       \
  OP " %" #a0 ", %[f" P "], %" #a0 "\n\t" OP " %" #a1 ", %[f" P "], %" #a1 "\n\t"                            \
  OP " %" #a2 ", %[f" P "], %" #a2 "\n\t" OP " %" #a3 ", %[f" P "], %" #a3 "\n\t"                            \
  OP " %" #a4 ", %[f" P "], %" #a4 "\n\t" OP " %" #a5 ", %[f" P "], %" #a5 "\n\t"                            \
  OP " %" #a6 ", %[f" P "], %" #a6 "\n\t" OP " %" #a7 ", %[f" P "], %" #a7 "\n\t"
#define QSV_LANE(T, M, O, OP)                                                                               \
  /* the parts of a phase that depend on the thread: factor C, signs f, string factors h (flags: */         \
  /* RegOpDev; bits 2, 256 << a, 16 << h) */                                                                \
  __device__ __forceinline__ void lane16(cx<T>* v, cx<T> C, const M* f, const cx<T>* h, uint32_t flags,     \
                                         const uint32_t* rsg) {                                             \
    T t, u;                                                                                                 \
    asm(QSV_WITHOUT("m", "0xfff2", "7") QSV_UNLESS("m", "1", "1")                                            \
        QSV_X(QSV_FAC8, O, QSV_N8A) QSV_X(QSV_FAC8, O, QSV_N8B) "1:\n\t"                                    \
        QSV_WITHOUT("m", "0xf00", "2") QSV_UNLESS("m", "8", "1")                                            \
        QSV_X(QSV_FL, OP, "0", QSV_B0) QSV_X(QSV_FL, OP, "0", QSV_D0) "1:\n\t" QSV_UNLESS("m", "9", "1")    \
        QSV_X(QSV_FL, OP, "1", QSV_B1) QSV_X(QSV_FL, OP, "1", QSV_D1) "1:\n\t" QSV_UNLESS("m", "10", "1")   \
        QSV_X(QSV_FL, OP, "2", QSV_B2) QSV_X(QSV_FL, OP, "2", QSV_D2) "1:\n\t" QSV_UNLESS("m", "11", "1")   \
        QSV_X(QSV_FL, OP, "3", QSV_B3) QSV_X(QSV_FL, OP, "3", QSV_D3) "1:\n2:\n\t"                         \
        QSV_UNLESS("m", "4", "7")                                                                           \
        QSV_STR16(O, "0") QSV_UNLESS("m", "5", "7") QSV_STR16(O, "1") QSV_UNLESS("m", "6", "7")             \
        QSV_STR16(O, "2") QSV_UNLESS("m", "7", "7") QSV_STR16(O, "3") "7:"                                  \
        : QSV_E16(v), [t] "=&v"(t), [u] "=&v"(u)                                                            \
        : [cr] "v"(C.re), [ci] "v"(C.im), [f0] "v"(f[0]), [f1] "v"(f[1]), [f2] "v"(f[2]), [f3] "v"(f[3]),   \
          [hr0] "v"(h[0].re), [hi0] "v"(h[0].im), [hr1] "v"(h[1].re), [hi1] "v"(h[1].im),                   \
          [hr2] "v"(h[2].re), [hi2] "v"(h[2].im), [hr3] "v"(h[3].re), [hi3] "v"(h[3].im), [m] "s"(flags),   \
          [g0] "s"(rsg[0]), [g1] "s"(rsg[1]), [g2] "s"(rsg[2]), [g3] "s"(rsg[3])                            \
        : "scc", "vcc");                                                                                    \
  }                                                                                                         \
  __device__ __forceinline__ void lane8(cx<T>* v, cx<T> C, const M* f, const cx<T>* h, uint32_t flags,      \
                                        const uint32_t* rsg) {                                              \
    T t, u;                                                                                                 \
    asm(QSV_WITHOUT("m", "0xfff2", "7") QSV_UNLESS("m", "1", "1")                                            \
        QSV_X(QSV_FAC8, O, QSV_N8A) "1:\n\t" QSV_WITHOUT("m", "0x700", "2") QSV_UNLESS("m", "8", "1")       \
        QSV_X(QSV_FL, OP, "0", QSV_B0) "1:\n\t" QSV_UNLESS("m", "9", "1")                                   \
        QSV_X(QSV_FL, OP, "1", QSV_B1) "1:\n\t" QSV_UNLESS("m", "10", "1")                                  \
        QSV_X(QSV_FL, OP, "2", QSV_B2) "1:\n2:\n\t" QSV_UNLESS("m", "4", "7")                              \
        QSV_STR8(O, "0") QSV_UNLESS("m", "5", "7") QSV_STR8(O, "1") QSV_UNLESS("m", "6", "7")               \
        QSV_STR8(O, "2") QSV_UNLESS("m", "7", "7") QSV_STR8(O, "3") "7:"                                    \
        : QSV_E8(v), [t] "=&v"(t), [u] "=&v"(u)                                                             \
        : [cr] "v"(C.re), [ci] "v"(C.im), [f0] "v"(f[0]), [f1] "v"(f[1]), [f2] "v"(f[2]),                   \
          [hr0] "v"(h[0].re), [hi0] "v"(h[0].im), [hr1] "v"(h[1].re), [hi1] "v"(h[1].im),                   \
          [hr2] "v"(h[2].re), [hi2] "v"(h[2].im), [hr3] "v"(h[3].re), [hi3] "v"(h[3].im), [m] "s"(flags),   \
          [g0] "s"(rsg[0]), [g1] "s"(rsg[1]), [g2] "s"(rsg[2]), [g3] "s"(rsg[3])                            \
        : "scc", "vcc");                                                                                    \
  }                                                                                                         \
  /* 8 elements times 8 uniform factors (flag 1) */                                                         \
  __device__ __forceinline__ void tab8(cx<T>* v, const cx<T>* f, uint32_t flags) {                          \
    T t, u;                                                                                                 \
    asm(QSV_UNLESS("m", "0", "1") QSV_CM(O, "0", "1", "%[t]", "%[a0]", "%[b0]")                             \
            QSV_CM(O, "2", "3", "%[u]", "%[a1]", "%[b1]") QSV_CM(O, "4", "5", "%[t]", "%[a2]", "%[b2]")      \
            QSV_CM(O, "6", "7", "%[u]", "%[a3]", "%[b3]") QSV_CM(O, "8", "9", "%[t]", "%[a4]", "%[b4]")      \
            QSV_CM(O, "10", "11", "%[u]", "%[a5]", "%[b5]") QSV_CM(O, "12", "13", "%[t]", "%[a6]", "%[b6]")  \
            QSV_CM(O, "14", "15", "%[u]", "%[a7]", "%[b7]") "1:"                                             \
        : QSV_E8(v), [t] "=&v"(t), [u] "=&v"(u)                                                             \
        : [a0] "s"(f[0].re), [b0] "s"(f[0].im), [a1] "s"(f[1].re), [b1] "s"(f[1].im), [a2] "s"(f[2].re),    \
          [b2] "s"(f[2].im), [a3] "s"(f[3].re), [b3] "s"(f[3].im), [a4] "s"(f[4].re), [b4] "s"(f[4].im),    \
          [a5] "s"(f[5].re), [b5] "s"(f[5].im), [a6] "s"(f[6].re), [b6] "s"(f[6].im), [a7] "s"(f[7].re),    \
          [b7] "s"(f[7].im), [m] "s"(flags)                                                                 \
        : "scc");                                                                                           \
  }
QSV_LANE(float, uint32_t, "f32", "v_xor_b32")
QSV_LANE(double, double, "f64", "v_mul_f64")
__device__ __forceinline__ uint32_t flip_arg(float, uint32_t par) { return par << 31; }
__device__ __forceinline__ double flip_arg(double, uint32_t par) { return par ? -1.0 : 1.0; }

// Exchange of the pairs of register bit P (bit P of xch) in the lanes of m; pair
// g (elements ins1<P>(g) and its partner) where bit 8 + g is set.
#define QSV_SW32(a, b, c, d) "v_swap_b32 %" #a ", %" #c "\n\tv_swap_b32 %" #b ", %" #d "\n\t"
#define QSV_MV64(a, c) "v_mov_b64 %[t], %" #a "\n\tv_mov_b64 %" #a ", %" #c "\n\tv_mov_b64 %" #c ", %[t]\n\t"
#define QSV_SW64(a, b, c, d) QSV_MV64(a, c) QSV_MV64(b, d)
#define QSV_XP(S, G, a0, a1, b0, b1) QSV_UNLESS("x", "8+" G, "2") S(a0, a1, b0, b1) "2:\n\t"
#define QSV_XC4(S, G0, G1, G2, G3, a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7)           \
  QSV_XP(S, G0, a0, a1, b0, b1) QSV_XP(S, G1, a2, a3, b2, b3) QSV_XP(S, G2, a4, a5, b4, b5)                  \
  QSV_XP(S, G3, a6, a7, b6, b7)
#define QSV_XB16(S, P)                                                                                      \
  QSV_UNLESS("x", #P, "3") QSV_X(QSV_XC4, S, "0", "1", "2", "3", QSV_A##P, QSV_B##P)                         \
  QSV_X(QSV_XC4, S, "4", "5", "6", "7", QSV_C##P, QSV_D##P) "3:\n\t"
#define QSV_XB8(S, P) \
  QSV_UNLESS("x", #P, "3") QSV_X(QSV_XC4, S, "0", "1", "2", "3", QSV_A##P, QSV_B##P) "3:\n\t"
#define QSV_XHEAD \
  "s_and_b32 vcc_lo, %[x], 15\n\ts_cbranch_scc0 7f\n\ts_mov_b64 vcc, exec\n\ts_and_b64 exec, exec, %[l]\n\t"
#define QSV_XCH(T, S)                                                                                       \
  __device__ __forceinline__ void xch16(cx<T>* v, uint64_t m, uint32_t xch) {                               \
    T t;                                                                                                    \
    asm(QSV_XHEAD QSV_XB16(S, 0) QSV_XB16(S, 1) QSV_XB16(S, 2) QSV_XB16(S, 3) "s_mov_b64 exec, vcc\n7:"      \
        : QSV_E16(v), [t] "=&v"(t)                                                                          \
        : [l] "s"(m), [x] "s"(xch)                                                                          \
        : "scc", "vcc");                                                                                    \
  }                                                                                                         \
  __device__ __forceinline__ void xch8(cx<T>* v, uint64_t m, uint32_t xch) {                                \
    T t;                                                                                                    \
    asm(QSV_XHEAD QSV_XB8(S, 0) QSV_XB8(S, 1) QSV_XB8(S, 2) "s_mov_b64 exec, vcc\n7:"                        \
        : QSV_E8(v), [t] "=&v"(t)                                                                           \
        : [l] "s"(m), [x] "s"(xch)                                                                          \
        : "scc", "vcc");                                                                                    \
  }                                                                                                         \
  /* the pairs (a[k], b[k]): register bit 4 of 32 elements, half of them (bit 3 of x) */                    \
  __device__ __forceinline__ void xch_pairs8(cx<T>* a, cx<T>* b, uint64_t m, uint32_t xch) {                \
    T t;                                                                                                    \
    asm(QSV_XHEAD QSV_XB16(S, 3) "s_mov_b64 exec, vcc\n7:"                                                  \
        : QSV_E8(a), QSV_E8(b), [t] "=&v"(t)                                                                \
        : [l] "s"(m), [x] "s"(xch)                                                                          \
        : "scc", "vcc");                                                                                    \
  }
QSV_XCH(float, QSV_SW32)
QSV_XCH(double, QSV_SW64)

// A uniform value in a scalar register.
__device__ __forceinline__ uint32_t su(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// A value that is read only where the op's flags say that it was set (no
// instruction to initialise it).
template <typename T>
__device__ __forceinline__ T unset() {
  T x;
  asm("" : "=v"(x));
  return x;
}

// Uniform values in scalar registers, whichever way they were read.
__device__ __forceinline__ int su(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t su(uint64_t x) { return uint64_t(su(uint32_t(x >> 32))) << 32 | su(uint32_t(x)); }
__device__ __forceinline__ float su(float x) { return __uint_as_float(su(__float_as_uint(x))); }
__device__ __forceinline__ double su(double x) {
  return __hiloint2double(su(__double2hiint(x)), su(__double2loint(x)));
}
template <typename R>
__device__ __forceinline__ cx<R> su(cx<R> x) {
  return {su(x.re), su(x.im)};
}

// Keeps a uniform value read here: the read is neither moved to its use nor repeated.
template <typename T>
__device__ __forceinline__ void read_now(T& x) {
  x = su(x);
  asm volatile("" : "+s"(x));
}
template <typename R>
__device__ __forceinline__ void read_now(cx<R>& x) {
  read_now(x.re);
  read_now(x.im);
}

__device__ __forceinline__ float sgn_xor(float x, uint32_t m) { return __uint_as_float(__float_as_uint(x) ^ m); }
__device__ __forceinline__ double sgn_xor(double x, uint32_t m) {
  return __hiloint2double(__double2hiint(x) ^ int(m), __double2loint(x));
}

// Parity of (tau & tm) and (base & gm), 0 or 1: per thread, the tile's part uniform.
__device__ __forceinline__ uint32_t ph_par(uint32_t tau, uint32_t tm, uint64_t base, uint64_t gm) {
  return (uint32_t(__popc(tau & tm)) + uint32_t(__popcll(base & gm))) & 1u;
}

// The phase of a kind-11 op: every diagonal factor that is due at a point of
// the pass, in one sweep of the thread's elements. What depends on register
// bits alone (one-qubit diagonals, CZ and Z strings among them) is a table of
// NR complex factors that the host forms in FP64, read through the scalar
// cache: one complex product per element, however many gates it stands for.
// CZ between a register bit and other bits is a parity of the thread index and
// the tile base: a sign flip of half the elements. Z strings across register
// and other bits turn the elements by an angle whose sign is such a parity;
// their factors are multiplied per string pattern first. What does not touch
// the registers at all becomes one factor of the whole thread.
template <typename R, int RB, int NS>
__device__ __forceinline__ void phase_apply(cx<R> (&v)[NS][1 << RB], const RegHeadDev& hd, const RegOpDev& op,
                                            const PhaseEntDev* __restrict__ ents, const cx<R>* __restrict__ pool,
                                            uint32_t tau, uint64_t base) {
  constexpr int NR = 1 << RB;
  const uint32_t fl = su(hd.flags);
  typedef decltype(flip_arg(R(0), 0u)) M;
  cx<R> C = {unset<R>(), unset<R>()}, H[kRegMaxH];
  M f[RB];
#pragma unroll
  for (int a = 0; a < RB; ++a) f[a] = unset<M>();
#pragma unroll
  for (int h = 0; h < kRegMaxH; ++h) H[h] = {unset<R>(), unset<R>()};
  if (fl & 0xf6u) {
    if (fl & 2u) {
      // kEntStep entries at a time, their records and values read together (one by
      // one, each entry waits for both in turn: parametric RY RZ CNOT ring of 8 layers
      // on 13 qubits complex64, 8 entries in most passes, 118.4 and 115.2 us)
      uint32_t sg = 0;
      C = {R(1), R(0)};
      const int n0 = int(hd.ent_counts & 0xffffu), n2 = int(hd.ent_counts >> 16);
      const PhaseEntDev* E = ents + hd.ent_begin;
      const cx<R>* V = pool + hd.ent_moff;
      for (int e = 0; e < n0; e += kEntStep) {
        uint32_t t[kEntStep];
        uint64_t g[kEntStep];
        cx<R> z0[kEntStep], z1[kEntStep];
#pragma unroll
        for (int j = 0; j < kEntStep; ++j) {
          t[j] = E[e + j].tm;
          g[j] = E[e + j].gm;
          z0[j] = V[2 * (e + j)];
          z1[j] = V[2 * (e + j) + 1];
        }
#pragma unroll
        for (int j = 0; j < kEntStep; ++j) {
          read_now(t[j]);
          read_now(g[j]);
          read_now(z0[j]);
          read_now(z1[j]);
        }
#pragma unroll
        for (int j = 0; j < kEntStep; ++j)
          if (e + j < n0) C = csel(ph_par(tau, t[j], base, g[j]) != 0, z1[j], z0[j]) * C;
      }
      E += n0;
      for (int e = 0; e < n2; e += kEntStep) {
        uint32_t t[kEntStep], t2[kEntStep];
        uint64_t g[kEntStep], g2[kEntStep];
#pragma unroll
        for (int j = 0; j < kEntStep; ++j) {
          t[j] = E[e + j].tm;
          t2[j] = E[e + j].tm2;
          g[j] = E[e + j].gm;
          g2[j] = E[e + j].gm2;
        }
#pragma unroll
        for (int j = 0; j < kEntStep; ++j) {
          read_now(t[j]);
          read_now(t2[j]);
          read_now(g[j]);
          read_now(g2[j]);
        }
#pragma unroll
        for (int j = 0; j < kEntStep; ++j)
          if (e + j < n2) sg ^= ph_par(tau, t[j], base, g[j]) & ph_par(tau, t2[j], base, g2[j]);
      }
      C = {sgn_xor(C.re, sg << 31), sgn_xor(C.im, sg << 31)};
    }
    if (fl & 4u) {
#pragma unroll
      for (int a = 0; a < RB; ++a) {
        const uint32_t w = a < 2 ? hd.tm01 : (a < 4 ? hd.tm23 : hd.tm4);
        f[a] = flip_arg(R(0), ph_par(tau, (w >> (16 * (a & 1))) & 0xffffu, base, op.gm[a]));
      }
    }
    if (fl & 0xf0u) {
#pragma unroll
      for (int h = 0; h < kRegMaxH; ++h) {
        if (!(fl >> (4 + h) & 1u)) continue;
        cx<R> z = {R(1), R(0)};
        const int nh = op.h_count[h];
        const PhaseEntDev* E = ents + op.h_begin[h];
        const cx<R>* V = pool + op.h_moff[h];
        for (int e = 0; e < nh; e += kEntStep) {
          uint32_t t[kEntStep];
          uint64_t g[kEntStep];
          cx<R> f[kEntStep];
#pragma unroll
          for (int j = 0; j < kEntStep; ++j) {
            t[j] = E[e + j].tm;
            g[j] = E[e + j].gm;
            f[j] = V[e + j];
          }
#pragma unroll
          for (int j = 0; j < kEntStep; ++j) {
            read_now(t[j]);
            read_now(g[j]);
            read_now(f[j]);
          }
#pragma unroll
          for (int j = 0; j < kEntStep; ++j)
            if (e + j < nh) z = cx<R>{f[j].re, sgn_xor(f[j].im, ph_par(tau, t[j], base, g[j]) << 31)} * z;
        }
        H[h] = z;
      }
    }
  }
  const uint32_t rsg[4] = {su(hd.h_rsg[0]), su(hd.h_rsg[1]), su(hd.h_rsg[2]), su(hd.h_rsg[3])};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if constexpr (RB == 3) {
      lane8(v[s], C, f, H, fl, rsg);
    } else {
      // (32 elements: bit 4 is set in the second half; its sign as bit 3's of
      // a pass over that half whose other parts are masked out)
      lane16(v[s], C, f, H, fl, rsg);
      if constexpr (RB == 5) {
        const uint32_t hi[4] = {rsg[0] >> 16, rsg[1] >> 16, rsg[2] >> 16, rsg[3] >> 16};
        lane16(v[s] + 16, C, f, H, fl, hi);
        const M f4[4] = {f[4], f[4], f[4], f[4]};
        cx<R>* const w = v[s] + 16;
        cx<R> x[16];
#pragma unroll
        for (int k = 0; k < 8; ++k) {  // (elements 16 .. 23 as the set ones, then 24 .. 31)
          x[k] = w[k];
          x[k + 8] = w[k];
        }
        lane16(x, C, f4, H, fl >> 12 & 1u ? 0x800u : 0u, hi);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          w[k] = x[k + 8];
          x[k + 8] = w[k + 8];
        }
        lane16(x, C, f4, H, fl >> 12 & 1u ? 0x800u : 0u, hi);
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k + 8] = x[k + 8];
      }
    }
  }
  const cx<R>* T = pool + hd.moff;  // (read also by an op without a table: the pool ends with a spare one)
#pragma unroll
  for (int r = 0; r < NR; r += 8) {
    cx<R> z[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) z[k] = T[r + k];
#pragma unroll
    for (int s = 0; s < NS; ++s) tab8(v[s] + r, z, fl);
  }
}

// The rotations of a kind-11 op: a layer on distinct register bits, the shears
// of bit p at coef[p].
template <typename R, int RB>
__device__ __forceinline__ void rot_layer(cx<R>* v, uint32_t rot, const cx<R>* __restrict__ coef) {
  cx<R> c[RB];
#pragma unroll
  for (int p = 0; p < RB; ++p) c[p] = coef[p];
  static_assert(RB >= 3 && RB <= 5, "8, 16 or 32 elements");
  if constexpr (RB == 3) {
    rot8(v, c, rot);
  } else {
    rot16(v, c, rot);
    if constexpr (RB == 5) {
      rot16(v + 16, c, rot);
      const uint32_t r4 = (rot >> 1) & 0x808u;  // bit 4 in the place of bit 3
      rot_pairs8(v, v + 16, c[4], r4);
      rot_pairs8(v + 8, v + 24, c[4], r4);
    }
  }
}

// Lanes in which a kind-11 op's exchange acts: controls on thread bits and
// non-local qubits.
__device__ __forceinline__ uint64_t exchange_mask(uint32_t xch, const RegOpDev& op, uint32_t tau, uint64_t base) {
  uint64_t m = 0;
  if (xch) m = __ballot((tau & op.ti_cm) == op.ti_cv && (base & op.gcm) == op.gcv);
  return m;
}

// The exchange of a kind-11 op (X, controlled X on a register bit).
template <typename R, int RB>
__device__ __forceinline__ void exchange(cx<R>* v, uint32_t xch, uint64_t m) {
  if constexpr (RB == 3) {
    xch8(v, m, xch);
  } else {
    xch16(v, m, xch);
    if constexpr (RB == 5) {  // (the pairs of the second half; register bit 4)
      const uint32_t hi = (xch & 0xfu) | ((xch >> 16 & 0xffu) << 8);
      xch16(v + 16, m, hi);
      const uint32_t b4 = xch >> 1 & 8u;
      xch_pairs8(v, v + 16, m, b4 | (xch & 0xff00u));
      xch_pairs8(v + 8, v + 24, m, b4 | (xch >> 8 & 0xff00u));
    }
  }
}

// Factor table of a diagonal op (k <= 2) for this thread: index bits from
// thread and non-local targets are fixed; register targets become the bits
// a < b of the table index.
template <typename R>
__device__ __forceinline__ void diag_table(const RegOpDev& op, const cx<R>* __restrict__ d, uint32_t tau,
                                           uint64_t base, cx<R>* g, int& a, int& b) {
  int fixed = 0, ja = 0, jb = 0;
  a = -1;
  b = -1;
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // (k <= 2)
    if (j >= op.k) break;
    if (op.dsrc[j] == 1) fixed |= int((tau >> op.dbit[j]) & 1) << j;
    else if (op.dsrc[j] == 2) fixed |= int((base >> op.dbit[j]) & 1) << j;
    else if (a < 0) {
      a = op.dbit[j];
      ja = j;
    } else {
      b = op.dbit[j];
      jb = j;
    }
  }
  if (b >= 0 && b < a) {
    const int t = a, tj = ja;
    a = b;
    ja = jb;
    b = t;
    jb = tj;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int idx = fixed;
    if (a >= 0 && (e & 1)) idx |= 1 << ja;
    if (b >= 0 && (e & 2)) idx |= 1 << jb;
    g[e] = d[idx];
  }
}

// Orders this wavefront's LDS accesses (a compiler barrier: the hardware
// performs one wavefront's LDS operations in issue order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS addresses of a layout. The swizzle is linear over XOR and a local index
// is the XOR of its register part and its thread part, so the byte offset of
// element i is the per-thread part XOR a part that depends only on i and the
// layout (uniform across the workgroup: a table the planner fills, read
// through the scalar cache). Kernels using it declare no static LDS and put
// the tile first in their dynamic LDS, so it starts at LDS address 0 and the
// base folds into the per-thread part: one vector XOR per element remains.
template <typename R, int RB>
struct LdsMap {
  uint32_t thr;           // per-thread part, in bytes
  uint32_t reg[1 << RB];  // per-element parts, in bytes (uniform)
  __device__ __forceinline__ LdsMap(const uint32_t* regt, uint32_t thr_) : thr(thr_) {
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) reg[i] = regt[i];
  }
  typedef R R2 __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(3))) R2 lds_r2;
  __device__ __forceinline__ lds_r2* at(char* lds, int i) const {
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(lds));
    return reinterpret_cast<lds_r2*>(uintptr_t((base + thr) ^ reg[i]));
  }
  __device__ __forceinline__ void put(char* lds, int i, const cx<R>& x) const {
    R2 w;
    w.x = x.re;
    w.y = x.im;
    *at(lds, i) = w;
  }
  __device__ __forceinline__ cx<R> get(char* lds, int i) const {
    const R2 w = *at(lds, i);
    return {w.x, w.y};
  }
};

// The thread's bits as masks (all ones where bit k of the index is set): the
// linear maps of a pass are XORs of columns over them, one v_bitop3 (j ^ (c &
// m)) each.
template <int TB>
struct ThrMask {
  uint32_t m[TB];
  __device__ __forceinline__ explicit ThrMask(uint32_t tau) {
#pragma unroll
    for (int k = 0; k < TB; ++k) m[k] = 0u - ((tau >> k) & 1u);
  }
  // truth table of a ^ (b & c): 0x78 with a = 0xf0, b = 0xcc, c = 0xaa
  __device__ __forceinline__ uint32_t map(uint32_t cst, const uint32_t* col) const {
    uint32_t j = cst;
#pragma unroll
    for (int k = 0; k < TB; ++k) j = __builtin_amdgcn_bitop3_b32(j, col[k], m[k], 0x78);
    return j;
  }
};

// A kind-11 op.
template <typename R, int RB>
__device__ __forceinline__ void reg_super(const RegHeadDev& hd, const RegOpDev& op, cx<R> (&v)[1][1 << RB],
                                          uint32_t tau, uint64_t base, const PhaseEntDev* __restrict__ ents,
                                          const cx<R>* __restrict__ pool) {
  phase_apply<R, RB, 1>(v, hd, op, ents, pool, tau, base);
  rot_layer<R, RB>(v[0], su(hd.rot), pool + hd.roff);
  exchange<R, RB>(v[0], su(hd.xch), exchange_mask(hd.xch, op, tau, base));
}

// Any other op. Ops with non-local controls that do not match this tile do
// nothing; ops on LDS (kind 3) go through the tile in LDS; controls on thread
// bits are per lane.
template <typename R, int RB, int KMAX, int TB>
__device__ __forceinline__ void reg_general(const RegHeadDev& hd, const RegOpDev& op, cx<R> (&v)[1][1 << RB], const RegSegDev& S,
                                            const ThrMask<TB>& tm, uint32_t tau, uint64_t base, Swz<sizeof(R) == 4 ? 5 : 4> sw,
                                            char* smem, const TileOpDev* __restrict__ lops,
                                            const cx<R>* __restrict__ pool, int L) {
  constexpr int NR = 1 << RB;
  // (dense products without controls need the head alone, which is there already:
  // nothing waits for the record before the matrix is read)
  const cx<R>* m = pool + hd.moff;
  int key = int(hd.xch);
  uint32_t cm = 0, cv = 0;
  bool lane = true;
  cx<R> g[4];
  if (!(hd.flags & 1u)) {
    if ((base & op.gcm) != op.gcv) return;  // non-local controls: uniform per tile
    if (op.kind == 3) {
      const LdsMap<R, RB> ms(S.get_reg, tm.map(0u, S.tcol) >> 16);
      __syncthreads();  // (a preceding cross-wave re-map's reads are done)
#pragma unroll
      for (int i = 0; i < NR; ++i) ms.put(smem, i, v[0][i]);
      __syncthreads();
      lds_op<R, KMAX>(reinterpret_cast<cx<R>*>(smem), lops[op.lop], pool, L, base, sw);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NR; ++i) v[0][i] = ms.get(smem, i);
      __syncthreads();
      return;
    }
    int a = op.p1, b = op.p2;
    if (op.kind == 2) diag_table<R>(op, m, tau, base, g, a, b);
    key = op.key;
    cm = op.ri_cm;
    cv = op.ri_cv;
    lane = (tau & op.ti_cm) == op.ti_cv;
  }
  reg_apply<R, NR>(v[0], key, m, g, cm, cv, lane);
}

// Register budget (the launch bound's second argument: wavefronts per SIMD):
// complex64 tiles of 16 amplitudes per thread keep four (128 VGPRs; with 32
// KiB of LDS per 256 threads, four workgroups of 256 or two of 512 per compute
// unit); wider tiles and complex128 take what they need.
template <typename R, int RB>
constexpr int tile_waves_per_simd() {
  return (sizeof(R) == 4 && RB == 4) ? 4 : 1;
}

// HBM side of a pass: amplitudes of a thread in a layout's order. Per thread
// part of the address th (with base), uniform parts per register element.
template <typename R, int RB, bool STORE>
__device__ __forceinline__ void tile_io(R* __restrict__ psi, cx<R>* v, uint64_t th, const RegSegDev& S) {
  constexpr int NR = 1 << RB;
  uint64_t greg[RB];
#pragma unroll
  for (int k = 0; k < RB; ++k) greg[k] = S.gcol_r[k];
  // complex64: register bit 0 is local bit 0 in the first and last layouts of
  // a pass (16-byte pairs)
  constexpr int V = sizeof(R) == 4 ? 2 : 1;
#pragma unroll
  for (int i = 0; i < NR; i += V) {
    uint64_t x = th;
#pragma unroll
    for (int k = V - 1; k < RB; ++k)
      if ((i >> k) & 1) x |= greg[k];
    if constexpr (STORE) AmpIO<R, V>::store(psi, x, &v[i]);
    else AmpIO<R, V>::load(psi, x, &v[i]);
  }
}

// Index of the first amplitude of tile g.
__device__ __forceinline__ uint64_t pass_base(const TilePassDev& P, uint32_t g) {
  uint64_t base = 0;
  for (int r = 0; r < P.nrun; ++r) base |= uint64_t((g >> P.rsrc[r]) & ((1u << P.rlen[r]) - 1)) << P.rdst[r];
  return base;
}

// A pass's tables are read through the scalar cache, a record when it is due, and
// every launch finds that cache empty: where few workgroups share them, each read
// is a trip to memory in a chain of dozens. So every thread reads a cache line of
// each table first, all at once, into the L2 of its XCD -- in the first workgroups of
// a pass (32 per XCD): later ones find them there. Measured with fewer taken
// branches per op (rot16, lane16): that ring 115.2 -> 110.1 us, on 17 qubits
// complex128 209.5 -> 196.3. The value has to be kept until the reads have come back.
constexpr uint32_t kWarmTiles = 256;
__device__ __forceinline__ uint32_t touch(const void* p, uint32_t bytes, uint32_t tau) {
  uint32_t x = 0;
  if (tau * 128u < bytes) x = *reinterpret_cast<const uint32_t*>(static_cast<const char*>(p) + tau * 128u);
  return x;
}

// KMAX 0: passes of kind-11 ops only. Workgroups are persistent: workgroup b
// takes tiles b, b + grid, ... and (KMAX 0) issues the loads of its next tile before
// it computes on the current one. General products need those registers: with
// the read-ahead they spilled. Measured at 24 qubits complex64 with it and without:
// six layers of dense two-qubit blocks 905 and 864 us, of controlled unitaries 881
// and 804, of non-unitary one-qubit matrices 1150 and 918, two layers of dense
// four-qubit blocks 1277 and 1108 (heads alone read for uncontrolled products
// included: reg_general). LDS (32 KiB tiles in granules of 1280 bytes)
// holds four workgroups on a compute unit, four wavefronts per SIMD, so a
// wavefront has 128 registers: 32 amplitude words, 32 of the next tile. Bound
// by vector issue: at 30 qubits complex64 (15 passes of the layered circuit,
// 1897 vector instructions per wavefront and tile) a pass takes 4.91 ms, 66%
// of it vector issue; its read and write of the state alone take 3.9 ms. With
// matrix products in two register arrays (3320 to 4740 instructions) it took
// 5.6 to 6.3 ms, over fresh workgroups per tile.
template <typename R, int RB, int KMAX, int TB>
__device__ __forceinline__ void tile_pass(R* __restrict__ psi, const TilePassDev& P, uint32_t g, uint32_t step,
                                          uint32_t ntiles, uint32_t warm_tiles, const RegSegDev* __restrict__ segs,
                                          const RegHeadDev* __restrict__ heads, const RegOpDev* __restrict__ rops,
                                          const TileOpDev* __restrict__ lops, const PhaseEntDev* __restrict__ ents,
                                          const cx<R>* __restrict__ pool, char* smem) {
  constexpr int NR = 1 << RB;
  constexpr int SB = sizeof(R) == 4 ? 5 : 4;
  const Swz<SB> sw;
  const int L = P.L;
  const uint32_t tau = threadIdx.x;
  const ThrMask<TB> tm(tau);
  const RegSegDev* const S0 = &segs[P.seg_begin];
  int nseg = P.seg_count;
  read_now(nseg);
  uint32_t warm = 0;
  if (g < warm_tiles)
    warm = touch(S0, uint32_t(nseg) * uint32_t(sizeof(RegSegDev)), tau) ^
           touch(heads + P.rop_begin, uint32_t(P.rop_count) * uint32_t(sizeof(RegHeadDev)), tau) ^
           touch(rops + P.rop_begin, uint32_t(P.rop_count) * uint32_t(sizeof(RegOpDev)), tau) ^
           touch(ents + P.ent_begin, uint32_t(P.ent_count) * uint32_t(sizeof(PhaseEntDev)), tau) ^
           touch(pool + P.pool_begin, uint32_t(P.pool_count) * uint32_t(sizeof(cx<R>)), tau);
  const RegSegDev* const SL = S0 + (nseg - 1);
  uint64_t th0 = 0, thL = 0;
#pragma unroll
  for (int k = 0; k < TB; ++k) {
    const uint64_t on = uint64_t(int64_t(int32_t(tm.m[k])));
    th0 |= S0->gcol_t[k] & on;
    thL |= SL->gcol_t[k] & on;
  }
  constexpr bool AHEAD = KMAX == 0;
  cx<R> v[1][NR], pf[AHEAD ? NR : 1];
  uint64_t base = pass_base(P, g);
  if constexpr (AHEAD) tile_io<R, RB, false>(psi, pf, base | th0, *S0);
  for (;;) {
    const uint32_t gn = g + step;  // (ntiles <= 2^27: no overflow)
    const uint64_t nbase = gn < ntiles ? pass_base(P, gn) : 0;
    if constexpr (AHEAD) {
#pragma unroll
      for (int i = 0; i < NR; ++i) v[0][i] = pf[i];
      if (gn < ntiles) tile_io<R, RB, false>(psi, pf, nbase | th0, *S0);
    } else {
      tile_io<R, RB, false>(psi, v[0], base | th0, *S0);
    }
    const RegSegDev* S = S0;
    int oi = S->op_begin;
    RegHeadDev next = heads[oi];  // the next op's head, read one op ahead
    for (int sgi = 0; sgi < nseg; ++sgi) {
      const RegSegDev* Sn = S0 + sgi;
      int oe = Sn->op_begin + Sn->op_count;
      if (sgi > 0) {
        // re-map through LDS, applying the ops folded into it on the way; when
        // both layouts share the wave bits (and no folded op targets one), every
        // wavefront reads back only what it wrote, and LDS operations of one
        // wavefront complete in order: no workgroup barrier is needed
        const bool xw = (Sn->xwave & 1) != 0;
        const bool xpre = (Sn->xwave & 2) != 0;
        // (both address maps are formed before the barriers: one wait for their tables)
        const uint32_t j = tm.map(Sn->tcst, Sn->tcol);
        const LdsMap<R, RB> mo(Sn->put_reg, j & 0xffffu);
        const LdsMap<R, RB> mn(Sn->get_reg, j >> 16);
        read_now(oe);
        if (xpre) __syncthreads();
#pragma unroll
        for (int i = 0; i < NR; ++i) mo.put(smem, i, v[0][i]);
        if (xw) __syncthreads();
        else wave_sync();
#pragma unroll
        for (int i = 0; i < NR; ++i) v[0][i] = mn.get(smem, i);
        // a cross-wave re-map's closing barrier waits for the next LDS write
        // (marked on the next re-map; ops through LDS always wait first), so
        // the segment's register ops overlap the wavefronts' skew
        if (!xw) wave_sync();
      }
      S = Sn;
      // (a pass's ops are contiguous: the read ahead goes on across segments)
      while (oi < oe) {
        const RegHeadDev hd = next;
        const RegOpDev& op = rops[oi];
        next = heads[++oi];
        if constexpr (KMAX > 0) {
          if ((hd.flags >> 24) != 11) {
            reg_general<R, RB, KMAX, TB>(hd, op, v, *S, tm, tau, base, sw, smem, lops, pool, L);
            continue;
          }
        }
        reg_super<R, RB>(hd, op, v, tau, base, ents, pool);
      }
    }
    if (P.scale_off >= 0) {  // the sign left by the pass's rotations, when no phase op took it
      const R f = pool[P.scale_off].re;
      if (f != R(1)) {
#pragma unroll
        for (int i = 0; i < NR; ++i) v[0][i] = {f * v[0][i].re, f * v[0][i].im};
      }
    }
    tile_io<R, RB, true>(psi, v[0], base | thL, *SL);
    if (gn >= ntiles) break;
    g = gn;
    base = nbase;
    __syncthreads();  // every wavefront has read its last re-map: LDS is free
  }
  asm volatile("" ::"v"(warm));
}

template <typename R, int RB, int KMAX, int TB>
__global__ void __launch_bounds__(1 << TB, (tile_waves_per_simd<R, RB>()))
    k_tile_reg(R* __restrict__ psi, const TilePassDev* __restrict__ passes, int pass_idx, uint32_t ntiles,
               const RegSegDev* __restrict__ segs, const RegHeadDev* __restrict__ heads,
               const RegOpDev* __restrict__ rops, const TileOpDev* __restrict__ lops, const PhaseEntDev* __restrict__ ents,
               const cx<R>* __restrict__ pool) {
  extern __shared__ __align__(16) char smem[];
  // (the grid has at most ntiles workgroups)
  tile_pass<R, RB, KMAX, TB>(psi, passes[pass_idx], blockIdx.x, gridDim.x, ntiles, kWarmTiles, segs, heads, rops, lops,
                             ents, pool, smem);
}

}  // namespace qsv

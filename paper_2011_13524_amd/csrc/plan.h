// Fusion plans: gates merged into dense blocks (section 5.4) and blocks
// scheduled into tile passes, each pass applying many blocks per read and
// write of the state.
#pragma once

#include <vector>

#include "circuit.h"

struct qsv_plan;

namespace qsv {

constexpr int kTileMaxOps = 4096;
constexpr int kTileMaxHigh = 16;
constexpr int kTileMaxGlobal = 40;

// One operation inside a tile pass, in the tile's local index space (local
// bit p <-> qubit local[p]).
struct TileOpDev {
  int kind;        // 0 dense on local targets, 1 diagonal (targets local or not),
                   // 2 gradient rotation of the reverse sweep (k = Pauli id),
                   // 3 gradient term of a multi-qubit Pauli rotation (reverse sweep;
                   //   no update): off[0] local flip mask, off[1] local Z/Y mask,
                   //   off[2] phase exponent (P x = i^off[2] (-1)^|x & zy| (x ^ f)
                   //   up to the tile's sign), off[3..4] Z/Y mask on non-local
                   //   qubits (low, high word), ins[0] row, ins[1] slot in the pass
                   // register-resident passes only:
                   // 4 rotation in the plane of a qubit's two amplitudes (xswap: axis,
                   //   1 X, 2 Y) on the local target lt[0]
                   // 5 phase (diagonal, sub-kind PhaseSub in sub)
                   //   both: m = 1 in the reverse sweep: with a gradient row
  int k;           // number of targets
  int m;           // number of inserted zero positions (dense: targets + local controls)
  int moff;        // offset of the matrix / diagonal in the pool (complex elements);
                   // register-resident passes: offset in the plan's host values
  int lt[5];       // dense: local target positions; diag: local position or -1
  int gq[5];       // diag: global qubit of a non-local target, or -1
  int ins[10];     // dense: sorted local positions with zero bits (targets + local controls);
                   // gradient: ins[0] = row of the gradient, ins[1] = its slot in the pass
  int xswap;       // 1: the one-qubit matrix is Pauli X (a pure exchange); kind 4: the axis
  int sub;         // kind 5: PhaseSub
  uint32_t lcm, lcv;  // local control mask / values (local index space)
  uint64_t gcm, gcv;  // non-local control mask / values (global index space)
  uint32_t off[32];   // dense: local offset of the i-th element of B1
};

// Kinds of phase ops: a diagonal one-qubit factor (two values), the sign of
// CZ (no value), exp(+i t Z...Z / 2) on any number of qubits (one value: cos +
// i sin of t/2).
enum PhaseSub { PH_DIAG1 = 0, PH_CZ = 1, PH_ZSTR = 2 };

struct TilePassDev {
  int L, b, nh, ng;
  int op_begin, op_count;
  int seg_begin, seg_count;  // register-resident execution (seg_count > 0)
  int row_begin, row_count;  // reverse sweep: gradient rows of the pass (slot s -> rows[row_begin + s])
  int hq[kTileMaxHigh];      // qubits of local bits b..L-1
  int gpos[kTileMaxGlobal];  // non-local qubits, ascending
  // the same map from tile index to tile base as runs of consecutive
  // non-local qubits: base = OR over r of ((g >> rsrc[r]) & (2^rlen[r] - 1)) << rdst[r]
  int nrun;
  int rsrc[kTileMaxHigh + 1], rdst[kTileMaxHigh + 1], rlen[kTileMaxHigh + 1];
  // register-resident execution: pool offset of a real factor that the tile is
  // multiplied by when it is stored (the sign the pass's rotations left), -1: none
  int scale_off;
  int general;  // the pass holds ops other than kind 11 (selects the kernel)
  // register-resident execution: the pass's ops, entries and pool values
  int rop_begin, rop_count, ent_begin, ent_count, pool_begin, pool_count;
};

// Register-resident tiles: the 2^L tile is spread over 2^TB threads holding
// 2^RB amplitudes each. A segment fixes which local bits index a thread's
// registers (reg) and which index the thread (thr: lanes first, then the
// wavefront index); ops of the segment whose dense targets are register bits
// run without touching LDS.
constexpr int kRegMaxBits = 6;
constexpr int kRegThreadBits = 8;      // default: 256-thread workgroups
constexpr int kRegMaxThreadBits = 9;   // up to 512-thread workgroups

struct RegSegDev {
  int reg[kRegMaxBits];        // local positions of register-index bits, ascending
  int thr[kRegMaxThreadBits];  // local position of thread-index bit k
  int xwave;                   // re-map into this layout: bit 0 across wavefronts (a
                               // barrier between writes and reads; none after the
                               // reads), bit 1 a workgroup barrier before the writes
  int op_begin, op_count;
  // the re-map into this layout writes local index x of the previous layout
  // to position M x ^ mcst (folded X / controlled-X ops); mcol[p] = M e_p
  uint32_t mcol[kTileMaxHigh + 8];
  uint32_t mcst;
  // LDS byte offsets, XOR-swizzled (filled by the planner for the plan's
  // dtype): element i of the thread with index tau sits at
  //   (tcst ^ XOR of tcol[k] over the set bits k of tau) ^ reg[i]
  // put_*: the previous layout written through the map above (the re-map
  // into this layout); get_*: this layout (tcst = 0).
  // The thread parts of both come packed: put in the low half of tcol[k] and
  // tcst, get in the high half of tcol[k] (a tile is at most 64 KiB).
  uint32_t put_reg[1 << (kRegMaxBits - 1)];
  uint32_t get_reg[1 << (kRegMaxBits - 1)];
  uint32_t tcol[kRegMaxThreadBits], tcst;
  // global index bit of thread-index bit k and of register-index bit k in this
  // layout (HBM addresses of the first and last segments of a pass)
  uint64_t gcol_t[kRegMaxThreadBits], gcol_r[kRegMaxBits];
};

constexpr int kRegMaxH = 4;  // string patterns of one phase op

// One op of a segment. Kind 11 -- almost every op -- is a phase (diagonal
// factors), then a layer of rotations on distinct register bits, then an
// exchange, each part optional. The other kinds are general products.
struct RegOpDev {
  int kind;             // 0 dense one-qubit, 1 dense two-qubit, 2 diagonal (k <= 2), 3 via LDS,
                        // 11 phase / rotations / exchange; reverse sweep: 8 gradient of a Pauli string
  uint32_t flags;       // kind 11: 1 table over the register bits, 2 factor of the thread, 4 signs,
                        // 8 gradient rows of Z rotations, 16 << h: string pattern h, 256 << a: sign of
                        // register bit a
  int moff;             // pool offset of the op's values (kind 11: of the table)
  int roff;             // kind 11: pool offset of the rotations' shears (one per register bit)
  uint32_t rot;         // kind 11: register bits rotated about Y (bits 0-7) and X (8-15); bits 16-23:
                        // with a gradient (reverse sweep)
  uint32_t xch;         // kind 11: exchange of the pairs of one register bit (one-hot), bits 8-23: the
                        // pairs whose register bits match the controls
  // kind 11: entries of the thread's factor: ent_count of PhaseEntDev kind 0, whose
  // pairs of values follow each other from pool offset ent_moff, then ent_cz of kind 2
  int ent_begin, ent_count, ent_cz, ent_moff;
  int row_begin, row_count;  // kind 11: gradient rows (kind 4)
  // kind 11: string factors (kind 3) of pattern h, their values from h_moff
  int h_begin[kRegMaxH], h_count[kRegMaxH], h_moff[kRegMaxH];
  uint32_t h_rsg[kRegMaxH];  // bit r: the sign of element r in pattern h
  // kind 11: elements with register bit a set change sign when the parity of
  // (thread index & tm[a]) and (tile base & gm[a]) is odd
  uint32_t tm[kRegMaxBits];
  uint64_t gm[kRegMaxBits];
  uint64_t gcm, gcv;      // controls on non-local qubits (exchange, kinds 0-3)
  uint32_t ti_cm, ti_cv;  // controls on thread bits (thread-index space)
  uint32_t ri_cm, ri_cv;  // controls on register bits (register-index space)
  int key;              // kinds 0, 1, 2: variant of the register op (reg_key)
  int lop;              // index of the equivalent TileOpDev (LDS execution)
  int p1, p2;           // register bits of matrix index bits 0 and 1
  int k;
  int dsrc[2], dbit[2]; // diagonal targets: source 0 register bit, 1 thread bit, 2 global qubit
  int aux[kRegMaxBits]; // gradients: slot of the row in the pass (rotations: per register bit)
  // kind 8 (reverse sweep): gradient term of a multi-qubit Pauli rotation,
  // evaluated with psi staged in LDS: the partner of element i sits at its LDS
  // address XOR pf_lds; the sign parity is that of (i & pz_reg), (thread index
  // & pz_thr) and (tile base & pz_glob); phase exponent pph (0..3)
  uint32_t pf_lds, pz_reg, pz_thr;
  int pph;
  uint64_t pz_glob;
};

// What every op of a segment needs of its RegOpDev (same index), in one cache
// line that the kernels read one op ahead. A spare record follows the last.
struct alignas(64) RegHeadDev {
  uint32_t flags;  // RegOpDev::flags; bits 24-31: the kind (kinds 0, 1: flag 1 without controls)
  uint32_t rot, xch;  // (kinds 0, 1 without controls: xch is the key)
  int moff, roff;
  int ent_begin, ent_moff;
  uint32_t ent_counts;  // kind 0, << 16 kind 2
  int row_count;
  uint32_t h_rsg[kRegMaxH];
  uint32_t tm01, tm23, tm4;  // tm[], 16 bits each
};

// A factor of a phase that depends on the thread or the tile. par(t, g) is the
// parity of (thread index & t) and (tile base & g). Kinds in this order:
//   0 every element times the par(tm, gm)-th of the entry's two values
//   2 every element times (-1)^(par(tm, gm) par(tm2, gm2))
//   3 a factor c + i s (-1)^par(tm, gm) of a string pattern, (c, s) the entry's
//     value: the product of its factors multiplies element r, conjugated where the
//     pattern's bit r is set
//   4 reverse sweep: gradient row (slot moff) of a rotation about Z, with the
//     sign of par(tm, gm) and, where ra >= 0, of register bit ra
// The kernels read the entries and values of kEntStep entries at once: the pool
// offsets are the op's, and kEntStep - 1 spare records end the table.
constexpr int kEntStep = 4;
struct PhaseEntDev {
  int kind;
  int moff;  // kind 4: the slot
  uint32_t tm, tm2;
  uint64_t gm, gm2;
  int ra;
  uint32_t rsg;  // (planner: the pattern of kind 3)
};

// How the device pool is formed from the host values (the plan's matrices,
// phases and rotations for one theta), in FP64.
struct TabComp {
  int type;  // 0 one-qubit diagonal: times val[src + bit a of r]; 1 two-qubit: val[src + (bit a | bit b << 1)];
             // 2 sign of bits a and b both set; 3 val[src], conjugated where bit r of rsg is set;
             // 4 times the real part of val[src + 1] (the sign a rotation left)
  int src, a, b;
  uint32_t rsg;
};
struct PoolRec {
  int type;  // 0 copy n values from src; 1 table of n entries: product of the comps
  int dst, src, n;
  std::vector<TabComp> comps;
};

// Register-resident layout of a tile: 2^reg_bits amplitudes per thread,
// 2^thread_bits threads.
struct SegCfg {
  int reg_bits, thread_bits;
  bool c64;  // complex64: the HBM layouts keep local bit 0 in registers (16-byte pairs)
};

// Register-resident form of the passes built so far.
struct SegBuild {
  std::vector<RegSegDev> segs;
  std::vector<RegOpDev> rops;
  std::vector<PhaseEntDev> ents;
  std::vector<PoolRec> recs;
  int pool_elems = 0;
};

// Splits the ops of pass d (ho[d.op_begin ..]) into register segments,
// appending them to out; d.seg_count is incremented per segment (the caller
// sets d.seg_begin = segs.size() and d.seg_count = 0 first). Ops executed
// through LDS get their pool offset written back to ho.
int build_reg_segments(const SegCfg& cfg, std::vector<TileOpDev>& ho, TilePassDev& d, SegBuild& out);

// Fills the run-length form of d.gpos (d.nrun, rsrc, rdst, rlen).
void pass_runs(TilePassDev& d);

// Spare elements at the end of an assembled pool (ops without a table or
// rotations read theirs from offset 0).
constexpr int kPoolSpare = 64;

// The heads of a SegBuild's ops, and its entries with the spare ones.
std::vector<RegHeadDev> op_heads(const SegBuild& sb);
std::vector<PhaseEntDev> op_entries(const SegBuild& sb);

// The device pool of a SegBuild from the host values (FP64; the caller rounds).
void assemble_pool(const SegBuild& sb, const std::vector<cd>& vals, std::vector<cd>& pool);

// Values of a rotation exp(+i t P / 2) about X or Y for a kind-4 op: (tan(t/4),
// -sin(t/2)) for the angle reduced to |t/2| <= pi/2, then the sign (+-1, 0) that
// the reduction left. With x, y the two components it turns, x += tan y, y -=
// sin x, x += tan y is the rotation: three FMAs per component pair, in place,
// of determinant 1 whatever the rounding of the two factors.
void rotation_shears(double t, cd* out);

// A one-qubit unitary U (up to a real factor) as diag(out[4], out[5]) times a
// rotation about Y (its shears and sign out[2..3]) times diag(out[0], out[1]).
void unitary_to_rotation(const cd* u, cd* out);

// Whether u (2 x 2) is unitary up to a real factor within tol.
bool is_unitary2(const cd* u, double tol);

// Whether u runs as a rotation between diagonals in passes of that dtype (else as a
// general product). complex64: unitary to 1e-9 (the factors are rounded to 6e-8
// anyway, as the entries would be). complex128: the factors have to give u back to
// half a unit in the last place of 1 (H does): entries are used as they
// come in a product, while three phases and two shears, each rounded, are off by
// 2e-16 for a matrix whose rows are orthogonal only to rounding -- the same error on
// every amplitude. Ten layers of Haar one-qubit gates and CZ on 16 qubits: 8.6e-15
// off with every unitary as a rotation, 1.3e-15 as products.
bool runs_as_rotation(const cd* u, bool c64);

// An elementary op of a plan or of the reverse sweep, before it is placed in a
// pass: what the pass scheduler needs.
struct PassOp {
  uint64_t nd = 0, dg = 0;  // qubits acted on non-diagonally / diagonally
  uint64_t local = 0;       // qubits that have to be local
  bool lazy = false;        // a phase: placed in the pass of the first op that needs it
  int rows = 0;             // gradient rows
  int weight = 1;           // what placing it is worth
};

// Assigns ops to passes of at most L local qubits (the low b always among
// them) and at most max_rows gradient rows; fills the op lists (in execution
// order) and the local sets (L qubits each, or all n).
int schedule_passes(const std::vector<PassOp>& ops, int n, int L, int b, int max_rows,
                    std::vector<std::vector<int>>& pass_ops, std::vector<uint64_t>& pass_local);

// A host value that depends on a parameter: type 0 a rotation's shears and sign
// (two values), 1 a rotation about Z's diagonal (two values), 2 the phase of a
// string of Z's (one value), at voff, for the angle sgn * theta[slot].
struct DynVal {
  int type, voff, slot;
  double sgn;
};

// Tables of a reverse sweep (host side; the values for the theta given, or
// with theta null the constant ones: register-resident sweeps only, and refused
// where a value other than those of DynVal depends on theta).
struct AdjTables {
  int L = 0, kmax = 1;
  bool reg = false;
  int thread_bits = 8;  // register-resident passes
  std::vector<TilePassDev> hp;
  std::vector<TileOpDev> ho;
  SegBuild sb;
  std::vector<cd> vals;
  std::vector<DynVal> dyn;
  std::vector<int> prow;      // gradient rows of each pass, in slot order
  std::vector<int> row_slot;  // parameter slot of each row
};
template <typename R>
int adjoint_tables(const qsv_circuit* c, const double* theta, AdjTables& T);


// Reverse-sweep tables kept with a forward plan: those that do not depend on
// theta, on the host and on the device that first needed them.
struct AdjCache {
  AdjTables T;
  bool usable = false;
  void* dev = nullptr;
  int device = -1;
};
// The tables of c's reverse sweep kept with `plan` (made on the first call), or
// null where they cannot be: c is not the plan's circuit, its sweep is not
// register-resident, or values other than rotations' and Z strings' depend on
// theta.
template <typename R>
AdjCache* adjoint_cache(qsv_plan* plan, const qsv_circuit* c);
void adjoint_cache_free(AdjCache* a);
// T.vals with the values that depend on theta.
void adjoint_values(const AdjTables& T, const double* theta, std::vector<cd>& vals);

constexpr int kAdjMaxRows = 64;  // gradient rows per pass (LDS slots)

// Structure of one gate: targets/controls after control extraction and
// whether the remaining target matrix is diagonal (value-independent for
// rotations: Z rotations are diagonal for every angle).
struct GateInfo {
  std::vector<int> targets, controls, ctrl_vals;
  std::vector<cd> mat;  // extracted matrix (MATRIX gates only)
  bool diagonal = false;
  bool exchange = false;  // extracted matrix is Pauli X on one target
  uint64_t qubits = 0;
};

// A fused block: gates (indices into the circuit) applied in order, acting on
// `qubits` (ascending). Single-gate blocks keep the gate's control structure.
struct Block {
  std::vector<int> gates;
  std::vector<int> qubits;  // all qubits the block touches
  bool diagonal = false;
  bool xswap = false;  // single gate whose extracted matrix is Pauli X (CNOT, X)
  // structure used on the device (targets + controls after extraction)
  std::vector<int> targets;
  std::vector<int> controls, ctrl_vals;
};

// How an elementary op's host values come from its block.
enum LopVal {
  LV_BLOCK = 0,  // the block's matrix (dense) or diagonal
  LV_NONE,       // no value (CZ)
  LV_ROT,        // rotation about X / Y of gate `gate`: 2 values
  LV_DIAG1,      // product of the one-qubit diagonal gates gates[0..] on one qubit: 2 values
  LV_ZSTR,       // product of Pauli-Z strings gates[0..]: 1 value
  LV_U_FIRST,    // first diagonal of the block's unitary: 6 values for it and the two below
  LV_U_ROT,
  LV_U_LAST
};

struct Lop {
  int kind = 0;  // TileOpDev kinds 0, 1, 4, 5
  int sub = 0;   // kind 5
  int axis = 0;  // kind 4
  bool xswap = false;
  std::vector<int> targets, controls, ctrl_vals;
  int block = 0, lv = LV_BLOCK;
  std::vector<int> gates;
  int voff = 0;  // offset of its values
};

}  // namespace qsv

struct qsv_plan {
  int n = 0;
  qsv_dtype dtype = QSV_C128;
  int max_k = 2;
  bool heavy = false;  // commutation-aware merging (QSV_PLAN_HEAVY)
  bool nomerge = false;  // every gate its own block (values follow parameters one by one)
  int L = 12, b = 5;
  const qsv_circuit* circ = nullptr;  // borrowed structure snapshot below
  qsv_circuit circ_copy;
  std::vector<qsv::GateInfo> info;  // of circ_copy's gates
  std::vector<qsv::Block> blocks;
  std::vector<qsv::Lop> lops;  // the blocks as elementary ops
  int nvals = 0;               // host values of the lops
  struct Pass {
    std::vector<int> local;  // ascending local qubits (first b are 0..b-1)
    std::vector<int> ops;    // lop indices in execution order
  };
  std::vector<Pass> passes;
  // host copies of the device tables (uploaded on first apply)
  std::vector<int> pass_grid;  // workgroups that the device holds at once, per pass (first apply)
  std::vector<qsv::TilePassDev> h_pass;
  std::vector<qsv::TileOpDev> h_ops;
  qsv::SegBuild sb;
  int reg_bits = 0;  // > 0: passes run register-resident
  int thread_bits = qsv::kRegThreadBits;  // workgroup = 2^thread_bits threads
  int kmax_dense = 1;  // widest dense op (selects the kernel instantiation)
  // device buffers
  qsv::TilePassDev* d_pass = nullptr;
  qsv::TileOpDev* d_ops = nullptr;
  qsv::RegSegDev* d_segs = nullptr;
  qsv::RegOpDev* d_rops = nullptr;
  qsv::PhaseEntDev* d_ents = nullptr;
  qsv::RegHeadDev* d_heads = nullptr;
  void* d_pool = nullptr;  // uploaded once (circuit without parameters) or at each apply
  size_t pool_cap = 0;  // complex elements
  // pinned staging for per-apply uploads
  void* h_stage = nullptr;
  size_t stage_bytes = 0;
  hipEvent_t stage_ev = nullptr;
  qsv::AdjCache* adj = nullptr;  // reverse-sweep tables (first gradient with this plan)
  bool stage_used = false;
};

namespace qsv {
// Host-side plan of a circuit without merged gates (the caller deletes it), and
// its host values: the constant ones, and those that depend on parameters.
int plan_unmerged(const qsv_circuit* c, qsv_dtype dtype, qsv_plan** out);
void plan_free(qsv_plan* p);
void plan_symbolic(const qsv_plan* p, std::vector<cd>& vals, std::vector<DynVal>& dyn);
}  // namespace qsv

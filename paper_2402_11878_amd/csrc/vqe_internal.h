// Internal definitions shared by the host side (planner, Hamiltonian tables,
// C ABI) and the HIP kernels of the VQE library.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/vqe.h"

namespace vqe {

// ---------------------------------------------------------------- limits
constexpr int kMaxWindow = 7;     // qubits fused per pass (specialised kernels)
static_assert(kMaxWindow == VQE_MAX_WINDOW, "public and internal window limits differ");
constexpr int kInterpWindow = 5;  // qubits fused per pass by the interpreted kernels
constexpr int kMaxOps = 64;       // logical kernel ops per pass of an interpreted plan
constexpr int kMaxPhysOps = 160;  // ops per interpreted pass after inserting lane transposes
constexpr int kMaxMats = 32;      // 2x2 matrices per interpreted pass (kernel arguments)
constexpr int kMaxGradSlots = 24; // parameterised gates per pass (any plan)
constexpr int kInterpGradSlots = 16;  // ... of an interpreted pass (LDS accumulators)
constexpr int kBlock = 256;       // threads per block of every streaming kernel
constexpr int kMaxBlocks = 2048;  // grid-stride kernels use at most this many blocks
constexpr int kMaxPartBlocks = 1 << 17;  // blocks writing per-block partial sums
constexpr int kTileBits = 10;     // amplitudes per Hamiltonian tile = 2^kTileBits
constexpr int kTileMaxBits = 13;      // qubits of a tile pass (specialised kernels)
constexpr int kMaxPlanWindow = 13;  // largest window the planner forms (tile passes)

// Per-pass limits of the fusion planner.
struct PlanLimits {
    int kmax;   // window qubits
    int ops;    // logical ops (gates + gradient terms)
    int mats;   // gates carrying a 2x2 matrix
    int slots;  // distinct parameters (gradient slots)
};
// Interpreted kernels: ops and matrices travel as kernel arguments.
constexpr PlanLimits kInterpLimits = {kInterpWindow, kMaxOps, kMaxMats, kInterpGradSlots};
// Specialised kernels: ops are compiled in, matrices read from a device table,
// gradient slots accumulate in registers (2 VGPRs each in FP64).
constexpr PlanLimits kJitLimits = {kMaxWindow, 96, 64, kMaxGradSlots};

// ---------------------------------------------------------------- kernel ops
// A fused pass is a list of ops on the local bits 0..K-1 of a window.
enum OpType : uint8_t {
    OP_U2 = 0,    // general complex 2x2 on bit a, matrix mats[slot]
    OP_R2 = 1,    // real 2x2 on bit a (re parts of mats[slot])
    OP_DIAG = 2,  // diag(m00, m11) on bit a
    OP_CNOT = 3,  // control a, target b
    OP_CZ = 4,    // phase -1 where bits a and b are both set
    OP_XFLIP = 5, // Pauli X on bit a
    OP_GX = 6,    // gradient slot += Im<lam| X_a |psi>
    OP_GY = 7,    // gradient slot += Im<lam| Y_a |psi>
    OP_GZ = 8,    // gradient slot += Im<lam| Z_a |psi>
    OP_TPOSE = 9, // lane-split layout: swap the roles of register bit a and lane slot b
    // Excitation gates: rotation by mats[slot] = [[c, -s], [s, c]] between the
    // patterns A and B of a 2- or 4-bit subset (specialised kernels only).
    OP_PAIR2 = 10,  // A = {a = 1, b = 0}, B = {a = 0, b = 1}
    OP_PAIR4 = 11,  // A = {a = b = 1, c = d = 0}, B = {a = b = 0, c = d = 1}
    OP_GPAIR2 = 12, // gradient slot += Re<lam| K |psi>, K = |B><A| - |A><B| of OP_PAIR2
    OP_GPAIR4 = 13, // ... of OP_PAIR4
};

struct KOp {
    uint8_t type, a, b, slot;
    uint8_t c, d;  // third and fourth bit of OP_PAIR4 / OP_GPAIR4
    uint8_t pad[2];
};

// Bit subset and the A / B patterns of a pair op (over the op's local bits).
inline void pair_patterns(const KOp& k, uint32_t& mask, uint32_t& A, uint32_t& B) {
    if (k.type == OP_PAIR2 || k.type == OP_GPAIR2) {
        A = 1u << k.a;
        B = 1u << k.b;
    } else {
        A = (1u << k.a) | (1u << k.b);
        B = (1u << k.c) | (1u << k.d);
    }
    mask = A | B;
}

// Matrix of a 2x2 op: row-major entries u00 u01 u10 u11, each (re, im).
template <typename T>
struct Mat2 {
    T v[8];
};

template <typename T>
struct PassArgs {
    uint64_t n_cosets;      // 2^(n-K): one coset = the 2^K amplitudes of a window
    uint32_t K;
    uint32_t n_ops;
    uint32_t n_gslots;
    uint32_t split;            // lane-split bits S (0: every window bit in registers)
    uint32_t pos[kMaxWindow];  // window qubits, ascending
    // Lane-split layout: qubit held by physical slot s at load / at store
    // (slots 0..K-S-1 are register bits, K-S.. lane slots).
    uint32_t pos_in[kMaxWindow];
    uint32_t pos_out[kMaxWindow];
    KOp ops[kMaxPhysOps];
    Mat2<T> mats[kMaxMats];
};

// Arguments of a specialised (run-time compiled) window kernel; its ops are
// compiled in and its matrices come from a device table.
struct JitArgs {
    uint64_t n_cosets;
    uint32_t pos[kMaxWindow];      // window qubits, ascending
    uint32_t pos_in[kMaxWindow];   // qubit held by physical slot s at load
    uint32_t pos_out[kMaxWindow];  // ... and at store
};

// Lane-split bits S of a window pass: S of the K window bits live in lane bits
// 6-S .. 5, the other K-S in registers.  Specialised kernels keep
// K-S = 6 (complex64 forward), 5 (complex64 reverse, complex128 forward) or
// 4 (complex128 reverse): 128 VGPRs of state per thread.  Measured at 32
// qubits with 7-qubit windows, one more register bit (and one lane bit less)
// than a 64-VGPR state is 13-15% faster per evaluation: fewer lane
// transposes and longer contiguous runs per load outweigh the lower
// occupancy.  Interpreted kernels split 5-qubit windows only, to
// K-S = 5 / 4 / 4 / 3 (their op dispatch needs the smaller state).
inline int split_bits_for(bool jit, bool is_double, int K, bool two_vectors) {
    const int kl = (jit ? 6 : 5) - (is_double ? 1 : 0) - (two_vectors ? 1 : 0);
    if (!jit && K != kInterpWindow) return 0;
    return K > kl ? K - kl : 0;
}

// ---------------------------------------------------------------- Hamiltonian tables
// Terms grouped by x mask.  For group g, terms [begin, end) carry z masks and
// the coefficient c = w * (-i)^popcount(x&z) split as (cre, cim), so that
// (H psi)[b] = sum_g psi[b ^ x_g] * sum_t c_t (-1)^popcount(z_t & b).
struct GroupDesc {
    uint64_t x;
    uint32_t begin, end;
    uint32_t hbit;     // highest set bit of x (0 for x = 0)
    uint32_t pad;
};

template <typename T>
struct TermDesc {
    uint64_t z;
    T cre, cim;
};

// ---------------------------------------------------------------- launchers (kernels.hip)
hipError_t launch_set_basis(int dtype, void* psi, uint64_t dim, uint64_t b, hipStream_t st);
hipError_t launch_zero(double* p, uint64_t n, hipStream_t st);
hipError_t launch_copy(int dtype, const void* src, void* dst, uint64_t dim, hipStream_t st);

// Interpreted window passes (K <= kInterpWindow).  in == out allowed (in
// place).  n = qubits of the state.
template <typename T>
hipError_t launch_window_fwd(const PassArgs<T>& a, int n, const void* in, void* out, hipStream_t st);

// Reverse pass on (psi, lam); writes per-block gradient partials
// [blocks][n_gslots] into gpart.  Returns the block count used via *nblocks.
template <typename T>
hipError_t launch_window_rev(const PassArgs<T>& a, int n, const void* psi_in, void* psi_out,
                             const void* lam_in, void* lam_out, double* gpart,
                             uint32_t* nblocks, hipStream_t st);

// Specialised kernel launch (fn = hipFunction_t of the pass, see jit.cpp):
// S lane-split bits, mats = this pass's matrix table on the device; reverse
// passes use the persistent grid; *nblocks = blocks used.
hipError_t launch_window_jit(void* fn, const JitArgs& a, int S, const void* mats, bool reverse, const void* in0,
                             void* out0, const void* in1, void* out1, double* gpart, uint32_t* nblocks,
                             hipStream_t st);


// ---------------------------------------------------------------- specialised kernels (jit.cpp)
int jit_mode();
int jit_set_mode(int mode);
// Kernel symbol of a generated pass: vqe_window_{fwd,rev}_{c64,c128}.
const char* jit_kernel_name(int NV, bool dbl);
// HIP source of the specialised kernel of one pass: K window bits, S lane-split
// bits, NV = 1 (forward) or 2 (reverse, psi and lam), ops on physical slots.
std::string jit_source(bool dbl, int K, int S, int NV, const std::vector<KOp>& ops, uint32_t n_gslots);
// Compiles (in parallel) and loads on the current device every source not yet
// cached; fns[i] = kernel of srcs[i] (nullptr for an empty source).
int jit_prepare(const std::vector<std::string>& srcs, std::vector<void*>& fns, std::string& err);
size_t jit_cached();

// ---------------------------------------------------------------- H psi by window passes
// lam = H psi as a few passes over qubit windows of kHwBits qubits that all
// contain qubits 0 .. kHwLow-1 (contiguous runs per load): every X group lies
// in one window, a pass stages each coset (the 2^kHwBits amplitudes that
// differ only in the window bits) of psi in LDS and adds the contributions of
// its groups to lam (written by the first pass, read-modify-written by the
// others); the last pass also reduces (Re<psi|lam>, <psi|psi>).
//
// Window-local pattern j = t + 2^kHwThreadBits r: thread t of a block holds
// the patterns of all r < 2^(kHwBits - kHwThreadBits).  For a group x,
//   D_x(b) = sum_z c_z (-1)^{z.b} = sum_{zl} (-1)^{zl.j} A_{x,zl}(coset),
//   A_{x,zl} = sum_{z: z & window = zl} c_z (-1)^{(z & ~window).base},
// so the terms of a group with equal in-window z bits form one class whose
// coefficient A is uniform over a coset (computed once per coset); the sign
// (-1)^{zl.j} splits into a thread part (zl bits below kHwThreadBits) and a
// register part, and the classes of a group are sorted into buckets by the
// register part, whose 2^(kHwBits - kHwThreadBits) bucket sums give D for
// every r through one Walsh-Hadamard transform.
// 13-qubit windows measured faster than 12 on both 32-qubit workloads (Hubbard
// 4 passes instead of 5, molecule-shaped 21 instead of 26) at the same 16 waves
// per CU (one 1024-thread block with a 128 KiB complex128 coset in LDS).
constexpr int kHwBits = 13;
static_assert(kHwBits == VQE_HPSI_WINDOW_QUBITS, "public and internal window sizes differ");
constexpr int kHwLow = 3;
constexpr int kHwThreadBits = 10;       // 1024 threads per block
constexpr int kHwRegBits = kHwBits - kHwThreadBits;
constexpr int kHwMaxClasses = 512;      // classes per pass (their coefficients are staged in LDS)

struct HwDesc {
    uint32_t pos[kHwBits];    // window qubits, ascending
    uint32_t g_begin, g_end;  // this pass's groups in the group table
    uint32_t c_begin, c_end;  // this pass's classes in the class table (at most kHwMaxClasses)
};

struct HwGroup {
    uint32_t xl;                       // x mask in window-local bits
    uint32_t cb[(1 << kHwRegBits) + 1];  // bucket u (register-part z bits = u): classes [cb[u], cb[u + 1])
    uint32_t zrm;                      // OR of the register-part z bits of its classes (empty buckets outside it)
    uint32_t pad;
};

struct HwClass {
    uint32_t zt;              // in-window z bits on the thread part (window-local bits below kHwThreadBits)
    uint32_t k_begin, k_end;  // its terms in the term table
    uint32_t pad;
};

template <typename T>
struct HwTerm {
    uint64_t zo;  // z bits outside the window (parity from the coset base)
    T cre, cim;   // folded coefficient, as in TermDesc
};

// One window pass; returns the block count (partials of the last pass).
// lam == nullptr: energy-only pass (no lam traffic); its partials hold this
// pass's share of Re<psi|H psi> and, for the first pass, <psi|psi>.
// real: every folded coefficient has a zero imaginary part (the real form
// of the pass, half the arithmetic).
template <typename T>
hipError_t launch_hwin(int n, const HwDesc& w, const void* psi, void* lam, const HwGroup* groups,
                       const HwClass* classes, const HwTerm<T>* terms, bool real, bool first, bool last,
                       double* part, uint32_t* nblocks, hipStream_t st);

// One window pass of lam = H psi for one item of a batch of mid-size
// states (one launch covers the pass of every item): blocks [blk_begin,
// blk_begin + n_blk) of the launch; after the item's last pass block blk
// writes its energy and norm partials to part[part_off + blk] and
// part[part_off + n_blk + blk].
struct HwItem {
    HwDesc w;
    const void* psi;
    void* lam;
    const HwGroup* groups;
    const HwClass* classes;
    const void* terms;  // HwTerm<T>
    uint64_t n_cosets, part_off;
    uint32_t blk_begin, n_blk, first, last;
};
template <typename T>
hipError_t launch_hwin_batch(const HwItem* d, uint32_t n_desc, uint32_t grid, bool real, double* part,
                             hipStream_t st);

// ---------------------------------------------------------------- dense window by MFMA
// psi' = U psi on kDenseK qubits, all >= 4 (16 consecutive cosets are 16
// consecutive amplitudes), U given to the kernel as the real 2^(k+1) square
// matrix [[Re U, -Im U], [Im U, Re U]] in row-major order, rows = output
// pattern (bit i of a pattern is qubit q[i]).  In place allowed.
constexpr int kDenseK = 5;

struct DenseArgs {
    uint64_t n_tiles;           // 2^(n - kDenseK) / 16
    uint32_t q[kDenseK];        // window qubits in pattern-bit order
    uint32_t sorted[kDenseK];   // the same, ascending
};

template <typename T>
hipError_t launch_dense(const DenseArgs& a, const T* ur, const void* in, void* out, hipStream_t st);

// H psi tile kernel.  mode 0: lam = H psi and (Re<psi|lam>, <psi|psi>) partials.
// mode 1: energy partials only, off-tile groups visited once per pair.  At
// most max_blocks blocks (each owns a contiguous run of tiles), each writing
// two partials.
template <typename T>
hipError_t launch_hpsi(int n, const void* psi, void* lam, const GroupDesc* groups, uint32_t n_groups,
                       const TermDesc<T>* terms, int mode, uint32_t max_blocks, double* part, uint32_t* nblocks,
                       hipStream_t st);
// Blocks that launch_hpsi uses at n qubits under max_blocks, and that a
// window pass of H psi (launch_hwin) uses at n qubits.
uint32_t hpsi_blocks(int n, uint32_t max_blocks);
uint32_t hwin_blocks(int n);
// Grouped energy-only sweeps (vqe_expect_pauli and its no-allocation form)
// launch at most this many blocks: one block count, hence one reduction
// order, for both.
constexpr uint32_t kEnergyPartBlocks = 4096;

// out[0] = sums[0] / sums[1], out[1] = sums[1] (one thread; device memory).
hipError_t launch_energy_ratio(const double* sums, double* out, hipStream_t st);

// One term: partials of Re<psi|P(x,z)|psi> (pair-halved) and <psi|psi>.
template <typename T>
hipError_t launch_expect_term(int n, const void* psi, uint64_t x, uint64_t z, double* part,
                              uint32_t* nblocks, hipStream_t st);

// out[map ? map[s] : s] = (accumulate 0), += (1) or -= (-1) the sum over blocks
// of part[block][s], fixed order, FP64.
hipError_t launch_reduce(const double* part, uint32_t nblocks, uint32_t nslots,
                         const int32_t* map, double* out, int accumulate, hipStream_t st);

// ---------------------------------------------------------------- planner (plan.cpp)
struct Gate {
    int kind, q0, q1, pidx;
    double angle;
    int q2 = 0, q3 = 0;  // DEXC only
};

// Qubits of a gate (1, 2 or 4); returns the count.
inline int gate_qubits(const Gate& g, int q[4]) {
    q[0] = g.q0;
    switch (g.kind) {
        case VQE_GATE_CNOT:
        case VQE_GATE_CZ:
        case VQE_GATE_SEXC:
            q[1] = g.q1;
            return 2;
        case VQE_GATE_DEXC:
            q[1] = g.q1;
            q[2] = g.q2;
            q[3] = g.q3;
            return 4;
        default:
            return 1;
    }
}

struct PlannedPass {
    int K = 0;
    int pos[kMaxPlanWindow] = {0};
    std::vector<int> gates;      // indices into the circuit's gate list, execution order
};

// Partition gates into fused passes.  Returns false (with msg) on failure.
// lim.kmax = largest window (<= kMaxPlanWindow).
bool plan_passes(int n, const std::vector<Gate>& gates, const PlanLimits& lim, std::vector<PlannedPass>& out,
                 std::string& msg);

// Tile passes: windows of `bits` qubits that all contain qubits 0 .. low-1
// (contiguous runs of 2^low amplitudes per load).  Unlike plan_passes, a
// pass keeps its whole window in pos[0 .. K-1], also qubits no gate touches.
struct TileLimits {
    int bits, low;
    int gates;   // gates per pass (code size of its kernel)
    int pushes;  // parameterised gates per pass
    int width = 48;  // states of the beam search
};
bool plan_tiles(int n, const std::vector<Gate>& gates, const TileLimits& lim, std::vector<PlannedPass>& out,
                std::string& msg);

// ---------------------------------------------------------------- tile passes (tile.cpp)
// One pass over a window of T = 12 or 13 qubits: a block of 256 threads holds
// a coset (2^T amplitudes of psi, in reverse passes of lam too) in registers,
// 2^R amplitudes per thread and vector, reads and writes the state once and
// applies all gates of the window, in stages that each keep another R of the
// T window bits in registers; the vectors change layout between stages
// through LDS.  The amplitudes of a wave's access are runs of 128 bytes (64 in the
// 12-qubit tiles of complex64): the 2^low lowest ones are in every window.
struct TileShape {
    int T, R, low;
};
// n < kTileBigQubits: smaller complex64 tiles, so that a 20-qubit state still
// fills the 256 CUs.
constexpr int kTileMinQubits = 14;
constexpr int kTileBigQubits = 23;
inline TileShape tile_shape(bool dbl, int n) {
    if (dbl) return {12, 4, 3};
    return n >= kTileBigQubits ? TileShape{13, 5, 4} : TileShape{12, 4, 3};
}
constexpr int kTileThreads = 256;
constexpr int kTileMaxGates = 256;   // gates per pass (code size)
constexpr int kTileFlagBytes = kTileMaxGates / 8;
constexpr int kTileMaxPushes = 128;  // gradient terms per pass: two per lane of a wave

// Host numbers of one pass's table: for every entry what to compute from the
// angles of an evaluation (see fill_tile_table).
enum TileFill : uint8_t {
    TF_ROT,    // t of an unnormalised rotation, and a flag: a half turn (x, y) -> (-y, x) comes first
    TF_PHASE,  // 2^m phases (re, im) of the merged diagonal gates on m bits, times the pending scale
    TF_SCALE,  // the pending scale alone
    TF_R2,     // a real 2x2 matrix (H, excitations): u00 u01 u10 u11
};
struct TileEntry {
    TileFill kind;
    uint32_t off;                // first scalar in the pass's table
    int gate = -1;               // TF_ROT, TF_R2
    uint32_t flag_word = 0, flag_bit = 0;  // TF_ROT: the flag, in the table as 32-bit words
    uint32_t any_word = 0, any = 0;        // ... and a word with bits to be set if it is
    uint32_t mask = 0;           // TF_PHASE: register bits of its index, ascending
    std::vector<int> diag;       // TF_PHASE: the merged RZ / CZ gates
    std::vector<uint32_t> diag_bits;  // ... and their register bits
    std::vector<int> rots;       // TF_PHASE, TF_SCALE: rotations whose norms are folded in
};
struct TileKernel {
    std::string src;
    std::vector<TileEntry> entries;
    uint32_t n_scalars = 0;
    uint32_t n_flags = 0;        // flags of half turns at the front of the table
    std::vector<int32_t> lane_param;  // reverse: parameter summed by column l of the partials (-1: none)
};
// Generates the kernel of one pass (dir 0 forward, 1 reverse).  Returns false
// with msg on failure.
bool tile_kernel(bool dbl, const TileShape& sh, const std::vector<Gate>& gates, const PlannedPass& p, int dir,
                 TileKernel& out, std::string& msg);
const char* tile_kernel_name(int NV, bool dbl);
// cos and sin of half the angle of every gate.
struct HalfAngle {
    double c, s;
};
// Largest tan(a/2) that an unnormalised rotation may have in an evaluation
// whose vectors have 2-norms up to `norm`: while max_pending() of them wait for
// their factors a vector grows by that much to the power of their number, which
// must leave the type's range (2^120, 2^1000) to the vector itself.  Rotations
// beyond it, by angles next to an odd multiple of pi, make a half turn by moves
// first.  Ordinary weights leave 2^27 and more.  With one limit of 2^26 for all,
// |lam| of 2^24 overflowed in complex64; with one of 4, every sixth angle took the
// half turn, whose moves cost about what the rotation does: 28 qubits complex64
// 49.9 ms against 46.7.
double turn_limit(bool dbl, double norm);
// Fills the table of one pass for the angles of an evaluation.
template <typename T>
void fill_tile_table(const TileKernel& k, const std::vector<Gate>& gates, const HalfAngle* h, double limit, int dir,
                     T* tab);

// ---------------------------------------------------------------- batch programs (program.cpp, batch.hip)
// A tile of 2^bits amplitudes in LDS, kProgBits of its bits in registers at a
// time: 2^(bits - 4) threads with 16 amplitudes (per vector) each.
constexpr int kProgBits = 4;
// A stage is one of three kinds of records.
//   rows   straight-line, no branch: what a layer of RY, diagonal gates and
//          CNOTs along the register bits needs, in the order the scheduler
//          emits it (absent parts act as the identity)
//            forward   turns, phases, CNOTs 0-1, 1-2, 2-3
//            reverse   CNOTs 2-3, 1-2, 0-1, phases, Z terms, Y terms, turns
//   pairs  excitations, applied where their amplitudes lie in LDS
//   misc   everything else, one op per record
enum ProgKind : uint32_t { PK_ROWS, PK_PAIRS, PK_MISC };
constexpr uint32_t kRowHalf = 1u << 20;
template <typename T>
struct ProgRow {
    uint32_t flags;          // bit k < 3: CNOT of control k, target k + 1; bit 4: it has more; Z mask << 8; Y mask << 12;
                             // bit 16 + k: a half turn before the turn of bit k; kRowHalf in a stage's first row: one of its
                             // rows has such a bit (both filled in with the numbers)
    uint32_t z_slot, z_off;  // gradient slot of the Z term of bit k: z_slot + byte k of z_off
    uint32_t y_slot, y_off;
    uint32_t pad[3];
    T t[4];                  // RY on bit k: x - t y, y + t x
    T ph[32];                // phase (re, im) of every register entry
};
template <typename T>
struct ProgMisc {
    uint32_t code;  // type | bit << 8; PM_PERM: control << 2 | target of a CNOT, or 5 x bit: X; bit 31: PM_ROTX after a half turn
    uint32_t slot, pad[2];
    T t[4];
};
enum ProgMiscType : uint32_t {
    PM_ROTX,   // x - i t y, y - i t x, t = t[0]
    PM_R2,     // real matrix t[0..3]
    PM_PERM,
    PM_GX,     // gradient slot: Im<lam|X|psi>
};
// An excitation: a real matrix between the tile patterns x & 0xffff and x >> 16.
template <typename T>
struct ProgPair {
    uint32_t x, slot, grad, pad;  // grad = 1: first its gradient term to `slot`
    T s[4];
};
// A stage's block in the program's stream: the header of the next stage, then
// this one's records.
struct ProgStage {
    uint8_t pos[kProgBits];  // register bits, ascending tile bits
    uint16_t kind;           // ProgKind
    uint16_t n_ops;          // records
    uint32_t off, bytes;     // in the stream, multiples of 16
};
static_assert(sizeof(ProgStage) == 16, "four words");
constexpr uint32_t kProgBlock = 6144;  // longest block (two of them in LDS: one in use, one arriving)
struct Program {
    std::vector<ProgStage> stages;
    std::vector<uint32_t> stream;    // the blocks, numbers still zero
    TileKernel table;                // its entries: scalar offsets into the stream
    std::vector<int32_t> slot_param; // reverse: parameter of every gradient slot
    // stages emitted up to the end of every planned group: a checkpoint may
    // stand there, unless a later group's ops joined the last stage (~0u)
    std::vector<uint32_t> mark;
};
inline bool is_excitation_kind(int kind) { return kind == VQE_GATE_SEXC || kind == VQE_GATE_DEXC; }
// The gates `list` on a tile of `bits` bits, local[q] = tile bit of qubit q,
// grouped into stages (one plan for both directions: planning takes longer than
// building, and a circuit's first evaluation waits for it).
struct ProgramPlan {
    std::vector<Gate> gates;  // on tile bits
    std::vector<int> list;
    std::vector<PlannedPass> stages;
};
bool plan_program(int bits, const std::vector<Gate>& gates, const std::vector<int>& list, const int* local,
                  ProgramPlan& out, std::string& msg);
// Program of a plan (dir 0 forward, or 1: un-applied in reverse with the
// gradient terms).  flush: pending factors are applied at the end of every
// planned group, so that the tile holds the state there.
bool build_program(bool dbl, int bits, const std::vector<Gate>& gates, const ProgramPlan& plan, int dir, bool flush,
                   Program& out, std::string& msg);

// A small Hamiltonian as a stream of blocks of at most kProgBlock bytes, each
// of groups: a header, then its terms.  A group's terms are sorted by their z
// bits on the register part of the index (the kProgBits highest tile bits):
// count[u] of them (a byte each) have the bits u.
struct alignas(8) SmallGroup {
    uint32_t x, n_terms, pad[2];
    uint32_t count[4];
};
template <typename T>
struct SmallTerm {
    uint32_t zt, zr;  // z bits on the thread and on the register part
    T cre, cim;
};
struct SmallBlock {
    uint32_t off, bytes, n_groups, pad;
};

struct TileArgs {
    uint64_t n_units;              // cosets of the window
    uint32_t pos[kTileMaxBits];    // window qubits, ascending
    uint32_t first;                // forward: stage |0...0> instead of reading the state
};
// L: columns per block of the gradient partials gpart (reverse passes).
hipError_t launch_tile(void* fn, const TileArgs& a, bool reverse, const void* tab, const void* in0, void* out0,
                       const void* in1, void* out1, double* gpart, uint32_t L, hipStream_t st);
// Blocks of a tile pass over `units` cosets.
uint32_t tile_blocks(uint64_t units, bool reverse);
// out[p L + l] = sum over blocks b < nblocks of part[(p nblocks + b) L + l], p < n_pass, in a fixed order.
hipError_t launch_tile_reduce(const double* part, uint32_t n_pass, uint32_t nblocks, uint32_t L, double* out,
                              hipStream_t st);

// ---------------------------------------------------------------- batched small states (batch.hip)
constexpr int kBatchMaxQubitsC64 = 13;
constexpr int kBatchMaxQubitsC128 = 12;
constexpr int kBatchLdsBytes = 128 * 1024 + 2 * (int)kProgBlock;  // psi + lam + two program blocks in LDS
// Smaller states run as this many bits (a full wave of 16 amplitudes per
// thread), the qubits above n idle in |0>.
constexpr int kBatchMinBits = 10;
inline int batch_bits(int n) { return n < kBatchMinBits ? kBatchMinBits : n; }

// A checkpoint of a small state: psi is kept in buf after the forward stages
// [0, fwd_end) and restored after the reverse stages [0, rev_end).
struct BatchCkpt {
    void* buf;
    uint32_t fwd_end, rev_end;
};

template <typename T>
struct BatchDesc {
    int32_t n, bits;
    uint32_t n_fwd, n_rev;      // stages
    uint32_t n_blocks, n_slots;
    uint32_t real;              // every folded coefficient is real
    uint32_t n_ckpt;
    const BatchCkpt* ckpt;      // in forward order
    const ProgStage* fwd;
    const ProgStage* rev;
    const char* fwd_stream;     // this evaluation's
    const char* rev_stream;
    const SmallBlock* ham;      // the Hamiltonian's blocks
    const char* ham_stream;
    double* out;                // energy, norm, then the gradient sums by slot
    double* part;               // n_slots x 8 doubles: sums per wave
    void* psi_out;              // where the state ends up (nullptr: nowhere)
    void* lam_out;
};

template <typename T>
hipError_t launch_batch(const BatchDesc<T>* items, uint32_t n_items, int max_bits, hipStream_t st);
hipError_t batch_set_lds_limit();

// ---------------------------------------------------------------- batched mid-size states (batch.hip)
// Items above the LDS limit, up to kMidMaxQubits: psi and lam stay in device
// memory (held in the last-level cache between passes at the small end), and
// one launch applies one fused pass of every item of the batch.  A pass is a
// window of kMidWin qubits that holds the kMidLow lowest ones (plan_tiles); a
// block stages a coset of 2^kMidWin amplitudes in LDS, runs the pass's program
// there and writes it back.
constexpr int kMidWin = 12;
// States of the plan's beam search, of 4 to 16 layers: 4 find the passes that 48 do
// up to 20 qubits, but for 18 and 19 qubits x 8 layers (5 against 4), in a tenth of
// the time (19 x 16 0.3 against 2.4 ms, which a first evaluation waits for); above
// they find one or two more (24 x 8 8 against 6, 24 x 16 12 against 11; the 10-qubit
// windows of a greedy plan 9 and 16).
constexpr int kMidPlanWidth = 4;
constexpr int kMidLow = 2;
constexpr int kMidMaxQubits = 24;
constexpr int kMidMaxSlots = 128;         // parameterised gates per pass
constexpr uint32_t kMidMaxBlocks = 1024;  // blocks per item and launch
static_assert(kMidWin <= kMaxPlanWindow, "planner window");
static_assert(kMidMaxQubits == VQE_BATCH_MAX_QUBITS_MID, "public and internal mid-size limits differ");

// One item's pass in one launch.  Blocks [blk_begin, blk_begin + n_blk) of
// the launch take cosets blk, blk + n_blk, ...; in a reverse pass block blk
// writes gradient slot s of the pass to part[part_off + s n_blk + blk].
struct MidPass {
    void* psi;
    void* lam;
    const ProgStage* stages;
    const char* stream;
    uint64_t n_cosets;
    uint64_t part_off;
    uint32_t pos[kMidWin];  // window qubits, ascending
    uint32_t n_stages, n_slots;
    uint32_t blk_begin, n_blk;
    uint32_t first;         // forward pass 0: stage |0...0> instead of reading psi
    uint32_t pad;
};

// lam = H psi of one item over tiles of 2^kMidTileBits amplitudes; block blk
// writes its energy and norm partials to part[part_off + blk] and
// part[part_off + n_blk + blk].
constexpr int kMidTileBits = 10;
struct MidHam {
    const void* psi;
    void* lam;
    const GroupDesc* groups;
    const void* terms;      // TermDesc<T>
    uint64_t n_tiles;
    uint64_t part_off;
    uint32_t n_groups, blk_begin, n_blk, pad;
};

// out[k] = sum of part[part_off .. part_off + count) in a fixed order.
struct MidRed {
    uint64_t part_off;
    uint32_t count, pad;
};

template <typename T>
hipError_t launch_mid_pass(const MidPass* d, uint32_t n_desc, uint32_t grid, bool rev, double* part, hipStream_t st);
template <typename T>
hipError_t launch_mid_hpsi(const MidHam* d, uint32_t n_desc, uint32_t grid, double* part, hipStream_t st);
hipError_t launch_mid_reduce(const MidRed* r, uint32_t n, const double* part, double* out, hipStream_t st);

// ---------------------------------------------------------------- errors
void set_error(const std::string& m);

}  // namespace vqe

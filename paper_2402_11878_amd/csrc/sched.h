// Order of the ops of one stage: a few window bits of a pass held in
// registers, gates applied there one after the other.  Shared by the generator
// of the specialised tile kernels (tile.cpp), which emits source, and by the
// builder of batch programs (program.cpp), which emits op codes.
#pragma once

#include "vqe_internal.h"

namespace vqe {

enum OpKind { K_GRAD, K_ROTY, K_ROTX, K_R2, K_CNOT, K_FLIP, K_DIAG };

// One gate (or its gradient term) on the register bits of a stage.  On each of
// its bits it acts like Z (diagonal), like X, like Y, or otherwise; two ops
// commute if on every shared bit both act like the same Pauli.
struct StageOp {
    OpKind kind;
    int gate;    // index into the circuit's gate list
    int bit[4];  // register bits of its qubits
    uint32_t z = 0, x = 0, y = 0, other = 0;
};

inline bool commute(const StageOp& a, const StageOp& b) {
    const uint32_t ma = a.z | a.x | a.y | a.other, mb = b.z | b.x | b.y | b.other, shared = ma & mb;
    return (shared & ~((a.z & b.z) | (a.x & b.x) | (a.y & b.y))) == 0;
}

inline bool is_rot(OpKind k) { return k == K_ROTY || k == K_ROTX; }

// Stage op of gate g (or of its gradient term) on the given register bits.
inline StageOp stage_op(const Gate& g, int gate, const int* bits, bool grad) {
    StageOp k{};
    k.gate = gate;
    int q[4];
    const int nq = gate_qubits(g, q);
    uint32_t all = 0;
    for (int i = 0; i < nq; ++i) {
        k.bit[i] = bits[i];
        all |= 1u << bits[i];
    }
    switch (g.kind) {
        case VQE_GATE_RY: k.kind = K_ROTY; k.y = all; break;
        case VQE_GATE_RX: k.kind = K_ROTX; k.x = all; break;
        case VQE_GATE_RZ: k.kind = K_DIAG; k.z = all; break;
        case VQE_GATE_CZ: k.kind = K_DIAG; k.z = all; break;
        case VQE_GATE_X: k.kind = K_FLIP; k.x = all; break;
        case VQE_GATE_CNOT:
            k.kind = K_CNOT;
            k.z = 1u << k.bit[0];
            k.x = 1u << k.bit[1];
            break;
        case VQE_GATE_SEXC:
        case VQE_GATE_DEXC:
        default: k.kind = K_R2; k.other = all; break;  // excitations, H
    }
    if (grad) k.kind = K_GRAD;
    return k;
}

// Patterns between which an op acts: bit clear / set, or the A and B of an excitation.
inline void stage_pattern(const Gate& g, const StageOp& k, uint32_t& mask, uint32_t& A, uint32_t& B) {
    if (g.kind == VQE_GATE_SEXC) {
        A = 1u << k.bit[0];
        B = 1u << k.bit[1];
    } else if (g.kind == VQE_GATE_DEXC) {
        A = (1u << k.bit[0]) | (1u << k.bit[1]);
        B = (1u << k.bit[2]) | (1u << k.bit[3]);
    } else {
        A = 0;
        B = 1u << k.bit[0];
    }
    mask = A | B;
}

// Rotations that may wait for their factors at a time (turn_limit()).
inline int max_pending(bool dbl) { return dbl ? 14 : 4; }

struct StageScheduler {
    bool dbl = false;
    const std::vector<Gate>* gates = nullptr;
    TileKernel* out = nullptr;
    std::vector<int> pending;  // rotations whose factor is still to be applied

    virtual ~StageScheduler() = default;
    virtual void rot(const StageOp& k) = 0;                          // unnormalised RY / RX
    virtual void scale_by(uint32_t off) = 0;                         // every amplitude times tab[off]
    virtual void phase_by(uint32_t off, uint32_t mask) = 0;          // times the phase of its bits in mask
    virtual void matrix(const StageOp& k) = 0;                       // real 2x2 between two patterns
    virtual void rename(const StageOp& k) = 0;                       // CNOT, X
    virtual void gradient(const StageOp& k) = 0;                     // X, Y or excitation term
    virtual void gradient_z(const std::vector<StageOp>& ops) = 0;    // Z terms
    virtual uint32_t table_mask(uint32_t used) const { return used; } // bits a phase table is made for

    // Reserves `scalars` table entries; returns where they lie (or a handle of them).
    virtual uint32_t entry(TileEntry e, uint32_t scalars) {
        e.off = out->n_scalars;
        out->n_scalars += scalars;
        out->entries.push_back(std::move(e));
        return out->entries.back().off;
    }
    uint32_t gate_entry(TileFill kind, int gate, uint32_t scalars) {
        TileEntry e;
        e.kind = kind;
        e.gate = gate;
        return entry(std::move(e), scalars);
    }

    // Applies the pending factors.
    void scale() {
        if (pending.empty()) return;
        TileEntry e;
        e.kind = TF_SCALE;
        e.rots.swap(pending);
        scale_by(entry(std::move(e), 1));
    }

    // The diagonal gates `ops` as one phase per value of their bits, pending factors included.
    void phase(const std::vector<StageOp>& ops) {
        TileEntry e;
        e.kind = TF_PHASE;
        for (const StageOp& k : ops) {
            e.diag.push_back(k.gate);
            e.diag_bits.push_back(k.z);
            e.mask |= k.z;
        }
        e.rots.swap(pending);
        e.mask = table_mask(e.mask);
        const uint32_t mask = e.mask;
        phase_by(entry(std::move(e), 2u << __builtin_popcount(mask)), mask);
    }

    // Emits the ops of a stage in an order that respects every pair that does
    // not commute: gradient terms and register renames as soon as they are
    // ready, then rotations, diagonal gates last (so that they merge).
    // Gradient terms read normalised vectors (pending factors applied first).
    void stage(std::vector<StageOp> ops) {
        const size_t most = (size_t)max_pending(dbl);
        auto ready = [&](size_t i) {
            for (size_t j = 0; j < i; ++j)
                if (!commute(ops[j], ops[i])) return false;
            return true;
        };
        auto z_term = [&](const StageOp& k) { return k.kind == K_GRAD && (*gates)[k.gate].kind == VQE_GATE_RZ; };
        auto is_diag = [&](const StageOp& k) { return k.kind == K_DIAG || z_term(k); };
        while (!ops.empty()) {
            bool progress = false;
            for (size_t i = 0; i < ops.size();) {
                const StageOp& k = ops[i];
                if (is_diag(k) || is_rot(k.kind) || (k.kind == K_GRAD && !pending.empty()) || !ready(i)) {
                    ++i;
                    continue;
                }
                if (k.kind == K_GRAD) gradient(k);
                else if (k.kind == K_CNOT || k.kind == K_FLIP) rename(k);
                else matrix(k);
                ops.erase(ops.begin() + (long)i);
                progress = true;
                i = 0;
            }
            if (ops.empty()) break;
            for (size_t i = 0; i < ops.size();) {
                if (is_rot(ops[i].kind) && pending.size() < most && ready(i)) {
                    rot(ops[i]);
                    ops.erase(ops.begin() + (long)i);
                    progress = true;
                } else {
                    ++i;
                }
            }
            if (progress) continue;
            std::vector<StageOp> diag, zt;
            for (size_t i = 0; i < ops.size();) {
                if (is_diag(ops[i]) && ready(i)) {
                    (z_term(ops[i]) ? zt : diag).push_back(ops[i]);
                    ops.erase(ops.begin() + (long)i);
                } else {
                    ++i;
                }
            }
            if (!diag.empty()) phase(diag);
            if (!zt.empty()) {
                scale();
                gradient_z(zt);
            }
            if (diag.empty() && zt.empty()) scale();  // a gradient term or a rotation waits for the factors
        }
    }

};

}  // namespace vqe

// Batch programs: the gates of a tile (a whole small state, or one pass over a
// window of a mid-size one) as stages and op codes for the interpreter of
// batch.hip.  A stage keeps kProgBits of the tile's bits in registers; its ops
// are ordered and merged by the same scheduler as the specialised tile
// kernels (unnormalised rotations, phase tables, one product for the Z terms).
#include <algorithm>
#include <cstring>

#include "sched.h"

namespace vqe {
namespace {

struct Builder : StageScheduler {
    Program* prog = nullptr;
    int dir = 0;
    // One record of the stage being built: its header words and the table entries of its numbers.
    struct Rec {
        uint32_t w[8] = {0};
        int num[4] = {-1, -1, -1, -1};  // entry that fills t[k] (t[0 ..] for entries of several numbers)
        int phase = -1;                 // entry of the row's phases
    };
    std::vector<Rec> recs;
    ProgStage cur{};
    int part = -1;  // last part of the open row, -1: the next op starts a row
    std::vector<std::pair<int, uint32_t>> pair_slot;  // excitations whose gradient term is due: (gate, slot)

    // Order of the parts in a row: CNOT b -> b + 1 is a part of its own, as they run one after the other.
    int p_rot() const { return dir ? 6 : 0; }
    int p_phase() const { return dir ? 3 : 1; }
    int p_cnot(int b) const { return dir ? 2 - b : 2 + b; }
    static constexpr int kZ = 4, kY = 5;

    uint32_t scalar() const { return dbl ? 8 : 4; }
    uint32_t head(uint32_t kind) const { return kind == PK_ROWS ? 32 : 16; }
    uint32_t rec(uint32_t kind) const { return head(kind) + (kind == PK_ROWS ? 36 : 4) * scalar(); }

    uint32_t entry(TileEntry e, uint32_t) override {
        out->entries.push_back(std::move(e));
        return (uint32_t)out->entries.size() - 1;
    }

    void open(const uint8_t* pos) {
        for (int i = 0; i < kProgBits; ++i) cur.pos[i] = pos[i];
        part = -1;
    }

    // Ends the stage: lays out its block and tells its entries where their numbers lie.
    void close() {
        part = -1;
        if (recs.empty()) return;
        const uint32_t n = (uint32_t)recs.size(), size = rec(cur.kind), hd = head(cur.kind);
        std::vector<ProgStage>& st = prog->stages;
        uint32_t at = 0;
        const bool join = cur.kind == PK_PAIRS && !st.empty() && st.back().kind == PK_PAIRS &&
                          st.back().bytes + n * size <= kProgBlock;
        if (join) {  // excitations have no register bits: they may follow the ones before
            at = st.back().n_ops;
            for (uint32_t& m : prog->mark)
                if (m == st.size()) m = ~0u;
        } else {
            cur.off = (uint32_t)prog->stream.size() * 4;
            st.push_back(cur);
        }
        ProgStage& s = st.back();
        s.n_ops = (uint16_t)(at + n);
        s.bytes = 16 + (at + n) * size;
        prog->stream.resize((s.off + s.bytes) / 4, 0);
        for (uint32_t i = 0; i < n; ++i) {
            const Rec& r = recs[i];
            const uint32_t where = s.off + 16 + (at + i) * size, num = where + hd;
            std::copy(r.w, r.w + hd / 4, &prog->stream[where / 4]);
            for (int k = 0; k < 4; ++k) {
                if (r.num[k] < 0) continue;
                TileEntry& e = out->entries[r.num[k]];
                e.off = num / scalar() + (uint32_t)k;
                if (e.kind != TF_ROT) continue;
                e.flag_word = where / 4;
                e.flag_bit = cur.kind == PK_ROWS ? 16 + (uint32_t)k : 31;
                e.any_word = (s.off + 16) / 4;
                e.any = cur.kind == PK_ROWS ? kRowHalf : 0;
            }
            if (cur.kind != PK_ROWS) continue;
            if (r.phase >= 0) out->entries[r.phase].off = num / scalar() + 4;
            for (uint32_t p = 0; p < 16; ++p) {  // no phases: ones
                uint32_t* one = &prog->stream[num / 4 + (4 + 2 * p) * scalar() / 4];
                if (dbl) one[1] = 0x3ff00000u;
                else one[0] = 0x3f800000u;
            }
        }
        recs.clear();
    }

    // Makes room for one more record of a kind in the open stage, or starts another.
    void kind(uint32_t k) {
        if (cur.kind != k || 16 + ((uint32_t)recs.size() + 1) * rec(k) > kProgBlock) close();
        cur.kind = (uint16_t)k;
    }
    // The row that takes an op of part p next: the open one if its last part
    // comes before p, or is p and `fits`; else a new one.
    Rec& row(int p, bool fits) {
        if (cur.kind != PK_ROWS || part < 0 || p < part || (p == part && !fits) || recs.empty()) {
            kind(PK_ROWS);
            recs.emplace_back();
        }
        part = p;
        return recs.back();
    }
    static Rec& more(Rec& r) {  // the row is not CNOTs alone
        r.w[0] |= 1u << 4;
        return r;
    }
    Rec& misc(uint32_t type, uint32_t arg) {
        kind(PK_MISC);
        recs.emplace_back();
        recs.back().w[0] = type | (arg << 8);
        return recs.back();
    }
    uint32_t slot(int gate) {
        prog->slot_param.push_back((*gates)[gate].pidx);
        return (uint32_t)prog->slot_param.size() - 1;
    }

    void rot(const StageOp& k) override {
        const int e = (int)gate_entry(TF_ROT, k.gate, 1), b = k.bit[0];
        pending.push_back(k.gate);
        if (k.kind == K_ROTX) misc(PM_ROTX, (uint32_t)b).num[0] = e;
        else more(row(p_rot(), !recs.empty() && recs.back().num[b] < 0)).num[b] = e;
    }
    // Phases are made for every register entry; a scale alone is a row of equal phases.
    uint32_t table_mask(uint32_t) const override { return (1u << kProgBits) - 1; }
    void phase_by(uint32_t e, uint32_t) override { more(row(p_phase(), false)).phase = (int)e; }
    void scale_by(uint32_t e) override {
        out->entries[e].kind = TF_PHASE;
        out->entries[e].mask = table_mask(0);
        phase_by(e, 0);
    }
    void matrix(const StageOp& k) override {
        const Gate& g = (*gates)[k.gate];
        const int e = (int)gate_entry(TF_R2, k.gate, 4);
        if (!is_excitation_kind(g.kind)) {
            misc(PM_R2, (uint32_t)k.bit[0]).num[0] = e;
            return;
        }
        uint32_t mask, A, B, ta = 0, tb = 0;
        stage_pattern(g, k, mask, A, B);
        for (int i = 0; i < kProgBits; ++i) {
            ta |= ((A >> i) & 1u) << cur.pos[i];
            tb |= ((B >> i) & 1u) << cur.pos[i];
        }
        kind(PK_PAIRS);
        recs.emplace_back();
        Rec& r = recs.back();
        r.w[0] = ta | (tb << 16);
        r.num[0] = e;
        if (!pair_slot.empty() && pair_slot.back().first == k.gate) {
            r.w[1] = pair_slot.back().second;
            r.w[2] = 1;
            pair_slot.pop_back();
        }
    }
    void rename(const StageOp& k) override {
        const int c = k.bit[0], t = k.kind == K_CNOT ? k.bit[1] : c;
        if (k.kind == K_CNOT && t == c + 1) row(p_cnot(c), false).w[0] |= 1u << c;
        else misc(PM_PERM, (uint32_t)(c << 2 | t));
    }
    // Z or Y term of bit b to slot s: mask at `shift` of the flags, slot and offsets in words wi, wi + 1
    void term(int p, int shift, int wi, int b, uint32_t s) {
        const bool fits = !recs.empty() && !((recs.back().w[0] >> (shift + b)) & 1) && s - recs.back().w[wi] < 256;
        Rec& r = more(row(p, fits));
        if (!((r.w[0] >> shift) & 0xfu)) r.w[wi] = s;
        r.w[0] |= 1u << (shift + b);
        r.w[wi + 1] |= (s - r.w[wi]) << (8 * b);
    }
    void gradient(const StageOp& k) override {
        const Gate& g = (*gates)[k.gate];
        const uint32_t s = slot(k.gate);
        if (is_excitation_kind(g.kind)) pair_slot.emplace_back(k.gate, s);  // taken along by the gate's own pair, emitted next
        else if (g.kind == VQE_GATE_RX) misc(PM_GX, (uint32_t)k.bit[0]).w[1] = s;
        else term(kY, 12, 3, k.bit[0], s);
    }
    void gradient_z(const std::vector<StageOp>& all) override {
        for (const StageOp& k : all) term(kZ, 8, 1, k.bit[0], slot(k.gate));
    }
};

}  // namespace

bool plan_program(int bits, const std::vector<Gate>& gates, const std::vector<int>& list, const int* local,
                  ProgramPlan& out, std::string& msg) {
    std::vector<Gate>& lg = out.gates;
    lg.clear();
    for (int gi : list) {
        Gate g = gates[gi];
        g.q0 = local[g.q0];
        g.q1 = local[g.q1];
        g.q2 = local[g.q2];
        g.q3 = local[g.q3];
        lg.push_back(g);
    }
    out.list = list;
    const int big = 1 << 20;
    return plan_passes(bits, lg, PlanLimits{kProgBits, big, big, big}, out.stages, msg);
}

bool build_program(bool dbl, int bits, const std::vector<Gate>& gates, const ProgramPlan& plan, int dir, bool flush,
                   Program& out, std::string& msg) {
    out = Program();
    const std::vector<Gate>& lg = plan.gates;
    Builder b;
    b.dbl = dbl;
    b.gates = &gates;
    b.out = &out.table;
    b.prog = &out;
    b.dir = dir;
    for (size_t k = 0; k < plan.stages.size(); ++k) {
        const PlannedPass& s = plan.stages[dir ? plan.stages.size() - 1 - k : k];
        std::vector<int> r(s.pos, s.pos + s.K);
        for (int q = bits - 1; (int)r.size() < kProgBits; --q)
            if (std::find(r.begin(), r.end(), q) == r.end()) r.push_back(q);
        std::sort(r.begin(), r.end());
        int rbit[64];
        uint8_t pos[kProgBits];
        for (int i = 0; i < kProgBits; ++i) {
            pos[i] = (uint8_t)r[i];
            rbit[r[i]] = i;
        }
        std::vector<StageOp> ops;
        auto add = [&](int li, bool grad) {
            int q[4], at[4];
            const int nq = gate_qubits(lg[li], q);
            for (int i = 0; i < nq; ++i) at[i] = rbit[q[i]];
            ops.push_back(stage_op(lg[li], plan.list[li], at, grad));
        };
        if (dir == 0) {
            for (int li : s.gates) add(li, false);
        } else {
            for (size_t i = s.gates.size(); i-- > 0;) {
                if (lg[s.gates[i]].pidx >= 0) add(s.gates[i], true);
                add(s.gates[i], false);
            }
        }
        b.open(pos);
        b.stage(std::move(ops));
        if (flush || k + 1 == plan.stages.size()) b.scale();
        b.close();
        if (!b.pair_slot.empty()) {
            msg = "an excitation's gradient term without its gate (internal error)";
            return false;
        }
        out.mark.push_back((uint32_t)out.stages.size());
    }
    for (size_t i = 0; i + 1 < out.stages.size(); ++i)
        std::memcpy(&out.stream[out.stages[i].off / 4], &out.stages[i + 1], sizeof(ProgStage));
    return true;
}

}  // namespace vqe

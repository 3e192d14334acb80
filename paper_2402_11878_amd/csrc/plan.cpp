// Fusion planner: partitions a gate list into passes, each pass a window of at
// most lim.kmax qubits whose gates are applied with one read and one write
// of the state (one HBM sweep instead of one per gate).
//
// Gates on disjoint qubits commute, so a gate may run before any earlier gate
// it shares no qubit with; the order of every pair of gates sharing a qubit is
// kept.  Per qubit the gates form a chain; a gate is ready when it heads the
// chain of each of its qubits.  A pass takes a window W and schedules, to a
// fixed point, every ready gate whose qubits lie in W (its closure).  Windows
// are chosen greedily: candidates are every run of consecutive qubits and a
// window grown qubit by qubit from the earliest unscheduled gate; the
// candidate with the largest closure wins (ties: first found).  For the
// layered RY/RZ + CNOT-ladder ansatz this yields overlapping ladder windows
// that pipeline across layers.
#include <algorithm>
#include <array>
#include <set>

#include "vqe_internal.h"

namespace vqe {
namespace {

struct PlanGate {
    int q[4], nq;
    int ops, mats, slots;  // what it counts against the limits of a pass
};
struct PlanState {
    const PlanLimits* lim;
    std::vector<PlanGate> gates;
    std::vector<std::vector<int>> chain;  // per qubit, gate indices in order
};
// Per qubit, position of its next unscheduled gate.
using Heads = std::array<uint32_t, 64>;

bool is_param(const Gate& g) { return g.pidx >= 0; }

bool uses_matrix(const Gate& g) {
    return g.kind == VQE_GATE_RY || g.kind == VQE_GATE_RZ || g.kind == VQE_GATE_RX ||
           g.kind == VQE_GATE_H || g.kind == VQE_GATE_SEXC || g.kind == VQE_GATE_DEXC;
}

uint64_t gate_mask(const Gate& g) {
    int q[4];
    const int k = gate_qubits(g, q);
    uint64_t m = 0;
    for (int i = 0; i < k; ++i) m |= 1ull << q[i];
    return m;
}

// Closure of window W (bit mask over qubits) starting from `head`; appends the
// scheduled gates to `out` (if non-null) and advances `head`.  Respects the
// per-pass op / matrix / gradient-slot limits (a repeated parameter within a
// pass shares its slot, counted here once per gate: a safe overestimate).
int closure(const PlanState& ps, uint64_t W, Heads& head, std::vector<int>* out) {
    const PlanLimits& L = *ps.lim;
    int count = 0, ops_rev = 0, mats = 0, slots = 0;
    bool changed = true;
    while (changed) {
        changed = false;
        for (uint64_t m = W; m; m &= m - 1) {
            const int q = __builtin_ctzll(m);
            const std::vector<int>& ch = ps.chain[q];
            while (head[q] < ch.size()) {
                const int gi = ch[head[q]];
                const PlanGate& g = ps.gates[gi];
                bool ready = true;
                for (int i = 0; i < g.nq && ready; ++i)
                    ready = ((W >> g.q[i]) & 1) && ps.chain[g.q[i]][head[g.q[i]]] == gi;
                if (!ready) break;
                if (ops_rev + g.ops > L.ops || mats + g.mats > L.mats || slots + g.slots > L.slots) return count;
                ops_rev += g.ops;
                mats += g.mats;
                slots += g.slots;
                for (int i = 0; i < g.nq; ++i) head[g.q[i]]++;
                if (out) out->push_back(gi);
                ++count;
                changed = true;
            }
        }
    }
    return count;
}

int popcount64(uint64_t v) { return __builtin_popcountll(v); }

}  // namespace

bool plan_passes(int n, const std::vector<Gate>& gates, const PlanLimits& lim, std::vector<PlannedPass>& out,
                 std::string& msg) {
    out.clear();
    const int K = std::min(n, std::min(lim.kmax, kMaxPlanWindow));
    PlanState ps;
    Heads head{};
    ps.lim = &lim;
    ps.gates.resize(gates.size());
    ps.chain.assign(n, {});
    for (size_t i = 0; i < gates.size(); ++i) {
        PlanGate& g = ps.gates[i];
        g.nq = gate_qubits(gates[i], g.q);
        g.slots = is_param(gates[i]) ? 1 : 0;
        g.ops = 1 + g.slots;
        g.mats = uses_matrix(gates[i]) ? 1 : 0;
        for (int k = 0; k < g.nq; ++k) ps.chain[g.q[k]].push_back((int)i);
    }
    size_t scheduled = 0;
    std::vector<char> done(gates.size(), 0);
    size_t earliest = 0;
    while (scheduled < gates.size()) {
        while (done[earliest]) ++earliest;
        // Candidate windows.
        std::vector<uint64_t> cands;
        for (int a = 0; a + K <= n; ++a) cands.push_back(((K == 64 ? ~0ull : ((1ull << K) - 1))) << a);
        {
            uint64_t W = gate_mask(gates[earliest]);
            while (popcount64(W) < K) {
                int best_q = -1, best_c = -1;
                for (int q = 0; q < n; ++q) {
                    if ((W >> q) & 1) continue;
                    Heads h = head;
                    int c = closure(ps, W | (1ull << q), h, nullptr);
                    if (c > best_c) {
                        best_c = c;
                        best_q = q;
                    }
                }
                if (best_q < 0) break;
                W |= 1ull << best_q;
            }
            cands.push_back(W);
        }
        uint64_t bestW = 0;
        int bestC = 0;
        for (uint64_t W : cands) {
            Heads h = head;
            int c = closure(ps, W, h, nullptr);
            if (c > bestC) {
                bestC = c;
                bestW = W;
            }
        }
        if (bestC == 0) {
            msg = "planner made no progress (internal error)";
            return false;
        }
        PlannedPass p;
        closure(ps, bestW, head, &p.gates);
        // Shrink the window to the qubits actually touched.
        uint64_t used = 0;
        for (int gi : p.gates) used |= gate_mask(gates[gi]);
        p.K = 0;
        for (int q = 0; q < n; ++q)
            if ((used >> q) & 1) p.pos[p.K++] = q;
        for (int gi : p.gates) done[gi] = 1;
        scheduled += p.gates.size();
        out.push_back(std::move(p));
    }
    return true;
}

// Tile passes (see plan_tiles in vqe_internal.h): beam search over the order
// of the windows.  A state is the head of every qubit's chain; a step takes a
// candidate window to its closure.  After each depth the lim.width states with
// the most scheduled gates live on; the first to schedule every gate wins.
// Greedy (width 1) leaves the ends of the CNOT ladders to passes of their
// own: 13 passes at 32 qubits x 8 layers (12-qubit tiles, 3 low qubits)
// against 10 with 48.
bool plan_tiles(int n, const std::vector<Gate>& gates, const TileLimits& lim, std::vector<PlannedPass>& out,
                std::string& msg) {
    out.clear();
    if (gates.empty()) return true;
    const int K = std::min(n, lim.bits);
    const uint64_t all = n == 64 ? ~0ull : (1ull << n) - 1;
    const uint64_t low = ((1ull << std::min(lim.low, K)) - 1) & all;
    const size_t total = gates.size();
    std::vector<std::array<int, 4>> gq(total);
    std::vector<int> nq(total);
    std::vector<std::vector<int>> chain(n);
    for (size_t i = 0; i < total; ++i) {
        nq[i] = gate_qubits(gates[i], gq[i].data());
        for (int k = 0; k < nq[i]; ++k) chain[gq[i][k]].push_back((int)i);
    }
    using Head = std::vector<uint32_t>;
    size_t work = 0;
    auto close = [&](uint64_t W, Head& head, std::vector<int>* list) {
        int count = 0, pushes = 0;
        for (bool changed = true; changed;) {
            changed = false;
            for (int q = 0; q < n; ++q) {
                if (!((W >> q) & 1)) continue;
                while (head[q] < chain[q].size()) {
                    const int gi = chain[q][head[q]];
                    bool ready = true;
                    for (int k = 0; k < nq[gi] && ready; ++k) {
                        const int o = gq[gi][k];
                        ready = ((W >> o) & 1) && chain[o][head[o]] == gi;
                    }
                    if (!ready) break;
                    const int add = is_param(gates[gi]) ? 1 : 0;
                    if (count == lim.gates || pushes + add > lim.pushes) return count;
                    pushes += add;
                    for (int k = 0; k < nq[gi]; ++k) ++head[gq[gi][k]];
                    if (list) list->push_back(gi);
                    ++count;
                    changed = true;
                }
            }
            work += (size_t)K;
        }
        work += (size_t)count;
        return count;
    };
    struct Node {
        Head head;
        size_t count;
        int parent;
        uint64_t W;
    };
    constexpr size_t kWorkBudget = 4000000;  // steps of `close`, about 20 ms of planning
    std::vector<std::vector<Node>> depth(1);
    depth[0].push_back(Node{Head(n, 0), 0, -1, 0});
    int goal = -1;
    while (goal < 0) {
        const std::vector<Node>& cur = depth.back();
        std::vector<Node> next;
        std::set<Head> seen;
        for (size_t i = 0; i < cur.size() && goal < 0; ++i) {
            if (i > 0 && work > kWorkBudget) break;  // out of budget: go on greedily
            std::vector<uint64_t> cands;
            for (int a = 0; a < n; ++a) {  // the low qubits and the K - low next ones from a on
                uint64_t W = low;
                for (int q = a; q < n && popcount64(W) < K; ++q) W |= 1ull << q;
                if (popcount64(W) < K) break;
                if (cands.empty() || cands.back() != W) cands.push_back(W);
            }
            {  // a window grown from the first gate still open, for circuits without a ladder
                int first = -1;
                for (int q = 0; q < n; ++q)
                    if (cur[i].head[q] < chain[q].size()) {
                        const int gi = chain[q][cur[i].head[q]];
                        if (first < 0 || gi < first) first = gi;
                    }
                uint64_t W = low | gate_mask(gates[first]);
                for (int gi = first; gi < (int)total && popcount64(W) < K; ++gi) {
                    const uint64_t m = W | gate_mask(gates[gi]);
                    if (popcount64(m) <= K) W = m;
                }
                for (int q = 0; q < n && popcount64(W) < K; ++q) W |= 1ull << q;
                if (popcount64(W) <= K) cands.push_back(W);
            }
            for (uint64_t W : cands) {
                Head h = cur[i].head;
                const int c = close(W, h, nullptr);
                if (c == 0 || !seen.insert(h).second) continue;
                next.push_back(Node{std::move(h), cur[i].count + (size_t)c, (int)i, W});
                if (next.back().count == total) {
                    goal = (int)next.size() - 1;
                    break;
                }
            }
        }
        if (next.empty()) {
            msg = "tile planner made no progress (internal error)";
            return false;
        }
        if (goal < 0) {
            std::stable_sort(next.begin(), next.end(), [](const Node& a, const Node& b) { return a.count > b.count; });
            if (next.size() > (size_t)lim.width) next.resize((size_t)lim.width);
        }
        depth.push_back(std::move(next));
    }
    std::vector<uint64_t> wins;
    for (int d = (int)depth.size() - 1, i = goal; d > 0; --d) {
        wins.push_back(depth[d][i].W);
        i = depth[d][i].parent;
    }
    Head head(n, 0);
    for (size_t k = wins.size(); k-- > 0;) {
        PlannedPass p;
        close(wins[k], head, &p.gates);
        for (int q = 0; q < n; ++q)
            if ((wins[k] >> q) & 1) p.pos[p.K++] = q;
        out.push_back(std::move(p));
    }
    return true;
}

}  // namespace vqe

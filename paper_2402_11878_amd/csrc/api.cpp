// C ABI of the VQE library: state handles, circuits (fused pass plans),
// Hamiltonian tables and the energy / gradient drivers.  All device work is
// enqueued on the state's stream; host scalars are returned after one
// synchronisation of that stream.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <numeric>

#include "vqe_internal.h"

using namespace vqe;

namespace vqe {
namespace {
thread_local std::string g_last_error;
}
void set_error(const std::string& m) { g_last_error = m; }
}  // namespace vqe

#define VQE_HIP(call)                                                                  \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess) {                                                        \
            set_error(std::string(#call) + ": " + hipGetErrorString(e_));              \
            return VQE_ERR_DEVICE;                                                     \
        }                                                                              \
    } while (0)

#define VQE_GUARD_BEGIN try {
#define VQE_GUARD_END                                                                  \
    }                                                                                  \
    catch (const std::bad_alloc&) {                                                    \
        set_error("host allocation failed");                                           \
        return VQE_ERR_OOM;                                                            \
    }                                                                                  \
    catch (const std::exception& ex) {                                                 \
        set_error(std::string("internal error: ") + ex.what());                        \
        return VQE_ERR_STATE;                                                          \
    }

// ---------------------------------------------------------------- handles
struct vqe_state {
    int n = 0;
    int dtype = 0;
    void* data = nullptr;
    size_t bytes = 0;
    bool owned = false;
    hipStream_t stream = nullptr;
    int device = 0;
    double* d_part = nullptr;  // per-block partial sums (allocated on first use)
    double* d_res = nullptr;   // results (energies, gradients), grown on demand
    size_t res_cap = 0;
    double* h_res = nullptr;   // pinned host mirror of d_res
    void* d_mats = nullptr;    // matrix table of the specialised kernels, filled per evaluation
    void* h_mats = nullptr;    // pinned staging of d_mats
    // per pass, whether the shear forms of its reverse rotations flip the sign
    // of psi and lam an odd number of times (filled with the matrix table)
    std::vector<int8_t> rev_flip;
    size_t mats_cap = 0;
    hipEvent_t mats_ev = nullptr;  // completion of the last upload from h_mats
    vqe_batch* mid = nullptr;      // buffers of evaluations by batch programs (made on first use)
};

// Physical op list of a pass in the lane-split layout with S split bits.
struct SplitOps {
    std::vector<KOp> ops;
    uint8_t map_in[kMaxWindow] = {0}, map_out[kMaxWindow] = {0};  // physical slot -> window local bit
};

struct PassOps {
    std::vector<KOp> fwd, rev;
    std::vector<int> fwd_mat_gate, rev_mat_gate;  // matrix slot -> gate index
    std::vector<int32_t> slot_param;              // reverse gradient slot -> parameter
    // Per dtype (0: complex64, 1: complex128): lane-split bits of the forward
    // and reverse pass and, where S > 0, the ops lowered to physical slots.
    int S_f[2] = {0, 0}, S_r[2] = {0, 0};
    SplitOps fwd_l[2], rev_l[2];
};

// A fused pass plan: interpreted (windows <= kInterpWindow qubits, ops and
// matrices as kernel arguments) or specialised (windows <= kMaxWindow, one
// run-time compiled kernel per pass, matrices from a per-evaluation table).
struct Plan {
    bool jit = false;
    std::vector<PlannedPass> passes;
    std::vector<PassOps> ops;
    std::vector<int32_t> slotmap;   // all passes' gradient slot -> parameter maps
    int32_t* d_slotmap = nullptr;   // uploaded on first use on a device
    std::vector<size_t> slot_off;
    std::vector<size_t> mat_off;    // [2 pass + dir]: first matrix of the pass in the table
    size_t mat_total = 0;
    std::vector<void*> jfn[2][2];   // [dtype][dir] specialised kernels, built on first use
    int jit_dev[2] = {-1, -1};      // device they are loaded on
};

// Batch programs of one amplitude type (program.cpp), made on first use: two
// programs (forward, reverse) for a state that fits LDS, two per pass for a
// mid-size one, a pass p as programs 2 p and 2 p + 1.  An evaluation uploads the
// image (every program's stages, then their streams) with its numbers filled in.
struct BatchPlan {
    bool ready = false;
    std::vector<PlannedPass> passes;     // mid-size: windows of kMidWin qubits
    std::vector<Program> prog;
    std::vector<size_t> stage_off, stream_off;  // bytes in the image
    std::vector<char> image;             // numbers still zero
    std::vector<size_t> slot_off;        // first gradient slot of the program (reverse ones)
    std::vector<int32_t> slot_param;     // every reverse program's slots, in program order
};

// Tile passes of one amplitude type (tile.cpp), made on first use.
struct TilePlan {
    bool ready = false;
    int dev = -1;                        // device the kernels are loaded on
    std::vector<PlannedPass> passes;
    std::vector<TileKernel> k[2];        // [direction][pass]; sources dropped once loaded
    std::vector<size_t> tab_off[2];      // first scalar of the pass in an evaluation's table
    size_t tab_total = 0;                // scalars
    std::vector<void*> fn[2];
    uint32_t L = 0;                      // columns of the gradient partials, the same for every pass
};

struct vqe_circuit {
    int n = 0;
    std::vector<Gate> gates;
    size_t n_params = 0;
    Plan plan[2];  // [0]: interpreted (not built for circuits with excitation gates), [1]: specialised
    TilePlan tile[2];  // per dtype (0: complex64, 1: complex128)
    bool has_excitation = false;
    BatchPlan batch[2][2];  // per dtype; [1]: with the places of checkpoints (small states)
};

struct vqe_hamiltonian {
    int n = 0;
    std::vector<uint64_t> x, z;  // combined terms, sorted by (x, z)
    std::vector<double> w;
    std::vector<GroupDesc> groups;
    std::vector<TermDesc<float>> t32;
    std::vector<TermDesc<double>> t64;
    double identity = 0.0;
    double norm1 = 0.0;  // sum of |w|: bounds the 2-norm of H psi for a normalised psi
    // every folded coefficient real (each term has an even number of Y, as for
    // any real symmetric H): the window passes of H psi skip imaginary parts
    bool real_coeffs = true;
    // small states (n <= kBatchMaxQubitsC64): terms by register bucket
    // (batch.hip), per dtype: the blocks, then their stream
    std::vector<SmallBlock> sm_blocks[2];
    std::vector<char> sm_stream[2];
    SmallBlock* d_sm_blocks[2] = {nullptr, nullptr};
    char* d_sm_stream[2] = {nullptr, nullptr};
    // device tables, uploaded on first use on a device (in d_tables, then d_ready)
    bool d_ready = false;
    void* d_tables = nullptr;
    GroupDesc* d_groups = nullptr;
    TermDesc<float>* d_t32 = nullptr;
    TermDesc<double>* d_t64 = nullptr;
    // window-pass form of H psi (empty when the tile kernel moves fewer bytes
    // for both uses): hw_lam selects it for lam = H psi, hw_energy for the
    // energy-only sweep
    bool hw_lam = false, hw_energy = false;
    std::vector<HwDesc> hw_wins;
    std::vector<HwGroup> hw_groups;
    std::vector<HwClass> hw_classes;
    std::vector<HwTerm<float>> hw_t32;
    std::vector<HwTerm<double>> hw_t64;
    HwGroup* d_hw_groups = nullptr;
    HwClass* d_hw_classes = nullptr;
    HwTerm<float>* d_hw_t32 = nullptr;
    HwTerm<double>* d_hw_t64 = nullptr;
};

struct vqe_batch {
    int dtype = 0;
    hipStream_t stream = nullptr;
    int device = 0;
    void* d_buf = nullptr;   // items | gates | mats | out, one allocation
    size_t d_cap = 0;
    void* h_buf = nullptr;   // pinned staging of the same layout
    size_t h_cap = 0;
    // mid-size items: tables | out | partial sums | states (device), tables | out (pinned)
    void* md_buf = nullptr;
    size_t md_cap = 0;
    void* mh_buf = nullptr;
    size_t mh_cap = 0;
};

namespace {

size_t amp_bytes(int dtype) { return dtype == VQE_C64 ? 8 : 16; }

std::mutex g_upload_mu;  // lazy device uploads of shared handles

// ---------------------------------------------------------------- tracing
struct ProfRec {
    int kind;
    hipEvent_t a, b;
    double bytes;
};
struct ProfTotals {
    uint64_t launches = 0;
    double ms = 0.0, bytes = 0.0;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfRec> g_prof_pending;
ProfTotals g_prof_tot[VQE_KERNEL_KINDS];

// Brackets one kernel launch with events when tracing is on.
struct ProfScope {
    bool on;
    ProfRec r{};
    hipStream_t st;
    ProfScope(int kind, double bytes, hipStream_t s) : on(false), st(s) {
        std::lock_guard<std::mutex> g(g_prof_mu);
        if (!g_prof_on) return;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return;
        if (hipEventCreate(&r.a) != hipSuccess) return;
        if (hipEventCreate(&r.b) != hipSuccess) {
            (void)hipEventDestroy(r.a);
            return;
        }
        r.kind = kind;
        r.bytes = bytes;
        on = hipEventRecord(r.a, st) == hipSuccess;
    }
    void end() {
        if (!on) return;
        on = false;
        (void)hipEventRecord(r.b, st);
        std::lock_guard<std::mutex> g(g_prof_mu);
        g_prof_pending.push_back(r);
    }
    ~ProfScope() { end(); }
};

void prof_drain() {
    for (auto& r : g_prof_pending) {
        float ms = 0.f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            g_prof_tot[r.kind].launches += 1;
            g_prof_tot[r.kind].ms += ms;
            g_prof_tot[r.kind].bytes += r.bytes;
        }
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    g_prof_pending.clear();
}

int ensure_res(vqe_state* s, size_t count) {
    if (count <= s->res_cap) return VQE_OK;
    size_t cap = std::max<size_t>(count, 1024);
    if (s->d_res) {
        VQE_HIP(hipStreamSynchronize(s->stream));
        VQE_HIP(hipFree(s->d_res));
        s->d_res = nullptr;
    }
    if (s->h_res) {
        VQE_HIP(hipHostFree(s->h_res));
        s->h_res = nullptr;
    }
    s->res_cap = 0;
    if (hipMalloc((void**)&s->d_res, cap * sizeof(double)) != hipSuccess) {
        set_error("hipMalloc of the result buffer failed");
        return VQE_ERR_OOM;
    }
    if (hipHostMalloc((void**)&s->h_res, cap * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        set_error("hipHostMalloc of the result buffer failed");
        return VQE_ERR_OOM;
    }
    s->res_cap = cap;
    return VQE_OK;
}

int upload_plan(const Plan& cpl);
bool lower_split(const std::vector<KOp>& ops, int K, int S, size_t cap, SplitOps& out);

// Device copies of a Hamiltonian's tables; the handle publishes them only
// when they were allocated and copied (d_ready), so a failed upload leaves
// nothing half-built behind.
void free_hamiltonian_tables(vqe_hamiltonian* h) {
    if (h->d_tables) (void)hipFree(h->d_tables);
    h->d_tables = nullptr;
    h->d_ready = false;
}

// Uploads the grouped term tables to the current device (once): one allocation
// and one copy, which a first evaluation waits for.
int upload_hamiltonian(const vqe_hamiltonian* ch) {
    vqe_hamiltonian* h = const_cast<vqe_hamiltonian*>(ch);
    std::lock_guard<std::mutex> g(g_upload_mu);
    if (h->d_ready) return VQE_OK;
    free_hamiltonian_tables(h);  // leftovers of an earlier failed attempt
    std::vector<char> img;
    auto each = [&](auto&& f) {
        f(h->d_groups, h->groups);
        f(h->d_t32, h->t32);
        f(h->d_t64, h->t64);
        f(h->d_hw_groups, h->hw_groups);
        f(h->d_hw_classes, h->hw_classes);
        f(h->d_hw_t32, h->hw_t32);
        f(h->d_hw_t64, h->hw_t64);
        for (int d = 0; d < 2; ++d) {
            f(h->d_sm_blocks[d], h->sm_blocks[d]);
            f(h->d_sm_stream[d], h->sm_stream[d]);
        }
    };
    each([&](auto&, const auto& src) {
        const size_t at = (img.size() + 255) / 256 * 256, bytes = src.size() * sizeof(src[0]);
        img.resize(at + bytes);
        if (bytes) std::memcpy(&img[at], src.data(), bytes);
    });
    img.resize(img.size() + 256);  // an empty table at the end points inside too
    if (hipMalloc(&h->d_tables, img.size()) != hipSuccess) {
        h->d_tables = nullptr;
        set_error("hipMalloc of the Hamiltonian tables failed");
        return VQE_ERR_OOM;
    }
    if (hipMemcpy(h->d_tables, img.data(), img.size(), hipMemcpyHostToDevice) != hipSuccess) {
        set_error("hipMemcpy of the Hamiltonian tables failed");
        free_hamiltonian_tables(h);
        return VQE_ERR_DEVICE;
    }
    size_t at = 0;
    each([&](auto& dst, const auto& src) {
        at = (at + 255) / 256 * 256;
        dst = (std::remove_reference_t<decltype(dst)>)((char*)h->d_tables + at);
        at += src.size() * sizeof(src[0]);
    });
    h->d_ready = true;
    return VQE_OK;
}

// Greedy cover of the X masks xs (none inside `low`) by windows of kHwBits
// qubits that contain `low`.  A window grows one qubit at a time, taking the
// qubit with the largest sum over the uncovered masks containing it (and
// still fitting) of 1 / outside^p (outside = their bits not yet in the
// window), so that nearly complete masks weigh most; it takes every mask
// inside it.  With rng_state != 0 the scores are perturbed by a factor in
// [1, 1.001) from a splitmix64 stream, which only reorders near-ties.
// Returns the windows (empty if no progress is possible); *work counts the
// inner-loop steps.
std::vector<uint64_t> cover_windows(int n, const std::vector<uint64_t>& xs, uint64_t low, int p, uint64_t rng_state,
                                    size_t* work) {
    auto uniform = [&]() {
        uint64_t z = (rng_state += 0x9e3779b97f4a7c15ull);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        return (double)((z ^ (z >> 31)) >> 11) * 0x1.0p-53;
    };
    std::vector<uint64_t> rem = xs, wins;
    while (!rem.empty() || wins.empty()) {
        uint64_t W = low;
        while (__builtin_popcountll(W) < kHwBits) {
            int best = -1;
            double best_score = 0.0;
            const int inside = __builtin_popcountll(W);
            for (int q = 0; q < n; ++q) {
                if ((W >> q) & 1) continue;
                double sc = 0.0;
                for (uint64_t x : rem) {
                    if (!((x >> q) & 1)) continue;
                    const int outside = __builtin_popcountll(x & ~W);
                    if (inside + outside <= kHwBits) sc += 1.0 / std::pow((double)outside, p);
                }
                *work += rem.size();
                if (rng_state && sc > 0.0) sc *= 1.0 + 1e-3 * uniform();
                if (sc > best_score) {
                    best_score = sc;
                    best = q;
                }
            }
            if (best < 0) break;
            W |= 1ull << best;
        }
        for (int q = 0; q < n && __builtin_popcountll(W) < kHwBits; ++q) W |= 1ull << q;  // fill up
        std::vector<uint64_t> left;
        for (uint64_t x : rem)
            if (x & ~W) left.push_back(x);
        if (left.size() == rem.size() && !rem.empty()) return {};  // no progress
        rem.swap(left);
        wins.push_back(W);
    }
    return wins;
}

// Window-pass plan of lam = H psi (see HwDesc): the smallest of several
// greedy covers (cover_windows with p = 1, 2, 3, each deterministic and
// with seeded tie perturbations, as many restarts as a fixed work budget
// allows); the groups spread evenly over the windows holding them.  Used for
// lam = H psi if its (3 m - 1) S of traffic (m passes; psi read per pass, lam
// written once and read-modify-written m - 1 times) is below the tile
// kernel's (D + 2) S, and for the energy-only sweep if its m S (psi read per
// pass) is below the tile kernel's (1 + D / 2) S; kept if either holds.
void plan_hwin(vqe_hamiltonian* h) {
    const int n = h->n;
    if (n < kHwBits) return;
    const uint64_t low = (1ull << kHwLow) - 1;
    const size_t G = h->groups.size();
    std::vector<uint64_t> xs;
    for (size_t g = 0; g < G; ++g) {
        if (__builtin_popcountll(h->groups[g].x | low) > kHwBits) return;  // a mask no window can hold
        if (h->groups[g].x & ~low) xs.push_back(h->groups[g].x);
    }
    if (xs.size() > 4096) return;  // planning cost; such Hamiltonians stay on the tile kernel
    constexpr size_t kWorkBudget = 200000000;  // inner-loop steps over all restarts (well under a second)
    constexpr int kMaxRestarts = 12;
    std::vector<uint64_t> wins;
    size_t work = 0;
    for (int p = 1; p <= 3; ++p) {
        for (int r = 0; r <= kMaxRestarts; ++r) {
            const size_t before = work;
            std::vector<uint64_t> w = cover_windows(n, xs, low, p, r ? 0x5eedull * (uint64_t)(16 * p + r) : 0, &work);
            if (w.empty()) return;
            if (wins.empty() || w.size() < wins.size()) wins.swap(w);
            if (work + 3 * (work - before) > kWorkBudget) break;  // a later restart could overrun the budget
        }
        if (work > kWorkBudget) break;
    }
    // Each group goes to one of the windows holding its X mask.  A pass costs
    // about the larger of its memory time and a fixed amount of arithmetic per
    // group (the per-group bodies dominate; the class count matters little),
    // so the groups are spread evenly: those only one window holds first, then
    // the others, the most constrained first, each to the holding window where
    // it adds the least cost, max(kHwPassGroups x passes, groups) with passes =
    // ceil(classes / kHwMaxClasses); ties go to the window with fewer groups,
    // then fewer classes, then the lower index.
    constexpr size_t kHwPassGroups = 16;  // groups per pass whose arithmetic about matches its memory time
    const size_t Wn = wins.size();
    std::vector<std::vector<std::pair<int, size_t>>> cand(G);  // (window, classes of the group in it)
    std::vector<uint64_t> zw;
    for (size_t g = 0; g < G; ++g)
        for (size_t wi = 0; wi < Wn; ++wi) {
            if (h->groups[g].x & ~wins[wi]) continue;
            zw.clear();
            for (uint32_t t = h->groups[g].begin; t < h->groups[g].end; ++t) zw.push_back(h->t64[t].z & wins[wi]);
            std::sort(zw.begin(), zw.end());
            cand[g].emplace_back((int)wi, (size_t)(std::unique(zw.begin(), zw.end()) - zw.begin()));
        }
    std::vector<size_t> order(G);
    for (size_t g = 0; g < G; ++g) order[g] = g;
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return cand[a].size() < cand[b].size(); });
    std::vector<size_t> w_groups(Wn, 0), w_classes(Wn, 0);
    auto w_cost = [&](size_t groups, size_t classes) {
        const size_t passes = std::max<size_t>(1, (classes + kHwMaxClasses - 1) / kHwMaxClasses);
        return std::max(kHwPassGroups * passes, groups);
    };
    std::vector<int> win_of(G, -1);
    for (size_t g : order) {
        int best = -1;
        size_t best_add = 0, best_cls = 0;
        for (const auto& [wi, cls] : cand[g]) {
            const size_t add = w_cost(w_groups[wi] + 1, w_classes[wi] + cls) - w_cost(w_groups[wi], w_classes[wi]);
            if (best < 0 || add < best_add ||
                (add == best_add && (w_groups[wi] < w_groups[best] ||
                                     (w_groups[wi] == w_groups[best] && w_classes[wi] + cls < w_classes[best] + best_cls)))) {
                best = wi;
                best_add = add;
                best_cls = cls;
            }
        }
        if (best < 0) return;  // cannot happen for a cover; the tile form stays
        win_of[g] = best;
        w_groups[best] += 1;
        w_classes[best] += best_cls;
    }
    // Passes: per window its groups, the terms of a group merged into classes
    // of equal in-window z bits and sorted by them (register part first), at
    // most kHwMaxClasses classes per pass.  A window with more classes takes
    // several passes over the same qubits; lam accumulates over passes, so a
    // group's classes may also be split between two of them.
    std::vector<HwDesc> passes;
    std::vector<HwGroup> hgroups;
    std::vector<HwClass> hclasses;
    std::vector<HwTerm<float>> ht32;
    std::vector<HwTerm<double>> ht64;
    constexpr int kBuckets = 1 << kHwRegBits;
    const uint32_t tmask = (1u << kHwThreadBits) - 1;
    for (size_t wi = 0; wi < wins.size(); ++wi) {
        HwDesc d{};
        int k = 0, local[64];
        for (int q = 0; q < n; ++q)
            if ((wins[wi] >> q) & 1) {
                local[q] = k;
                d.pos[k++] = (uint32_t)q;
            }
        auto compress = [&](uint64_t m) {
            uint32_t r = 0;
            for (int q = 0; q < n; ++q)
                if ((m >> q) & 1) r |= 1u << local[q];
            return r;
        };
        d.g_begin = (uint32_t)hgroups.size();
        d.c_begin = (uint32_t)hclasses.size();
        for (size_t g = 0; g < G; ++g) {
            if (win_of[g] != (int)wi) continue;
            const GroupDesc& gd = h->groups[g];
            std::map<uint32_t, std::vector<uint32_t>> cls;  // in-window z bits -> terms
            for (uint32_t t = gd.begin; t < gd.end; ++t) cls[compress(h->t64[t].z & wins[wi])].push_back(t);
            auto it = cls.begin();
            while (it != cls.end()) {
                if (hclasses.size() - d.c_begin == (size_t)kHwMaxClasses) {  // pass full
                    d.g_end = (uint32_t)hgroups.size();
                    d.c_end = (uint32_t)hclasses.size();
                    passes.push_back(d);
                    d.g_begin = d.g_end;
                    d.c_begin = d.c_end;
                }
                HwGroup hg{};
                hg.xl = compress(gd.x);
                int u = 0;
                hg.cb[0] = (uint32_t)hclasses.size();
                for (; it != cls.end() && hclasses.size() - d.c_begin < (size_t)kHwMaxClasses; ++it) {
                    const int bucket = (int)(it->first >> kHwThreadBits);
                    while (u < bucket) hg.cb[++u] = (uint32_t)hclasses.size();
                    hg.zrm |= (uint32_t)bucket;
                    HwClass hc{};
                    hc.zt = it->first & tmask;
                    hc.k_begin = (uint32_t)ht64.size();
                    for (uint32_t t : it->second) {
                        const uint64_t zo = h->t64[t].z & ~wins[wi];
                        ht64.push_back(HwTerm<double>{zo, h->t64[t].cre, h->t64[t].cim});
                        ht32.push_back(HwTerm<float>{zo, h->t32[t].cre, h->t32[t].cim});
                    }
                    hc.k_end = (uint32_t)ht64.size();
                    hclasses.push_back(hc);
                }
                while (u < kBuckets) hg.cb[++u] = (uint32_t)hclasses.size();
                hgroups.push_back(hg);
            }
        }
        d.g_end = (uint32_t)hgroups.size();
        d.c_end = (uint32_t)hclasses.size();
        passes.push_back(d);
    }
    std::vector<uint64_t> hi;
    for (const auto& g : h->groups)
        if (g.x >> kTileBits) hi.push_back(g.x >> kTileBits);
    std::sort(hi.begin(), hi.end());
    const size_t D = std::unique(hi.begin(), hi.end()) - hi.begin();
    const size_t m = passes.size();
    h->hw_lam = 3 * m - 1 < D + 2;
    h->hw_energy = 2 * m < 2 + D;
    // batched mid-size states use the window passes whenever a cover exists
    // (their states stay in cache, so arithmetic, not bytes, decides)
    if (!h->hw_lam && !h->hw_energy && n > kMidMaxQubits) return;
    h->hw_wins.swap(passes);
    h->hw_groups.swap(hgroups);
    h->hw_classes.swap(hclasses);
    h->hw_t32.swap(ht32);
    h->hw_t64.swap(ht64);
}

// Blocks of a small Hamiltonian for the whole-state-in-LDS kernel: per group its
// terms sorted by their z bits on the kProgBits highest bits of the tile; a group
// that a block or a count of 255 cannot hold is continued in another of the same x.
template <typename T>
void plan_small(vqe_hamiltonian* h, const std::vector<TermDesc<T>>& terms, std::vector<SmallBlock>& blocks,
                std::vector<char>& stream) {
    const int sh = batch_bits(h->n) - kProgBits;
    auto room = [&] { return kProgBlock - blocks.back().bytes; };
    std::vector<uint32_t> order;
    for (const GroupDesc& g : h->groups) {
        uint32_t at[17] = {0};  // a counting sort
        for (uint32_t t = g.begin; t < g.end; ++t) ++at[1 + (h->z[t] >> sh)];
        for (int u = 0; u < 16; ++u) at[u + 1] += at[u];
        order.resize(g.end - g.begin);
        for (uint32_t t = g.begin; t < g.end; ++t) order[at[h->z[t] >> sh]++] = t;
        for (size_t i = 0; i < order.size();) {
            if (blocks.empty() || room() < sizeof(SmallGroup) + sizeof(SmallTerm<T>)) {
                SmallBlock b{};
                stream.resize((stream.size() + 15) / 16 * 16);
                b.off = (uint32_t)stream.size();
                blocks.push_back(b);
            }
            const size_t most = std::min((room() - sizeof(SmallGroup)) / sizeof(SmallTerm<T>), order.size() - i);
            SmallGroup sg{};
            sg.x = (uint32_t)g.x;
            const size_t start = stream.size();
            stream.resize(start + sizeof(SmallGroup) + most * sizeof(SmallTerm<T>));
            auto* tm = (SmallTerm<T>*)&stream[start + sizeof(SmallGroup)];
            for (; sg.n_terms < most; ++i, ++tm) {
                const uint32_t t = order[i], u = (uint32_t)(h->z[t] >> sh);
                if (((sg.count[u >> 2] >> (8 * (u & 3))) & 255u) == 255u) break;
                sg.count[u >> 2] += 1u << (8 * (u & 3));
                *tm = SmallTerm<T>{(uint32_t)h->z[t] & ((1u << sh) - 1), u, terms[t].cre, terms[t].cim};
                ++sg.n_terms;
            }
            stream.resize(start + sizeof(SmallGroup) + sg.n_terms * sizeof(SmallTerm<T>));
            std::memcpy(&stream[start], &sg, sizeof(sg));
            blocks.back().bytes = (uint32_t)(stream.size() - blocks.back().off);
            ++blocks.back().n_groups;
        }
    }
    // blocks are read 16 bytes at a time, the last one past its end
    stream.resize((stream.size() + 15) / 16 * 16);
}

// Per-block partial-sum buffer of a state: room for the largest launch
// (kMaxPartBlocks blocks x kMaxGradSlots slots).
size_t part_doubles() { return std::max((size_t)kMaxPartBlocks * kMaxGradSlots, (size_t)kMaxBlocks * 2); }

int ensure_part(vqe_state* s) {
    if (s->d_part) return VQE_OK;
    if (hipMalloc((void**)&s->d_part, part_doubles() * sizeof(double)) != hipSuccess) {
        s->d_part = nullptr;
        set_error("hipMalloc of the partial-sum buffer failed");
        return VQE_ERR_OOM;
    }
    return VQE_OK;
}

// Angle of gate g under params.
double angle_of(const Gate& g, const double* params) { return g.pidx >= 0 ? params[g.pidx] : g.angle; }

void half_angles(const vqe_circuit* c, const double* params, std::vector<HalfAngle>& h) {
    h.resize(c->gates.size());
    for (size_t i = 0; i < h.size(); ++i) {
        const double a = angle_of(c->gates[i], params) / 2;
        h[i] = HalfAngle{std::cos(a), std::sin(a)};
    }
}

template <typename T>
void fill_matrix(Mat2<T>& m, const Gate& g, double th, bool inverse) {
    if (inverse) th = -th;
    const double c = std::cos(th / 2), s = std::sin(th / 2);
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    switch (g.kind) {
        case VQE_GATE_RY:  // [[c, -s], [s, c]]
        case VQE_GATE_SEXC:  // the same rotation between the A and B patterns
        case VQE_GATE_DEXC:
            v[0] = c; v[2] = -s; v[4] = s; v[6] = c;
            break;
        case VQE_GATE_RZ:  // diag(e^{-i t/2}, e^{i t/2})
            v[0] = c; v[1] = -s; v[6] = c; v[7] = s;
            break;
        case VQE_GATE_RX:  // [[c, -i s], [-i s, c]]
            v[0] = c; v[3] = -s; v[5] = -s; v[6] = c;
            break;
        case VQE_GATE_H: {
            const double r = 1.0 / std::sqrt(2.0);
            v[0] = r; v[2] = r; v[4] = r; v[6] = -r;
            break;
        }
        default:
            break;
    }
    for (int i = 0; i < 8; ++i) m.v[i] = (T)v[i];
}

uint8_t mat_op(int kind) {
    switch (kind) {
        case VQE_GATE_RY: return OP_R2;
        case VQE_GATE_RZ: return OP_DIAG;
        case VQE_GATE_H: return OP_R2;
        default: return OP_U2;
    }
}

uint8_t grad_op(int kind) {
    switch (kind) {
        case VQE_GATE_RY: return OP_GY;
        case VQE_GATE_RZ: return OP_GZ;
        case VQE_GATE_SEXC: return OP_GPAIR2;
        case VQE_GATE_DEXC: return OP_GPAIR4;
        default: return OP_GX;
    }
}

bool is_excitation(int kind) { return kind == VQE_GATE_SEXC || kind == VQE_GATE_DEXC; }

int local_bit(const PlannedPass& p, int q) {
    for (int j = 0; j < p.K; ++j)
        if (p.pos[j] == q) return j;
    return -1;
}

// Appends the op that applies gate gi (or its inverse) to `ops`.
void emit_gate(const Gate& g, int gi, const PlannedPass& p, std::vector<KOp>& ops,
               std::vector<int>& mat_gate) {
    KOp op{};
    op.a = (uint8_t)local_bit(p, g.q0);
    switch (g.kind) {
        case VQE_GATE_CNOT:
            op.type = OP_CNOT;
            op.b = (uint8_t)local_bit(p, g.q1);
            break;
        case VQE_GATE_CZ:
            op.type = OP_CZ;
            op.b = (uint8_t)local_bit(p, g.q1);
            break;
        case VQE_GATE_X:
            op.type = OP_XFLIP;
            break;
        case VQE_GATE_SEXC:
        case VQE_GATE_DEXC:
            op.type = g.kind == VQE_GATE_SEXC ? OP_PAIR2 : OP_PAIR4;
            op.b = (uint8_t)local_bit(p, g.q1);
            if (g.kind == VQE_GATE_DEXC) {
                op.c = (uint8_t)local_bit(p, g.q2);
                op.d = (uint8_t)local_bit(p, g.q3);
            }
            op.slot = (uint8_t)mat_gate.size();
            mat_gate.push_back(gi);
            break;
        default:
            op.type = mat_op(g.kind);
            op.slot = (uint8_t)mat_gate.size();
            mat_gate.push_back(gi);
            // RY and RZ are plane rotations (of the amplitude pair, of each
            // amplitude's real and imaginary parts): the specialised reverse
            // kernels un-apply them as three shears (shear_coefficients)
            if (g.kind == VQE_GATE_RY || g.kind == VQE_GATE_RZ) op.c = 1;
            break;
    }
    ops.push_back(op);
}

template <typename T>
void build_args(const vqe_circuit* c, const Plan& pl, size_t pi, const double* params, bool reverse,
                PassArgs<T>& a) {
    const PlannedPass& p = pl.passes[pi];
    const PassOps& po = pl.ops[pi];
    std::memset(&a, 0, sizeof(a));
    a.K = (uint32_t)p.K;
    a.n_cosets = 1ull << (c->n - p.K);
    for (int j = 0; j < p.K; ++j) a.pos[j] = (uint32_t)p.pos[j];
    const int d = sizeof(T) == 8 ? 1 : 0;
    const int S = reverse ? po.S_r[d] : po.S_f[d];
    a.split = (uint32_t)S;
    const auto& mg = reverse ? po.rev_mat_gate : po.fwd_mat_gate;
    if (S == 0) {
        const auto& ops = reverse ? po.rev : po.fwd;
        a.n_ops = (uint32_t)ops.size();
        for (size_t i = 0; i < ops.size(); ++i) a.ops[i] = ops[i];
        for (int sl = 0; sl < p.K; ++sl) a.pos_in[sl] = a.pos_out[sl] = (uint32_t)p.pos[sl];
    } else {
        const SplitOps& so = reverse ? po.rev_l[d] : po.fwd_l[d];
        a.n_ops = (uint32_t)so.ops.size();
        for (size_t i = 0; i < so.ops.size(); ++i) a.ops[i] = so.ops[i];
        for (int sl = 0; sl < p.K; ++sl) {
            a.pos_in[sl] = (uint32_t)p.pos[so.map_in[sl]];
            a.pos_out[sl] = (uint32_t)p.pos[so.map_out[sl]];
        }
    }
    for (size_t i = 0; i < mg.size(); ++i) {
        const Gate& g = c->gates[mg[i]];
        fill_matrix(a.mats[i], g, angle_of(g, params), reverse);
    }
    a.n_gslots = reverse ? (uint32_t)po.slot_param.size() : 0;
}

int check_state(const vqe_state* s, const char* fn) {
    if (!s || !s->data) {
        set_error(std::string(fn) + ": null state");
        return VQE_ERR_ARG;
    }
    return VQE_OK;
}

int check_params(const vqe_circuit* c, const double* params, size_t n_params, const char* fn) {
    if (n_params != c->n_params) {
        set_error(std::string(fn) + ": n_params " + std::to_string(n_params) + " does not match the circuit's " +
                  std::to_string(c->n_params));
        return VQE_ERR_ARG;
    }
    if (n_params > 0 && !params) {
        set_error(std::string(fn) + ": null params");
        return VQE_ERR_ARG;
    }
    for (size_t i = 0; i < n_params; ++i)
        if (!std::isfinite(params[i])) {
            set_error(std::string(fn) + ": non-finite parameter");
            return VQE_ERR_ARG;
        }
    return VQE_OK;
}

std::mutex g_jit_plan_mu;

// The kernel form is process-wide and may change at any time: every entry point
// reads it once (jit_mode()) and hands it down, so that one evaluation keeps to
// one plan.

// True if an evaluation of c runs the specialised plan (see vqe_set_specialize).
bool use_specialised(const vqe_circuit* c, int form) {
    return form == VQE_SPECIALIZE_ALWAYS ||
           (form == VQE_SPECIALIZE_AUTO && (c->n >= VQE_SPECIALIZE_AUTO_MIN_QUBITS || c->has_excitation));
}

// VQE_OK if the kernel form can evaluate c (interpreted kernels have no
// excitation gates).
int check_form(const vqe_circuit* c, int form, const char* fn) {
    if (c->has_excitation && !use_specialised(c, form)) {
        set_error(std::string(fn) + ": excitation gates need specialised kernels (vqe_set_specialize)");
        return VQE_ERR_UNSUPPORTED;
    }
    return VQE_OK;
}

const Plan& plan_of(const vqe_circuit* c, int form) { return c->plan[use_specialised(c, form) ? 1 : 0]; }

// Physical ops, lane-split bits and slot positions of one specialised pass.
const std::vector<KOp>& jit_ops(const Plan& pl, size_t pi, int d, bool reverse, int* S, JitArgs* a, int n) {
    const PlannedPass& p = pl.passes[pi];
    const PassOps& po = pl.ops[pi];
    *S = reverse ? po.S_r[d] : po.S_f[d];
    if (a) {
        std::memset(a, 0, sizeof(*a));
        a->n_cosets = 1ull << (n - p.K);
        for (int j = 0; j < p.K; ++j) a->pos[j] = (uint32_t)p.pos[j];
    }
    if (*S == 0) {
        if (a)
            for (int j = 0; j < p.K; ++j) a->pos_in[j] = a->pos_out[j] = (uint32_t)p.pos[j];
        return reverse ? po.rev : po.fwd;
    }
    const SplitOps& so = reverse ? po.rev_l[d] : po.fwd_l[d];
    if (a)
        for (int sl = 0; sl < p.K; ++sl) {
            a->pos_in[sl] = (uint32_t)p.pos[so.map_in[sl]];
            a->pos_out[sl] = (uint32_t)p.pos[so.map_out[sl]];
        }
    return so.ops;
}

// Compiles and loads the specialised kernels of every pass of a specialised
// plan for dtype index d on the current device (once; cached).
int ensure_jit(const vqe_circuit* c, const Plan& cpl, int d) {
    Plan& pl = const_cast<Plan&>(cpl);
    int dev = 0;
    VQE_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(g_jit_plan_mu);
    const size_t P = pl.passes.size();
    if (pl.jit_dev[d] == dev && pl.jfn[d][0].size() == P) return VQE_OK;
    std::vector<std::string> srcs(2 * P);
    for (size_t pi = 0; pi < P; ++pi)
        for (int dir = 0; dir < 2; ++dir) {
            int S = 0;
            const auto& ops = jit_ops(pl, pi, d, dir == 1, &S, nullptr, c->n);
            srcs[2 * pi + dir] = jit_source(d == 1, pl.passes[pi].K, S, dir == 1 ? 2 : 1, ops,
                                            dir == 1 ? (uint32_t)pl.ops[pi].slot_param.size() : 0);
        }
    std::vector<void*> fns;
    std::string err;
    const int rc = jit_prepare(srcs, fns, err);
    if (rc) {
        set_error(err);
        return rc;
    }
    for (int dir = 0; dir < 2; ++dir) {
        pl.jfn[d][dir].assign(P, nullptr);
        for (size_t pi = 0; pi < P; ++pi) pl.jfn[d][dir][pi] = fns[2 * pi + dir];
    }
    pl.jit_dev[d] = dev;
    return VQE_OK;
}

// True if an evaluation of c runs tile passes: the specialised form from
// kTileMinQubits qubits on (below, a tile would leave most of the chip idle;
// the 7-qubit window passes remain).
bool use_tiles(const vqe_circuit* c, int form) { return use_specialised(c, form) && c->n >= kTileMinQubits; }

// Plans the tile passes of c for dtype index d, generates their kernels and
// loads them on the current device (once).
int ensure_tiles(const vqe_circuit* cc, int d) {
    vqe_circuit* c = const_cast<vqe_circuit*>(cc);
    TilePlan& tp = c->tile[d];
    int dev = 0;
    VQE_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(g_jit_plan_mu);
    if (tp.ready && tp.dev == dev) return VQE_OK;
    TilePlan np;
    std::string msg;
    const TileShape sh = tile_shape(d == 1, c->n);
    if (!plan_tiles(c->n, c->gates, TileLimits{sh.T, sh.low, kTileMaxGates, kTileMaxPushes}, np.passes, msg)) {
        set_error(msg);
        return VQE_ERR_STATE;
    }
    const size_t P = np.passes.size();
    std::vector<std::string> srcs;
    for (int dir = 0; dir < 2; ++dir) {
        np.k[dir].resize(P);
        for (size_t p = 0; p < P; ++p) {
            TileKernel& k = np.k[dir][p];
            if (!tile_kernel(d == 1, sh, c->gates, np.passes[p], dir, k, msg)) {
                set_error(msg);
                return VQE_ERR_STATE;
            }
            srcs.push_back(std::move(k.src));
            k.src.clear();
            np.tab_off[dir].push_back(np.tab_total);
            np.tab_total += (k.n_scalars + 15) / 16 * 16;  // whole cache lines per pass
            np.L = std::max(np.L, (uint32_t)k.lane_param.size());
        }
    }
    std::vector<void*> fns;
    if (int rc = jit_prepare(srcs, fns, msg)) {
        set_error(msg);
        return rc;
    }
    np.fn[0].assign(fns.begin(), fns.begin() + (long)P);
    np.fn[1].assign(fns.begin() + (long)P, fns.end());
    np.dev = dev;
    np.ready = true;
    tp = std::move(np);
    return VQE_OK;
}

// The state's matrix table (device) and its pinned staging copy, at least
// `bytes` long; waits until the previous upload from the staging copy is done.
int stage_mats(vqe_state* s, size_t bytes) {
    if (!s->mats_ev) VQE_HIP(hipEventCreateWithFlags(&s->mats_ev, hipEventDisableTiming));
    if (bytes > s->mats_cap) {
        VQE_HIP(hipStreamSynchronize(s->stream));
        if (s->d_mats) VQE_HIP(hipFree(s->d_mats));
        if (s->h_mats) VQE_HIP(hipHostFree(s->h_mats));
        s->d_mats = s->h_mats = nullptr;
        s->mats_cap = 0;
        if (hipMalloc(&s->d_mats, bytes) != hipSuccess || hipHostMalloc(&s->h_mats, bytes) != hipSuccess) {
            set_error("allocation of the matrix table failed");
            return VQE_ERR_OOM;
        }
        s->mats_cap = bytes;
    } else {
        VQE_HIP(hipEventSynchronize(s->mats_ev));
    }
    return VQE_OK;
}

// A plane rotation by a (x' = x cos a - y sin a, y' = x sin a + y cos a) as
// three shears x += k1 y, y += k2 x, x += k1 y with k1 = -tan(a/2) and
// k2 = sin a (Paeth's decomposition; three fused multiply-adds per plane
// instead of two products and two FMAs).  a is first brought into
// [-pi/2, pi/2] by a half turn, R(a) = -R(a -+ pi), so |k1|, |k2| <= 1;
// returns whether that flipped the sign.
template <typename T>
bool shear_coefficients(double a, Mat2<T>& m) {
    bool flip = false;
    if (a > M_PI / 2) {
        a -= M_PI;
        flip = true;
    } else if (a < -M_PI / 2) {
        a += M_PI;
        flip = true;
    }
    std::memset(&m, 0, sizeof(m));
    m.v[0] = (T)-std::tan(a / 2);
    m.v[1] = (T)std::sin(a);
    return flip;
}

// Fills the tables of a circuit's tile passes (both directions) for these
// parameters and uploads them on the state's stream; norm: see turn_limit().
template <typename T>
int upload_tables(vqe_state* s, const vqe_circuit* c, const TilePlan& tp, const double* params, double norm, const T** out) {
    const size_t bytes = std::max<size_t>(tp.tab_total, 1) * sizeof(T);
    if (int rc = stage_mats(s, bytes)) return rc;
    std::vector<HalfAngle> h;
    half_angles(c, params, h);
    const double limit = turn_limit(sizeof(T) == 8, norm);
    for (int dir = 0; dir < 2; ++dir)
        for (size_t p = 0; p < tp.passes.size(); ++p)
            fill_tile_table<T>(tp.k[dir][p], c->gates, h.data(), limit, dir, (T*)s->h_mats + tp.tab_off[dir][p]);
    VQE_HIP(hipMemcpyAsync(s->d_mats, s->h_mats, bytes, hipMemcpyHostToDevice, s->stream));
    VQE_HIP(hipEventRecord(s->mats_ev, s->stream));
    *out = (const T*)s->d_mats;
    return VQE_OK;
}

// Fills the matrix table of a specialised plan (every pass, both directions)
// for these parameters and uploads it on the state's stream.  The pinned
// staging buffer is reused only after its previous upload has completed.
template <typename T>
int upload_mats(vqe_state* s, const vqe_circuit* c, const Plan& pl, const double* params, const Mat2<T>** out) {
    const size_t bytes = std::max<size_t>(pl.mat_total, 1) * sizeof(Mat2<T>);
    if (int rc = stage_mats(s, bytes)) return rc;
    Mat2<T>* h = (Mat2<T>*)s->h_mats;
    s->rev_flip.assign(pl.passes.size(), 0);
    for (size_t pi = 0; pi < pl.passes.size(); ++pi)
        for (int dir = 0; dir < 2; ++dir) {
            const auto& mg = dir ? pl.ops[pi].rev_mat_gate : pl.ops[pi].fwd_mat_gate;
            Mat2<T>* m = h + pl.mat_off[2 * pi + dir];
            for (size_t i = 0; i < mg.size(); ++i) {
                const Gate& g = c->gates[mg[i]];
                if (dir == 1 && (g.kind == VQE_GATE_RY || g.kind == VQE_GATE_RZ)) {
                    // the inverse as a rotation: RY^-1 turns (a_0, a_1), RZ^-1 turns
                    // (Re, Im) of an amplitude with bit 0 (bit 1 by the opposite angle).
                    // Every amplitude takes part, so a half turn is a sign on the whole
                    // state; an excitation turns only its (A, B) patterns, where a half
                    // turn would not be, so excitations keep the matrix form.
                    Mat2<double> u;
                    fill_matrix(u, g, angle_of(g, params), true);
                    const double a = g.kind == VQE_GATE_RY ? std::atan2(u.v[4], u.v[0]) : std::atan2(u.v[1], u.v[0]);
                    s->rev_flip[pi] ^= (int8_t)shear_coefficients(a, m[i]);
                } else {
                    fill_matrix(m[i], g, angle_of(g, params), dir == 1);
                }
            }
        }
    VQE_HIP(hipMemcpyAsync(s->d_mats, s->h_mats, bytes, hipMemcpyHostToDevice, s->stream));
    VQE_HIP(hipEventRecord(s->mats_ev, s->stream));
    *out = (const Mat2<T>*)s->d_mats;
    return VQE_OK;
}

// psi <- U psi on one dense window (see DenseArgs).
template <typename T>
int apply_dense(vqe_state* s, const DenseArgs& a, const double* u) {
    constexpr int P = 1 << kDenseK, RR = 2 * P;
    if (int rc = stage_mats(s, sizeof(T) * RR * RR)) return rc;
    T* h = (T*)s->h_mats;
    for (int r = 0; r < P; ++r)
        for (int c = 0; c < P; ++c) {
            const double re = u[2 * (r * P + c)], im = u[2 * (r * P + c) + 1];
            h[r * RR + c] = (T)re;
            h[r * RR + P + c] = (T)-im;
            h[(P + r) * RR + c] = (T)im;
            h[(P + r) * RR + P + c] = (T)re;
        }
    VQE_HIP(hipMemcpyAsync(s->d_mats, s->h_mats, sizeof(T) * RR * RR, hipMemcpyHostToDevice, s->stream));
    VQE_HIP(hipEventRecord(s->mats_ev, s->stream));
    ProfScope ps(VQE_KERNEL_DENSE, 2.0 * (double)s->bytes, s->stream);
    VQE_HIP(launch_dense<T>(a, (const T*)s->d_mats, s->data, s->data, s->stream));
    return VQE_OK;
}

void tile_args(const PlannedPass& p, int n, TileArgs& a) {
    std::memset(&a, 0, sizeof(a));
    a.n_units = 1ull << (n - p.K);
    for (int j = 0; j < p.K; ++j) a.pos[j] = (uint32_t)p.pos[j];
}

template <typename T>
int forward_tiles(vqe_state* s, const vqe_circuit* c, const double* params, const std::vector<size_t>& bounds,
                  const std::vector<void*>& ckpt_ptr, bool zero, double norm, int chunk) {
    const int d = sizeof(T) == 8 ? 1 : 0;
    const TilePlan& tp = c->tile[d];
    const T* tab = nullptr;
    if (int rc = upload_tables<T>(s, c, tp, params, norm, &tab)) return rc;
    if (zero && tp.passes.empty()) VQE_HIP(launch_set_basis(s->dtype, s->data, 1ull << s->n, 0, s->stream));
    void* cur = s->data;
    TileArgs a;
    for (size_t pi = 0; pi < tp.passes.size(); ++pi) {
        void* out = s->data;
        for (size_t k = 0; k < bounds.size(); ++k)
            if (bounds[k] == pi + 1) out = ckpt_ptr[k];
        ProfScope ps(VQE_KERNEL_WINDOW_FWD, (zero && pi == 0 ? 1.0 : 2.0) * (double)s->bytes, s->stream);
        tile_args(tp.passes[pi], s->n, a);
        a.first = zero && pi == 0 ? 1u : 0u;
        VQE_HIP(launch_tile(tp.fn[0][pi], a, false, tab + tp.tab_off[0][pi], cur, out, nullptr, nullptr, nullptr, 0,
                            s->stream));
        ps.end();
        cur = out;
        if (chunk > 0 && (pi + 1) % (size_t)chunk == 0 && pi + 1 < tp.passes.size())
            VQE_HIP(hipStreamSynchronize(s->stream));
    }
    return VQE_OK;
}

// Forward passes from |0...0> (zero) or in place on the current state.
// ckpt_ptr[k] receives the state at boundary bounds[k] (pass index + 1); norm:
// bound on the 2-norms of the vectors of this evaluation (turn_limit()).
template <typename T>
int forward(vqe_state* s, const vqe_circuit* c, int form, const double* params, const std::vector<size_t>& bounds,
            const std::vector<void*>& ckpt_ptr, bool zero, double norm, int chunk = 0) {
    const int d = sizeof(T) == 8 ? 1 : 0;
    if (use_tiles(c, form)) {
        if (int rc = ensure_tiles(c, d)) return rc;
        return forward_tiles<T>(s, c, params, bounds, ckpt_ptr, zero, norm, chunk);
    }
    const Plan& pl = plan_of(c, form);
    void* cur = s->data;
    const Mat2<T>* mats = nullptr;
    if (pl.jit) {
        int rc = ensure_jit(c, pl, d);
        if (!rc) rc = upload_mats<T>(s, c, pl, params, &mats);
        if (rc) return rc;
    }
    if (zero) VQE_HIP(launch_set_basis(s->dtype, s->data, 1ull << s->n, 0, s->stream));
    PassArgs<T> a;
    JitArgs ja;
    for (size_t pi = 0; pi < pl.passes.size(); ++pi) {
        void* out = s->data;
        for (size_t k = 0; k < bounds.size(); ++k)
            if (bounds[k] == pi + 1) out = ckpt_ptr[k];
        ProfScope ps(VQE_KERNEL_WINDOW_FWD, 2.0 * (double)s->bytes, s->stream);
        if (pl.jit) {
            int S = 0;
            jit_ops(pl, pi, d, false, &S, &ja, s->n);
            VQE_HIP(launch_window_jit(pl.jfn[d][0][pi], ja, S, mats + pl.mat_off[2 * pi], false, cur, out, nullptr,
                                      nullptr, nullptr, nullptr, s->stream));
        } else {
            build_args<T>(c, pl, pi, params, false, a);
            VQE_HIP(launch_window_fwd<T>(a, s->n, cur, out, s->stream));
        }
        ps.end();
        cur = out;
        if (chunk > 0 && (pi + 1) % (size_t)chunk == 0 && pi + 1 < pl.passes.size())
            VQE_HIP(hipStreamSynchronize(s->stream));
    }
    return VQE_OK;
}

template <typename T>
const TermDesc<T>* terms_of(const vqe_hamiltonian* h);
template <>
const TermDesc<float>* terms_of<float>(const vqe_hamiltonian* h) { return h->d_t32; }
template <>
const TermDesc<double>* terms_of<double>(const vqe_hamiltonian* h) { return h->d_t64; }

template <typename T>
const HwTerm<T>* hw_terms_of(const vqe_hamiltonian* h);
template <>
const HwTerm<float>* hw_terms_of<float>(const vqe_hamiltonian* h) { return h->d_hw_t32; }
template <>
const HwTerm<double>* hw_terms_of<double>(const vqe_hamiltonian* h) { return h->d_hw_t64; }

double hpsi_bytes(const vqe_hamiltonian* h, const vqe_state* s, bool write);

// lam = H psi with the energy partials reduced into d_out[0..1]
// (Re<psi|lam>, <psi|psi>): window passes when planned, else the tile kernel.
// chunk > 0: waits for the stream after that many window passes, as the sweeps
// do.  A molecule-shaped Hamiltonian of 28 qubits runs tens of them, two blocks
// on every CU: queued at once they held the small requests of the served stream
// back for all of their time (12 qubits p99 29 ms at 58.6 requests/s, 16 qubits
// 53; 6 and 14 with one pass at a time here too).
template <typename T>
int apply_h(vqe_state* psi, void* lam, const vqe_hamiltonian* h, double* d_out, int chunk = 0) {
    hipStream_t st = psi->stream;
    uint32_t nb = 0;
    if (h->hw_lam) {
        const size_t m = h->hw_wins.size();
        for (size_t wi = 0; wi < m; ++wi) {
            ProfScope ps(VQE_KERNEL_HPSI, (wi ? 3.0 : 2.0) * (double)psi->bytes, st);
            VQE_HIP(launch_hwin<T>(psi->n, h->hw_wins[wi], psi->data, lam, h->d_hw_groups, h->d_hw_classes,
                                   hw_terms_of<T>(h), h->real_coeffs,
                                   wi == 0, wi + 1 == m, psi->d_part, &nb, st));
            ps.end();
            if (chunk > 0 && (wi + 1) % (size_t)chunk == 0 && wi + 1 < m) VQE_HIP(hipStreamSynchronize(st));
        }
    } else {
        ProfScope ps(VQE_KERNEL_HPSI, hpsi_bytes(h, psi, true), st);
        VQE_HIP(launch_hpsi<T>(psi->n, psi->data, lam, h->d_groups, (uint32_t)h->groups.size(), terms_of<T>(h), 0,
                               (uint32_t)kMaxPartBlocks, psi->d_part, &nb, st));
    }
    VQE_HIP(launch_reduce(psi->d_part, nb, 2, nullptr, d_out, 0, st));
    return VQE_OK;
}

// Algorithmic bytes of one H psi sweep: own tile + one partner tile per
// distinct out-of-tile partner offset (x >> tile bits), plus the write of lam.
// The energy-only sweep visits each out-of-tile pair once (half the partners).
double hpsi_bytes(const vqe_hamiltonian* h, const vqe_state* s, bool write) {
    const int tb = s->n < kTileBits ? s->n : kTileBits;
    std::vector<uint64_t> hi;
    for (const auto& g : h->groups) {
        const uint64_t xh = g.x >> tb;
        if (xh && (hi.empty() || hi.back() != xh)) hi.push_back(xh);
    }
    std::sort(hi.begin(), hi.end());
    const size_t D = std::unique(hi.begin(), hi.end()) - hi.begin();
    const double S = (double)s->bytes;
    return write ? (1.0 + (double)D) * S + S : (1.0 + 0.5 * (double)D) * S;
}

// Grouped energy sums (Re<psi|H|psi>, <psi|psi>) reduced into sums[0..1]
// on the device, with per-block partials in part (at most
// energy_part_blocks() blocks of 2): m energy-only window passes (m S read;
// per pass, its partials reduced and added in pass order) or one tile sweep
// that visits each out-of-tile pair once ((1 + D/2) S read).
uint32_t energy_part_blocks(const vqe_hamiltonian* h, int n) {
    return h->hw_energy ? hwin_blocks(n) : hpsi_blocks(n, kEnergyPartBlocks);
}

template <typename T>
int energy_grouped(vqe_state* s, const vqe_hamiltonian* h, double* part, double* sums) {
    uint32_t nb = 0;
    if (h->hw_energy) {
        const size_t m = h->hw_wins.size();
        for (size_t wi = 0; wi < m; ++wi) {
            ProfScope ps(VQE_KERNEL_EXPECT_HALF, (double)s->bytes, s->stream);
            VQE_HIP(launch_hwin<T>(s->n, h->hw_wins[wi], s->data, nullptr, h->d_hw_groups, h->d_hw_classes,
                                   hw_terms_of<T>(h), h->real_coeffs, wi == 0, wi + 1 == m, part, &nb, s->stream));
            ps.end();
            VQE_HIP(launch_reduce(part, nb, 2, nullptr, sums, wi ? 1 : 0, s->stream));
        }
        return VQE_OK;
    }
    {
        ProfScope ps(VQE_KERNEL_EXPECT_HALF, hpsi_bytes(h, s, false), s->stream);
        VQE_HIP(launch_hpsi<T>(s->n, s->data, nullptr, h->d_groups, (uint32_t)h->groups.size(), terms_of<T>(h), 1,
                               kEnergyPartBlocks, part, &nb, s->stream));
    }
    VQE_HIP(launch_reduce(part, nb, 2, nullptr, sums, 0, s->stream));
    return VQE_OK;
}

// Per-term partials: d_res[off + 2t] = <P_t>, d_res[off + 2t + 1] = norm.
template <typename T>
int energy_per_term(vqe_state* s, const vqe_hamiltonian* h, size_t off) {
    for (size_t t = 0; t < h->w.size(); ++t) {
        uint32_t nb = 0;
        ProfScope ps(VQE_KERNEL_PER_TERM, (double)s->bytes, s->stream);
        VQE_HIP(launch_expect_term<T>(s->n, s->data, h->x[t], h->z[t], s->d_part, &nb, s->stream));
        ps.end();
        VQE_HIP(launch_reduce(s->d_part, nb, 2, nullptr, s->d_res + off + 2 * t, 0, s->stream));
    }
    return VQE_OK;
}

double combine_per_term(const vqe_hamiltonian* h, const double* r, double* norm) {
    double e = 0.0;
    for (size_t t = 0; t < h->w.size(); ++t) e += h->w[t] * r[2 * t];
    *norm = h->w.empty() ? 0.0 : r[1];
    return e;
}

template <typename T>
int expect_impl(vqe_state* s, const vqe_hamiltonian* h, int mode, double* energy, double* norm) {
    const size_t need = mode == VQE_EXPECT_PER_TERM ? 2 * h->w.size() + 2 : 2;
    int rc = ensure_res(s, need);
    if (rc) return rc;
    if (mode == VQE_EXPECT_PER_TERM) {
        if (h->w.empty()) {
            set_error("vqe_expect_pauli: empty Hamiltonian");
            return VQE_ERR_ARG;
        }
        rc = energy_per_term<T>(s, h, 0);
        if (rc) return rc;
        VQE_HIP(hipMemcpyAsync(s->h_res, s->d_res, 2 * h->w.size() * sizeof(double), hipMemcpyDeviceToHost, s->stream));
        VQE_HIP(hipStreamSynchronize(s->stream));
        double nrm = 0.0;
        const double e = combine_per_term(h, s->h_res, &nrm);
        *energy = e / nrm;
        if (norm) *norm = nrm;
    } else {
        rc = energy_grouped<T>(s, h, s->d_part, s->d_res);
        if (rc) return rc;
        VQE_HIP(hipMemcpyAsync(s->h_res, s->d_res, 2 * sizeof(double), hipMemcpyDeviceToHost, s->stream));
        VQE_HIP(hipStreamSynchronize(s->stream));
        *energy = s->h_res[0] / s->h_res[1];
        if (norm) *norm = s->h_res[1];
    }
    return VQE_OK;
}

// Reverse tile passes on (psi, lam): column sums of the gradient terms of pass
// p to sums[p L ..].
template <typename T>
int reverse_tiles(vqe_state* psi, vqe_state* lam, const TilePlan& tp, const std::vector<size_t>& bounds,
                  const std::vector<void*>& ck, double* sums, int chunk) {
    const size_t P = tp.passes.size();
    const T* tab = (const T*)psi->d_mats;  // uploaded by forward_tiles()
    hipStream_t st = psi->stream;
    TileArgs a;
    size_t waiting = 0;  // passes whose partials wait in d_part, the last of them pi
    for (size_t pi = P; pi-- > 0;) {
        const void* pin = psi->data;
        for (size_t k = 0; k < bounds.size(); ++k)
            if (bounds[k] == pi + 1) pin = ck[k];
        tile_args(tp.passes[pi], psi->n, a);
        const uint32_t nb = tile_blocks(a.n_units, true);
        const size_t room = part_doubles() / ((size_t)nb * std::max(tp.L, 1u));  // passes that d_part holds
        ProfScope ps(VQE_KERNEL_WINDOW_REV, 4.0 * (double)psi->bytes, st);
        // the partials lie in ascending pass order, so a group is filled from its end
        const size_t group = std::min(room, waiting + pi + 1);
        ++waiting;
        VQE_HIP(launch_tile(tp.fn[1][pi], a, true, tab + tp.tab_off[1][pi], pin, psi->data, lam->data, lam->data,
                            psi->d_part + (group - waiting) * (size_t)nb * tp.L, tp.L, st));
        ps.end();
        if (waiting == group) {
            VQE_HIP(launch_tile_reduce(psi->d_part, (uint32_t)waiting, nb, tp.L, sums + pi * tp.L, st));
            waiting = 0;
        }
        if (chunk > 0 && (P - pi) % (size_t)chunk == 0 && pi > 0) VQE_HIP(hipStreamSynchronize(st));
    }
    return VQE_OK;
}

template <typename T>
int adjoint_impl(vqe_state* psi, vqe_state* lam, const vqe_circuit* c, int form, const double* params,
                 const vqe_hamiltonian* h, const vqe_grad_opts* o, double* energy, double* grad) {
    const int d = sizeof(T) == 8 ? 1 : 0;
    const bool tiles = use_tiles(c, form);
    const Plan& pl = plan_of(c, form);
    if (int rc0 = tiles ? ensure_tiles(c, d) : upload_plan(pl)) return rc0;
    const TilePlan& tp = c->tile[d];
    const size_t P = tiles ? tp.passes.size() : pl.passes.size();
    std::vector<size_t> bounds;
    std::vector<void*> ck;
    const int nck = o ? o->n_ckpt : 0;
    for (int k = 0; k < nck; ++k) {
        size_t b = (size_t)std::llround((double)(k + 1) * (double)P / (double)(nck + 1));
        if (b < 1 || b >= P) continue;
        if (std::find(bounds.begin(), bounds.end(), b) != bounds.end()) continue;
        bounds.push_back(b);
        ck.push_back(o->ckpt[k]->data);
    }
    const size_t n_sums = tiles ? P * tp.L : c->n_params;  // tile passes: column sums, added up by parameter at the end
    int rc = ensure_res(psi, 2 + n_sums);
    if (rc) return rc;
    double* d_e = psi->d_res;
    double* d_g = psi->d_res + 2;
    hipStream_t st = psi->stream;
    const int chunk = o && o->chunk_passes > 0 ? o->chunk_passes : 0;
    rc = forward<T>(psi, c, form, params, bounds, ck, true, h->norm1, chunk);
    if (rc) return rc;
    if (chunk) VQE_HIP(hipStreamSynchronize(st));
    rc = apply_h<T>(psi, lam->data, h, d_e, chunk);
    if (rc) return rc;
    if (chunk) VQE_HIP(hipStreamSynchronize(st));
    if (tiles) {
        rc = reverse_tiles<T>(psi, lam, tp, bounds, ck, d_g, chunk);
        if (rc) return rc;
        VQE_HIP(hipMemcpyAsync(psi->h_res, psi->d_res, (2 + n_sums) * sizeof(double), hipMemcpyDeviceToHost, st));
        VQE_HIP(hipStreamSynchronize(st));
        const double nrm = psi->h_res[1];
        *energy = psi->h_res[0] / nrm;
        std::fill(grad, grad + c->n_params, 0.0);
        for (size_t pi = 0; pi < P; ++pi) {
            const std::vector<int32_t>& lp = tp.k[1][pi].lane_param;
            for (size_t l = 0; l < lp.size(); ++l)
                if (lp[l] >= 0) grad[lp[l]] += psi->h_res[2 + pi * tp.L + l] / nrm;
        }
        return VQE_OK;
    }
    VQE_HIP(launch_zero(d_g, c->n_params, st));
    const Mat2<T>* mats = (const Mat2<T>*)psi->d_mats;  // uploaded by forward()
    PassArgs<T> a;
    JitArgs ja;
    // Half turns of the sheared rotations flip psi and lam together, so the
    // gradient terms (bilinear in them) keep their sign until psi is restored
    // from a checkpoint; from there on they carry the flips made before it.
    bool flipped = false, grad_neg = false;
    for (size_t pi = P; pi-- > 0;) {
        const void* pin = psi->data;
        for (size_t k = 0; k < bounds.size(); ++k)
            if (bounds[k] == pi + 1) pin = ck[k];
        if (pl.jit && pin != psi->data) grad_neg = flipped;
        uint32_t gb = 0;
        const uint32_t n_gslots = (uint32_t)pl.ops[pi].slot_param.size();
        ProfScope ps(VQE_KERNEL_WINDOW_REV, 4.0 * (double)psi->bytes, st);
        if (pl.jit) {
            int S = 0;
            jit_ops(pl, pi, d, true, &S, &ja, psi->n);
            VQE_HIP(launch_window_jit(pl.jfn[d][1][pi], ja, S, mats + pl.mat_off[2 * pi + 1], true, pin, psi->data,
                                      lam->data, lam->data, psi->d_part, &gb, st));
        } else {
            build_args<T>(c, pl, pi, params, true, a);
            VQE_HIP(launch_window_rev<T>(a, psi->n, pin, psi->data, lam->data, lam->data, psi->d_part, &gb, st));
        }
        ps.end();
        if (n_gslots)
            VQE_HIP(launch_reduce(psi->d_part, gb, n_gslots, pl.d_slotmap + pl.slot_off[pi], d_g, grad_neg ? -1 : 1,
                                  st));
        if (pl.jit && psi->rev_flip[pi]) flipped = !flipped;
        if (chunk > 0 && (P - pi) % (size_t)chunk == 0 && pi > 0) VQE_HIP(hipStreamSynchronize(st));
    }
    VQE_HIP(hipMemcpyAsync(psi->h_res, psi->d_res, (2 + c->n_params) * sizeof(double), hipMemcpyDeviceToHost, st));
    VQE_HIP(hipStreamSynchronize(st));
    const double nrm = psi->h_res[1];
    *energy = psi->h_res[0] / nrm;
    for (size_t k = 0; k < c->n_params; ++k) grad[k] = psi->h_res[2 + k] / nrm;
    return VQE_OK;
}

template <typename T>
int param_shift_impl(vqe_state* psi, const vqe_circuit* c, int form, const double* params, const vqe_hamiltonian* h,
                     int mode, double* energy, double* grad) {
    // Shift rule per parameter: two runs at +-pi/2 for the rotations (their
    // generators square to one); four runs at +-pi/2 and +-3pi/2 for the
    // excitation gates, whose generators have eigenvalues 0 and +-1 (the
    // four-term rule of Anselmetti et al. 2021).
    const size_t P = c->n_params;
    std::vector<char> exc(P, 0);
    for (const Gate& g : c->gates)
        if (g.pidx >= 0 && is_excitation(g.kind)) exc[g.pidx] = 1;
    std::vector<std::pair<size_t, double>> shifts;  // evaluation e >= 1: (parameter, shift)
    for (size_t k = 0; k < P; ++k) {
        shifts.push_back({k, M_PI / 2});
        shifts.push_back({k, -M_PI / 2});
        if (exc[k]) {
            shifts.push_back({k, 3 * M_PI / 2});
            shifts.push_back({k, -3 * M_PI / 2});
        }
    }
    const size_t per = mode == VQE_EXPECT_PER_TERM ? 2 * h->w.size() : 2;
    const size_t n_eval = 1 + shifts.size();
    int rc = ensure_res(psi, per * n_eval);
    if (rc) return rc;
    std::vector<double> th(params, params + P);
    const std::vector<size_t> nob;
    const std::vector<void*> nock;
    // Evaluation 0 last so that psi ends in U(theta)|0>.
    for (size_t e = n_eval; e-- > 0;) {
        std::copy(params, params + P, th.begin());
        if (e > 0) th[shifts[e - 1].first] += shifts[e - 1].second;
        rc = forward<T>(psi, c, form, th.data(), nob, nock, true, 1.0);
        if (rc) return rc;
        rc = mode == VQE_EXPECT_PER_TERM ? energy_per_term<T>(psi, h, e * per)
                                         : energy_grouped<T>(psi, h, psi->d_part, psi->d_res + e * per);
        if (rc) return rc;
    }
    VQE_HIP(hipMemcpyAsync(psi->h_res, psi->d_res, per * n_eval * sizeof(double), hipMemcpyDeviceToHost, psi->stream));
    VQE_HIP(hipStreamSynchronize(psi->stream));
    std::vector<double> E(n_eval);
    for (size_t e = 0; e < n_eval; ++e) {
        const double* r = psi->h_res + e * per;
        if (mode == VQE_EXPECT_PER_TERM) {
            double nrm = 0.0;
            const double v = combine_per_term(h, r, &nrm);
            E[e] = v / nrm;
        } else {
            E[e] = r[0] / r[1];
        }
    }
    *energy = E[0];
    const double d1 = (std::sqrt(2.0) + 1) / (4 * std::sqrt(2.0)), d2 = (std::sqrt(2.0) - 1) / (4 * std::sqrt(2.0));
    size_t e = 1;
    for (size_t k = 0; k < P; ++k) {
        if (exc[k]) {
            grad[k] = d1 * (E[e] - E[e + 1]) - d2 * (E[e + 2] - E[e + 3]);
            e += 4;
        } else {
            grad[k] = 0.5 * (E[e] - E[e + 1]);
            e += 2;
        }
    }
    return VQE_OK;
}


void free_circuit(vqe_circuit* c) {
    if (!c) return;
    for (auto& pl : c->plan)
        if (pl.d_slotmap) (void)hipFree(pl.d_slotmap);
    delete c;
}

// Plans fused passes within the given limits and lowers them to kernel op
// lists (forward, and reverse with gradient ops), per dtype also to the
// lane-split layout.
int build_plan(vqe_circuit* c, const PlanLimits& lim, bool jit, Plan& pl) {
    std::string msg;
    pl.jit = jit;
    if (!plan_passes(c->n, c->gates, lim, pl.passes, msg)) {
        set_error("vqe_circuit_create: " + msg);
        return VQE_ERR_STATE;
    }
    std::vector<int32_t>& slotmap = pl.slotmap;
    pl.ops.resize(pl.passes.size());
    for (size_t pi = 0; pi < pl.passes.size(); ++pi) {
        const PlannedPass& p = pl.passes[pi];
        PassOps& po = pl.ops[pi];
        for (int gi : p.gates) emit_gate(c->gates[gi], gi, p, po.fwd, po.fwd_mat_gate);
        std::map<int, int> pslot;
        for (auto it = p.gates.rbegin(); it != p.gates.rend(); ++it) {
            const Gate& g = c->gates[*it];
            if (g.pidx >= 0) {
                auto f = pslot.find(g.pidx);
                int slot;
                if (f == pslot.end()) {
                    slot = (int)po.slot_param.size();
                    pslot[g.pidx] = slot;
                    po.slot_param.push_back(g.pidx);
                } else {
                    slot = f->second;
                }
                KOp gop{};
                gop.type = grad_op(g.kind);
                gop.a = (uint8_t)local_bit(p, g.q0);
                if (is_excitation(g.kind)) gop.b = (uint8_t)local_bit(p, g.q1);
                if (g.kind == VQE_GATE_DEXC) {
                    gop.c = (uint8_t)local_bit(p, g.q2);
                    gop.d = (uint8_t)local_bit(p, g.q3);
                }
                gop.slot = (uint8_t)slot;
                po.rev.push_back(gop);
            }
            emit_gate(g, *it, p, po.rev, po.rev_mat_gate);
        }
        pl.slot_off.push_back(slotmap.size());
        slotmap.insert(slotmap.end(), po.slot_param.begin(), po.slot_param.end());
        pl.mat_off.push_back(pl.mat_total);
        pl.mat_total += po.fwd_mat_gate.size();
        pl.mat_off.push_back(pl.mat_total);
        pl.mat_total += po.rev_mat_gate.size();
        // interpreted kernels hold the lowered ops in their arguments
        const size_t cap = jit ? (size_t)-1 : (size_t)kMaxPhysOps;
        for (int d = 0; d < 2; ++d) {
            po.S_f[d] = split_bits_for(jit, d == 1, p.K, false);
            po.S_r[d] = split_bits_for(jit, d == 1, p.K, true);
            if ((po.S_f[d] && !lower_split(po.fwd, p.K, po.S_f[d], cap, po.fwd_l[d])) ||
                (po.S_r[d] && !lower_split(po.rev, p.K, po.S_r[d], cap, po.rev_l[d]))) {
                set_error("vqe_circuit_create: too many ops in a pass after lane transposes (internal limit)");
                return VQE_ERR_STATE;
            }
        }
    }
    return VQE_OK;
}


// Window bits an op needs in registers (the others it can apply per lane).
uint32_t reg_needs(const KOp& op) {
    switch (op.type) {
        case OP_U2:
        case OP_R2:
        case OP_XFLIP:
        case OP_GX:
        case OP_GY:
            return 1u << op.a;
        case OP_CNOT:
        case OP_PAIR2:
        case OP_GPAIR2:
            return (1u << op.a) | (1u << op.b);
        case OP_PAIR4:
        case OP_GPAIR4:
            return (1u << op.a) | (1u << op.b) | (1u << op.c) | (1u << op.d);
        default:  // OP_DIAG, OP_CZ, OP_GZ act per lane on a lane-resident bit
            return 0;
    }
}

// Lowers a logical op list (window local bits 0..K-1) to the lane-split layout
// with S of the K bits in lane slots.  The S bits needed in registers least
// often start in the lanes; before an op that needs a lane-resident bit in
// registers, a TPOSE swaps it with the register bit whose next use is
// furthest away.  Returns false if the op capacity would be exceeded.
bool lower_split(const std::vector<KOp>& ops, int K, int S, size_t cap, SplitOps& out) {
    const int KL = K - S;
    int cost[kMaxWindow] = {0};
    for (const auto& op : ops)
        for (int w = 0; w < K; ++w)
            if (reg_needs(op) >> w & 1) cost[w]++;
    int order[kMaxWindow];
    for (int w = 0; w < K; ++w) order[w] = w;
    std::sort(order, order + K, [&](int x, int y) { return cost[x] != cost[y] ? cost[x] < cost[y] : x > y; });
    int bit_at[kMaxWindow], slot_of[kMaxWindow];
    std::vector<int> regs;
    for (int j = 0; j < S; ++j) bit_at[KL + j] = order[j];
    for (int j = S; j < K; ++j) regs.push_back(order[j]);
    std::sort(regs.begin(), regs.end());
    for (int r = 0; r < KL; ++r) bit_at[r] = regs[r];
    for (int sl = 0; sl < K; ++sl) slot_of[bit_at[sl]] = sl;
    for (int sl = 0; sl < K; ++sl) out.map_in[sl] = (uint8_t)bit_at[sl];
    out.ops.clear();
    for (size_t i = 0; i < ops.size(); ++i) {
        const KOp& op = ops[i];
        const uint32_t need = reg_needs(op);
        for (int w = 0; w < K; ++w) {
            if (!(need >> w & 1) || slot_of[w] < KL) continue;
            // evict the register bit (not needed by this op) used furthest in the future
            int best_r = -1;
            size_t best_next = 0;
            for (int r = 0; r < KL; ++r) {
                const int wb = bit_at[r];
                if (need >> wb & 1) continue;
                size_t nxt = ops.size();
                for (size_t k = i + 1; k < ops.size(); ++k)
                    if (reg_needs(ops[k]) >> wb & 1) {
                        nxt = k;
                        break;
                    }
                if (best_r < 0 || nxt > best_next) {
                    best_r = r;
                    best_next = nxt;
                }
            }
            const int lane_slot = slot_of[w];
            KOp t{};
            t.type = OP_TPOSE;
            t.a = (uint8_t)best_r;
            t.b = (uint8_t)(lane_slot - KL);
            out.ops.push_back(t);
            const int wr = bit_at[best_r];
            bit_at[best_r] = w;
            bit_at[lane_slot] = wr;
            slot_of[w] = best_r;
            slot_of[wr] = lane_slot;
        }
        KOp ph = op;
        ph.a = (uint8_t)slot_of[op.a];
        if (op.type == OP_CNOT || op.type == OP_CZ || op.type == OP_PAIR2 || op.type == OP_GPAIR2 ||
            op.type == OP_PAIR4 || op.type == OP_GPAIR4)
            ph.b = (uint8_t)slot_of[op.b];
        if (op.type == OP_PAIR4 || op.type == OP_GPAIR4) {
            ph.c = (uint8_t)slot_of[op.c];
            ph.d = (uint8_t)slot_of[op.d];
        }
        out.ops.push_back(ph);
    }
    for (int sl = 0; sl < K; ++sl) out.map_out[sl] = (uint8_t)bit_at[sl];
    return out.ops.size() <= cap;
}

// Uploads the gradient slot maps of a plan to the current device (once).
int upload_plan(const Plan& cpl) {
    Plan& pl = const_cast<Plan&>(cpl);
    std::lock_guard<std::mutex> g(g_upload_mu);
    if (pl.d_slotmap || pl.slotmap.empty()) return VQE_OK;
    if (hipMalloc((void**)&pl.d_slotmap, pl.slotmap.size() * sizeof(int32_t)) != hipSuccess) {
        set_error("hipMalloc of the gradient slot map failed");
        return VQE_ERR_OOM;
    }
    VQE_HIP(hipMemcpy(pl.d_slotmap, pl.slotmap.data(), pl.slotmap.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    return VQE_OK;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int max_small(int dtype) { return dtype == VQE_C64 ? kBatchMaxQubitsC64 : kBatchMaxQubitsC128; }

// Plans the batch programs of c for dtype index d (once); ckpt: programs of a
// small state that may stop at checkpoints (the forward one is the same).
int ensure_batch(const vqe_circuit* cc, int d, bool ckpt = false) {
    vqe_circuit* c = const_cast<vqe_circuit*>(cc);
    BatchPlan& bp = c->batch[d][ckpt ? 1 : 0];
    std::lock_guard<std::mutex> g(g_upload_mu);
    if (bp.ready) return VQE_OK;
    BatchPlan np;
    std::string msg;
    int local[64];
    auto add = [&](int bits, const std::vector<int>& gates) {
        ProgramPlan plan;
        if (!plan_program(bits, c->gates, gates, local, plan, msg)) return false;
        for (int dir = 0; dir < 2; ++dir) {
            Program p;
            if (!build_program(d == 1, bits, c->gates, plan, dir, dir == 0 || ckpt, p, msg)) return false;
            np.slot_off.push_back(np.slot_param.size());
            np.slot_param.insert(np.slot_param.end(), p.slot_param.begin(), p.slot_param.end());
            np.prog.push_back(std::move(p));
        }
        return true;
    };
    bool ok = true;
    if (c->n <= max_small(d ? VQE_C128 : VQE_C64)) {
        std::vector<int> all(c->gates.size());
        std::iota(all.begin(), all.end(), 0);
        std::iota(local, local + 64, 0);
        ok = add(batch_bits(c->n), all);
    } else {
        ok = plan_tiles(c->n, c->gates, TileLimits{kMidWin, kMidLow, 1 << 20, kMidMaxSlots, kMidPlanWidth}, np.passes, msg);
        if (ok && np.passes.empty()) {  // no gates: one pass that only prepares |0...0>
            np.passes.emplace_back();
            for (int q = 0; q < kMidWin; ++q) np.passes[0].pos[np.passes[0].K++] = q;
        }
        for (size_t p = 0; ok && p < np.passes.size(); ++p) {
            for (int j = 0; j < kMidWin; ++j) local[np.passes[p].pos[j]] = j;
            ok = add(kMidWin, np.passes[p].gates);
        }
    }
    if (!ok) {
        set_error(msg);
        return VQE_ERR_STATE;
    }
    size_t at = 0;
    for (const Program& p : np.prog) {
        np.stage_off.push_back(at);
        at += p.stages.size() * sizeof(ProgStage);
    }
    for (const Program& p : np.prog) {
        at = align_up(at, 64);
        np.stream_off.push_back(at);
        at += p.stream.size() * 4;
    }
    np.image.assign(align_up(std::max<size_t>(at, 64), 64), 0);
    for (size_t k = 0; k < np.prog.size(); ++k) {
        Program& p = np.prog[k];
        if (!p.stages.empty()) std::memcpy(&np.image[np.stage_off[k]], p.stages.data(), p.stages.size() * sizeof(ProgStage));
        if (!p.stream.empty()) std::memcpy(&np.image[np.stream_off[k]], p.stream.data(), p.stream.size() * 4);
        std::vector<uint32_t>().swap(p.stream);
    }
    np.ready = true;
    bp = std::move(np);
    return VQE_OK;
}

// The image of a batch plan with the numbers of one evaluation, to dst.
template <typename T>
void fill_batch_image(const vqe_circuit* c, const BatchPlan& bp, const double* params, double norm,
                      std::vector<HalfAngle>& h, char* dst) {
    half_angles(c, params, h);
    const double limit = turn_limit(sizeof(T) == 8, norm);
    std::memcpy(dst, bp.image.data(), bp.image.size());
    for (size_t k = 0; k < bp.prog.size(); ++k)
        fill_tile_table<T>(bp.prog[k].table, c->gates, h.data(), limit, (int)(k & 1), (T*)(dst + bp.stream_off[k]));
}

// Descriptor of one small evaluation; image, out and part are device addresses.
template <typename T>
BatchDesc<T> small_desc(const vqe_circuit* c, const BatchPlan& bp, const vqe_hamiltonian* h, const char* image,
                        double* out, double* part) {
    BatchDesc<T> d{};
    d.n = c->n;
    d.bits = batch_bits(c->n);
    d.n_fwd = (uint32_t)bp.prog[0].stages.size();
    d.n_rev = (uint32_t)bp.prog[1].stages.size();
    const int dt = sizeof(T) == 8 ? 1 : 0;
    d.n_blocks = (uint32_t)h->sm_blocks[dt].size();
    d.n_slots = (uint32_t)bp.slot_param.size();
    d.real = h->real_coeffs ? 1 : 0;
    d.fwd = (const ProgStage*)(image + bp.stage_off[0]);
    d.rev = (const ProgStage*)(image + bp.stage_off[1]);
    d.fwd_stream = image + bp.stream_off[0];
    d.rev_stream = image + bp.stream_off[1];
    d.ham = h->d_sm_blocks[dt];
    d.ham_stream = h->d_sm_stream[dt];
    d.out = out;
    d.part = part;
    return d;
}

void small_results(const vqe_circuit* c, const BatchPlan& bp, const double* r, double* energy, double* grad) {
    *energy = r[0];
    std::fill(grad, grad + c->n_params, 0.0);
    for (size_t s = 0; s < bp.slot_param.size(); ++s) grad[bp.slot_param[s]] += r[2 + s];
}

// Raises the dynamic LDS limit of the small-state kernels once per process.
int small_lds_limit() {
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    std::call_once(once, [] { rc = batch_set_lds_limit(); });
    if (rc != hipSuccess) {
        set_error(std::string("cannot raise the LDS limit: ") + hipGetErrorString(rc));
        return VQE_ERR_DEVICE;
    }
    return VQE_OK;
}

// Small items: descriptors and tables in one copy, one launch, results
// written to the pinned buffer by the kernel itself.
template <typename T>
int batch_impl(vqe_batch* b, size_t n_items, const vqe_batch_item* items) {
    const int dt = sizeof(T) == 8 ? 1 : 0;
    size_t n_img = 0, n_out = 0, n_part = 0;
    int max_bits = kBatchMinBits;
    for (size_t i = 0; i < n_items; ++i) {
        const vqe_circuit* c = items[i].circuit;
        if (int rc = ensure_batch(c, dt)) return rc;
        if (int rc = upload_hamiltonian(items[i].hamiltonian)) return rc;
        n_img += c->batch[dt][0].image.size();
        n_out += 2 + c->batch[dt][0].slot_param.size();
        n_part += 8 * c->batch[dt][0].slot_param.size();
        max_bits = std::max(max_bits, batch_bits(c->n));
    }
    const size_t o_img = align_up(n_items * sizeof(BatchDesc<T>), 256);
    const size_t o_out = align_up(o_img + n_img, 256);  // pinned: results; device: sums per wave
    const size_t host = o_out + n_out * sizeof(double), dev = o_out + std::max<size_t>(n_part, 1) * sizeof(double);
    const size_t total = std::max(host, dev);
    if (total > b->d_cap) {
        VQE_HIP(hipStreamSynchronize(b->stream));
        if (b->d_buf) VQE_HIP(hipFree(b->d_buf));
        if (b->h_buf) VQE_HIP(hipHostFree(b->h_buf));
        b->d_buf = b->h_buf = nullptr;
        b->d_cap = b->h_cap = 0;
        const size_t cap = std::max(total * 2, (size_t)1 << 20);
        if (hipMalloc(&b->d_buf, cap) != hipSuccess || hipHostMalloc(&b->h_buf, cap, hipHostMallocDefault) != hipSuccess) {
            set_error("vqe_batch_energy_grad: staging allocation failed");
            return VQE_ERR_OOM;
        }
        b->d_cap = b->h_cap = cap;
    }
    char* h = (char*)b->h_buf;
    char* d = (char*)b->d_buf;
    double* out = (double*)(h + o_out);
    size_t img = o_img, o = 0, part = 0;
    std::vector<HalfAngle> ha;
    for (size_t i = 0; i < n_items; ++i) {
        const vqe_circuit* c = items[i].circuit;
        const BatchPlan& bp = c->batch[dt][0];
        ((BatchDesc<T>*)h)[i] = small_desc<T>(c, bp, items[i].hamiltonian, d + img, out + o, (double*)(d + o_out) + part);
        fill_batch_image<T>(c, bp, items[i].params, items[i].hamiltonian->norm1, ha, h + img);
        img += bp.image.size();
        o += 2 + bp.slot_param.size();
        part += 8 * bp.slot_param.size();
    }
    VQE_HIP(hipMemcpyAsync(d, h, o_img + n_img, hipMemcpyHostToDevice, b->stream));
    VQE_HIP(launch_batch<T>((const BatchDesc<T>*)d, (uint32_t)n_items, max_bits, b->stream));
    VQE_HIP(hipStreamSynchronize(b->stream));
    o = 0;
    for (size_t i = 0; i < n_items; ++i) {
        const BatchPlan& bp = items[i].circuit->batch[dt][0];
        small_results(items[i].circuit, bp, out + o, items[i].energy, items[i].grad);
        o += 2 + bp.slot_param.size();
    }
    return VQE_OK;
}

// vqe_energy_grad of one state that fits LDS: the same kernel, which also
// leaves the state where the reverse sweep ends.
template <typename T>
int small_grad(vqe_state* psi, vqe_state* lam, const vqe_circuit* c, const double* params, const vqe_hamiltonian* h,
               const vqe_grad_opts* o, double* energy, double* grad) {
    const int dt = sizeof(T) == 8 ? 1 : 0;
    if (int rc = small_lds_limit()) return rc;
    const bool ckpt = o && o->n_ckpt > 0;
    if (int rc = ensure_batch(c, dt, ckpt)) return rc;
    const BatchPlan& bp = c->batch[dt][ckpt ? 1 : 0];
    const size_t slots = bp.slot_param.size();
    if (int rc = ensure_res(psi, 2 + 8 * slots)) return rc;  // device: sums per wave; pinned: results
    // checkpoints at evenly spaced groups of stages
    std::vector<BatchCkpt> ck;
    const std::vector<uint32_t>&mf = bp.prog[0].mark, &mr = bp.prog[1].mark;
    for (int k = 0, n = o ? o->n_ckpt : 0; k < n; ++k) {
        const size_t at = (size_t)std::llround((double)(k + 1) * (double)mf.size() / (double)(n + 1));
        if (at < 1 || at >= mf.size() || (!ck.empty() && ck.back().fwd_end == mf[at - 1])) continue;
        if (mf[at - 1] == ~0u || mr[mf.size() - at - 1] == ~0u) continue;  // inside a stage of either program
        ck.push_back(BatchCkpt{o->ckpt[k]->data, mf[at - 1], mr[mf.size() - at - 1]});
    }
    const size_t o_ck = align_up(sizeof(BatchDesc<T>), 256);
    const size_t o_img = align_up(o_ck + ck.size() * sizeof(BatchCkpt), 256), bytes = o_img + bp.image.size();
    if (int rc = stage_mats(psi, bytes)) return rc;
    BatchDesc<T> d = small_desc<T>(c, bp, h, (const char*)psi->d_mats + o_img, psi->h_res, psi->d_res);
    d.psi_out = psi->data;
    d.lam_out = lam->data;
    d.n_ckpt = (uint32_t)ck.size();
    d.ckpt = (const BatchCkpt*)((char*)psi->d_mats + o_ck);
    std::memcpy(psi->h_mats, &d, sizeof(d));
    if (!ck.empty()) std::memcpy((char*)psi->h_mats + o_ck, ck.data(), ck.size() * sizeof(BatchCkpt));
    std::vector<HalfAngle> ha;
    fill_batch_image<T>(c, bp, params, h->norm1, ha, (char*)psi->h_mats + o_img);
    VQE_HIP(hipMemcpyAsync(psi->d_mats, psi->h_mats, bytes, hipMemcpyHostToDevice, psi->stream));
    {
        ProfScope ps(VQE_KERNEL_WINDOW_REV, 2.0 * (double)psi->bytes, psi->stream);
        VQE_HIP(launch_batch<T>((const BatchDesc<T>*)psi->d_mats, 1, d.bits, psi->stream));
    }
    VQE_HIP(hipEventRecord(psi->mats_ev, psi->stream));
    VQE_HIP(hipStreamSynchronize(psi->stream));
    small_results(c, bp, psi->h_res, energy, grad);
    return VQE_OK;
}

// Bytes of one state of n qubits in the mid-size buffer (256-byte aligned).
size_t st_bytes_half(int n, size_t amp) { return align_up(((size_t)1 << n) * amp, 256); }

// Grows a batch's mid-size buffers to at least dev / host bytes.
int mid_reserve(vqe_batch* b, size_t dev, size_t host) {
    if (dev <= b->md_cap && host <= b->mh_cap) return VQE_OK;
    VQE_HIP(hipStreamSynchronize(b->stream));
    if (dev > b->md_cap) {
        if (b->md_buf) VQE_HIP(hipFree(b->md_buf));
        b->md_buf = nullptr;
        b->md_cap = 0;
        const size_t cap = dev + dev / 4;
        if (hipMalloc(&b->md_buf, cap) != hipSuccess) {
            b->md_buf = nullptr;
            set_error("vqe_batch_energy_grad: device allocation of " + std::to_string(cap) +
                      " bytes for mid-size items failed");
            return VQE_ERR_OOM;
        }
        b->md_cap = cap;
    }
    if (host > b->mh_cap) {
        if (b->mh_buf) VQE_HIP(hipHostFree(b->mh_buf));
        b->mh_buf = nullptr;
        b->mh_cap = 0;
        const size_t cap = std::max(host + host / 4, (size_t)1 << 20);
        if (hipHostMalloc(&b->mh_buf, cap, hipHostMallocDefault) != hipSuccess) {
            b->mh_buf = nullptr;
            set_error("vqe_batch_energy_grad: pinned staging allocation failed");
            return VQE_ERR_OOM;
        }
        b->mh_cap = cap;
    }
    return VQE_OK;
}

// Mid-size items (LDS limit < n <= kMidMaxQubits): forward passes, one launch
// per pass index over every item that has that pass; lam = H psi; reverse
// passes likewise; one reduction launch that writes the results to the pinned
// buffer.  Per item: psi and lam in the batch's device buffer, n_blk =
// min(2^(n - kMidWin), kMidMaxBlocks) blocks per launch.  own: one item, on the
// states of an evaluation instead of the batch's buffer, with its options.
struct MidOwn {
    vqe_state *psi, *lam;
    const vqe_grad_opts* opts;
};
template <typename T>
int mid_impl(vqe_batch* b, const vqe_batch_item* items, const std::vector<size_t>& idx, const MidOwn* own = nullptr) {
    const int dt = sizeof(T) == 8 ? 1 : 0;
    const size_t m = idx.size();
    const size_t amp = 2 * sizeof(T);
    // lam = H psi: window passes (hwin_batch_kernel, one launch per pass index
    // and coefficient form) where the Hamiltonian has a window cover, else the
    // tile kernel (mid_hpsi_kernel; for a state of its own that of large states,
    // which reads a term once for several amplitudes: 101 X groups of 8 terms, no
    // cover, 4 layers, per call: 14 qubits complex64 362 us against 573, 19 qubits
    // complex128 583 against 1041).  A state of its own takes tiles also where the
    // plan of large states counts fewer bytes for them and groups have six terms or
    // less.  With more, windows, which sum a group's terms once per class: the
    // bytes come from the cache.  13 qubits complex128, groups x terms each, tiles
    // against windows: 4000 x 1 2450 us, 3860; 500 x 4 760, 872; 500 x 6 952, 970;
    // 500 x 10 1340, 1120; 60 x 30 516, 341; 1 x 2000 480, 250
    std::vector<uint32_t> nblk(m), nblk_e(m);
    std::vector<uint64_t> part_base(m), part_s(m), red_base(m), st_off(m), img_off(m);
    std::vector<char> use_hw(m);
    size_t n_img = 0, n_pass = 0, n_part = 0, n_red = 0, st_bytes = 0, n_hw = 0, n_tile = 0;
    size_t pmax = 0, hmax = 0;
    for (size_t k = 0; k < m; ++k) {
        const vqe_circuit* c = items[idx[k]].circuit;
        const vqe_hamiltonian* hh = items[idx[k]].hamiltonian;
        if (int rc = ensure_batch(c, dt)) return rc;
        if (int rc = upload_hamiltonian(hh)) return rc;
        const BatchPlan& bp = c->batch[dt][0];
        nblk[k] = (uint32_t)std::min<uint64_t>(1ull << (c->n - kMidWin), kMidMaxBlocks);
        use_hw[k] = !hh->hw_wins.empty() && !(own && !hh->hw_lam && hh->w.size() <= 6 * hh->groups.size());
        nblk_e[k] = (uint32_t)std::min<uint64_t>(1ull << (c->n - (use_hw[k] ? kHwBits : kMidTileBits)), kMidMaxBlocks);
        if (own && !use_hw[k]) nblk_e[k] = 1;  // apply_h() leaves the sums
        if (use_hw[k]) {
            n_hw += hh->hw_wins.size();
            hmax = std::max(hmax, hh->hw_wins.size());
        } else {
            ++n_tile;
        }
        part_base[k] = n_part;
        part_s[k] = n_part + 2 * (size_t)nblk_e[k];
        n_part += 2 * (size_t)nblk_e[k] + bp.slot_param.size() * (size_t)nblk[k];
        red_base[k] = n_red;
        n_red += 2 + bp.slot_param.size();
        st_off[k] = st_bytes;
        if (!own) st_bytes += 2 * st_bytes_half(c->n, amp);
        img_off[k] = n_img;
        n_img += bp.image.size();
        n_pass += bp.passes.size();
        pmax = std::max(pmax, bp.passes.size());
    }
    // host-written tables, then results (pinned) or partial sums | states (device)
    const size_t o_fwd = 0;
    const size_t o_rev = align_up(o_fwd + n_pass * sizeof(MidPass), 256);
    const size_t o_ham = align_up(o_rev + n_pass * sizeof(MidPass), 256);
    const size_t o_hw = align_up(o_ham + std::max<size_t>(n_tile, 1) * sizeof(MidHam), 256);
    const size_t o_red = align_up(o_hw + std::max<size_t>(n_hw, 1) * sizeof(HwItem), 256);
    const size_t o_img = align_up(o_red + n_red * sizeof(MidRed), 256);
    const size_t o_out = align_up(o_img + n_img, 256);
    const size_t o_st = align_up(o_out + n_part * sizeof(double), 256);
    if (int rc = mid_reserve(b, o_st + st_bytes, o_out + n_red * sizeof(double))) return rc;
    char* h = (char*)b->mh_buf;
    char* d = (char*)b->md_buf;
    auto* hf = (MidPass*)(h + o_fwd);
    auto* hr = (MidPass*)(h + o_rev);
    auto* hh = (MidHam*)(h + o_ham);
    auto* hred = (MidRed*)(h + o_red);
    auto* hw = (HwItem*)(h + o_hw);
    double* part = (double*)(d + o_out);
    double* out = (double*)(h + o_out);
    auto psi_of = [&](size_t k) { return own ? (char*)own->psi->data : d + o_st + st_off[k]; };
    auto lam_of = [&](size_t k) {
        return own ? (char*)own->lam->data : d + o_st + st_off[k] + st_bytes_half(items[idx[k]].circuit->n, amp);
    };
    // numbers, tile-form H psi and reduction descriptors per item
    size_t n_th = 0;
    uint32_t hblk = 0;
    std::vector<HalfAngle> ha;
    for (size_t k = 0; k < m; ++k) {
        const vqe_batch_item& it = items[idx[k]];
        const vqe_circuit* c = it.circuit;
        const BatchPlan& bp = c->batch[dt][0];
        fill_batch_image<T>(c, bp, it.params, it.hamiltonian->norm1, ha, h + o_img + img_off[k]);
        if (!use_hw[k] && !own) {
            MidHam mh{};
            mh.psi = psi_of(k);
            mh.lam = lam_of(k);
            mh.groups = it.hamiltonian->d_groups;
            mh.terms = terms_of<T>(it.hamiltonian);
            mh.n_tiles = 1ull << (c->n - kMidTileBits);
            mh.part_off = part_base[k];
            mh.n_groups = (uint32_t)it.hamiltonian->groups.size();
            mh.blk_begin = hblk;
            mh.n_blk = nblk_e[k];
            hh[n_th++] = mh;
            hblk += nblk_e[k];
        }
        hred[red_base[k]] = MidRed{part_base[k], nblk_e[k], 0};
        hred[red_base[k] + 1] = MidRed{part_base[k] + nblk_e[k], nblk_e[k], 0};
        for (size_t sl = 0; sl < bp.slot_param.size(); ++sl)
            hred[red_base[k] + 2 + sl] = MidRed{part_s[k] + sl * (uint64_t)nblk[k], nblk[k], 0};
    }
    // window-form H psi descriptors, grouped by launch: pass index, then real
    // coefficients or not
    struct HwLaunch {
        size_t off, cnt;
        uint32_t grid;
        bool real;
    };
    std::vector<HwLaunch> hw_launch;
    {
        size_t e = 0;
        for (size_t p = 0; p < hmax; ++p)
            for (int real = 1; real >= 0; --real) {
                HwLaunch L{e, 0, 0, real == 1};
                for (size_t k = 0; k < m; ++k) {
                    const vqe_hamiltonian* H = items[idx[k]].hamiltonian;
                    if (!use_hw[k] || p >= H->hw_wins.size() || H->real_coeffs != (real == 1)) continue;
                    const vqe_circuit* c = items[idx[k]].circuit;
                    HwItem x{};
                    x.w = H->hw_wins[p];
                    x.psi = psi_of(k);
                    x.lam = lam_of(k);
                    x.groups = H->d_hw_groups;
                    x.classes = H->d_hw_classes;
                    x.terms = hw_terms_of<T>(H);
                    x.n_cosets = 1ull << (c->n - kHwBits);
                    x.part_off = part_base[k];
                    x.blk_begin = L.grid;
                    x.n_blk = nblk_e[k];
                    x.first = p == 0 ? 1u : 0u;
                    x.last = p + 1 == H->hw_wins.size() ? 1u : 0u;
                    hw[e++] = x;
                    L.grid += nblk_e[k];
                    ++L.cnt;
                }
                if (L.cnt) hw_launch.push_back(L);
            }
    }
    // pass descriptors, grouped by launch
    std::vector<size_t> l_off(pmax), l_cnt(pmax);
    std::vector<uint32_t> l_grid(pmax);
    size_t e = 0;
    for (size_t p = 0; p < pmax; ++p) {
        l_off[p] = e;
        uint32_t blk = 0;
        for (size_t k = 0; k < m; ++k) {
            const vqe_circuit* c = items[idx[k]].circuit;
            const BatchPlan& bp = c->batch[dt][0];
            const size_t P = bp.passes.size();
            if (p >= P) continue;
            for (int dir = 0; dir < 2; ++dir) {
                const size_t q = dir ? P - 1 - p : p, pr = 2 * q + (size_t)dir;
                MidPass x{};
                x.psi = psi_of(k);
                x.lam = lam_of(k);
                x.stages = (const ProgStage*)(d + o_img + img_off[k] + bp.stage_off[pr]);
                x.stream = d + o_img + img_off[k] + bp.stream_off[pr];
                x.n_cosets = 1ull << (c->n - kMidWin);
                x.part_off = part_s[k] + (uint64_t)bp.slot_off[pr] * nblk[k];
                for (int j = 0; j < kMidWin; ++j) x.pos[j] = (uint32_t)bp.passes[q].pos[j];
                x.n_stages = (uint32_t)bp.prog[pr].stages.size();
                x.n_slots = (uint32_t)bp.prog[pr].slot_param.size();
                x.blk_begin = blk;
                x.n_blk = nblk[k];
                x.first = (dir == 0 && p == 0) ? 1u : 0u;
                (dir ? hr : hf)[e] = x;
            }
            blk += nblk[k];
            ++e;
        }
        l_cnt[p] = e - l_off[p];
        l_grid[p] = blk;
    }
    VQE_HIP(hipMemcpyAsync(d, h, o_img + n_img, hipMemcpyHostToDevice, b->stream));
    const double S = own ? (double)own->psi->bytes : 0.0;
    auto prof = [&](int kind, double bytes) {  // only evaluations of a state are traced
        return own ? std::make_unique<ProfScope>(kind, bytes, b->stream) : nullptr;
    };
    // own: after that many passes psi is copied to a checkpoint, and from it before they are un-applied
    std::vector<size_t> bounds;
    std::vector<void*> ck;
    for (int k = 0, n = own && own->opts ? own->opts->n_ckpt : 0; k < n; ++k) {
        const size_t at = (size_t)std::llround((double)(k + 1) * (double)pmax / (double)(n + 1));
        if (at < 1 || at >= pmax || (!bounds.empty() && bounds.back() == at)) continue;
        bounds.push_back(at);
        ck.push_back(own->opts->ckpt[k]->data);
    }
    const size_t chunk = own && own->opts && own->opts->chunk_passes > 0 ? (size_t)own->opts->chunk_passes : 0;
    auto launch = [&](size_t p, bool rev) {
        const size_t done = rev ? pmax - p : p + 1;  // passes applied: before a reverse pass, after a forward one
        const auto at = std::find(bounds.begin(), bounds.end(), done);
        void* c = at == bounds.end() ? nullptr : ck[(size_t)(at - bounds.begin())];
        if (c && rev) VQE_HIP(hipMemcpyAsync(own->psi->data, c, own->psi->bytes, hipMemcpyDeviceToDevice, b->stream));
        {
            // the first pass stages |0...0> and only writes
            auto ps = prof(rev ? VQE_KERNEL_WINDOW_REV : VQE_KERNEL_WINDOW_FWD, (rev ? 4.0 : p ? 2.0 : 1.0) * S);
            VQE_HIP(launch_mid_pass<T>((const MidPass*)(d + (rev ? o_rev : o_fwd)) + l_off[p], (uint32_t)l_cnt[p],
                                       l_grid[p], rev, part, b->stream));
        }
        if (c && !rev) VQE_HIP(hipMemcpyAsync(c, own->psi->data, own->psi->bytes, hipMemcpyDeviceToDevice, b->stream));
        const bool end = p + 1 == pmax;
        if (chunk && ((p + 1) % chunk == 0 || end) && !(rev && end)) VQE_HIP(hipStreamSynchronize(b->stream));
        return (int)VQE_OK;
    };
    for (size_t p = 0; p < pmax; ++p)
        if (int rc = launch(p, false)) return rc;
    if (n_th) VQE_HIP(launch_mid_hpsi<T>((const MidHam*)(d + o_ham), (uint32_t)n_th, hblk, part, b->stream));
    if (own && !use_hw[0])  // hw_lam is false: tiles
        if (int rc = apply_h<T>(own->psi, own->lam->data, items[idx[0]].hamiltonian, part + part_base[0])) return rc;
    for (size_t l = 0; l < hw_launch.size(); ++l) {
        const HwLaunch& L = hw_launch[l];
        auto ps = prof(VQE_KERNEL_HPSI, (l ? 3.0 : 2.0) * S);
        VQE_HIP(launch_hwin_batch<T>((const HwItem*)(d + o_hw) + L.off, (uint32_t)L.cnt, L.grid, L.real, part,
                                     b->stream));
        if (chunk && ((l + 1) % chunk == 0 || l + 1 == hw_launch.size())) VQE_HIP(hipStreamSynchronize(b->stream));
    }
    for (size_t p = 0; p < pmax; ++p)
        if (int rc = launch(p, true)) return rc;
    VQE_HIP(launch_mid_reduce((const MidRed*)(d + o_red), (uint32_t)n_red, part, out, b->stream));
    VQE_HIP(hipStreamSynchronize(b->stream));
    for (size_t k = 0; k < m; ++k) {
        const vqe_batch_item& it = items[idx[k]];
        const vqe_circuit* c = it.circuit;
        const std::vector<int32_t>& sp = c->batch[dt][0].slot_param;
        const double* o = out + red_base[k];
        const double nrm = o[1];
        *it.energy = o[0] / nrm;
        for (size_t q = 0; q < c->n_params; ++q) it.grad[q] = 0.0;
        for (size_t sl = 0; sl < sp.size(); ++sl) it.grad[sp[sl]] += o[2 + sl] / nrm;
    }
    return VQE_OK;
}
}  // namespace

// ================================================================ exported
extern "C" {

const char* vqe_last_error(void) { return g_last_error.c_str(); }

const char* vqe_version(void) { return "1.0.0"; }

int vqe_device_count(void) {
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess) return 0;
    return n;
}

int vqe_state_alloc(int n_qubits, int dtype, void* device_buf, size_t buf_bytes, void* hip_stream, vqe_state** out) {
    VQE_GUARD_BEGIN
    if (!out) {
        set_error("vqe_state_alloc: null out");
        return VQE_ERR_ARG;
    }
    if (n_qubits < 1 || n_qubits > 40) {
        set_error("vqe_state_alloc: n_qubits must be in [1, 40]");
        return VQE_ERR_ARG;
    }
    if (dtype != VQE_C64 && dtype != VQE_C128) {
        set_error("vqe_state_alloc: dtype must be VQE_C64 or VQE_C128");
        return VQE_ERR_ARG;
    }
    const size_t need = (size_t(1) << n_qubits) * amp_bytes(dtype);
    if (device_buf && buf_bytes < need) {
        set_error("vqe_state_alloc: device buffer of " + std::to_string(buf_bytes) + " bytes is smaller than the " +
                  std::to_string(need) + " bytes the state needs");
        return VQE_ERR_ARG;
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) {
        set_error("vqe_state_alloc: no HIP device");
        return VQE_ERR_DEVICE;
    }
    auto* s = new vqe_state();
    s->n = n_qubits;
    s->dtype = dtype;
    s->bytes = need;
    s->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&s->device) != hipSuccess) {
        delete s;
        set_error("vqe_state_alloc: hipGetDevice failed");
        return VQE_ERR_DEVICE;
    }
    if (device_buf) {
        s->data = device_buf;
    } else {
        if (hipMalloc(&s->data, need) != hipSuccess) {
            delete s;
            set_error("vqe_state_alloc: hipMalloc of " + std::to_string(need) + " bytes failed");
            return VQE_ERR_OOM;
        }
        s->owned = true;
    }
    int rc = ensure_res(s, 1024);
    if (rc) {
        if (s->owned) (void)hipFree(s->data);
        delete s;
        return rc;
    }
    if (launch_set_basis(dtype, s->data, 1ull << n_qubits, 0, s->stream) != hipSuccess) {
        set_error("vqe_state_alloc: initialisation kernel failed");
        (void)hipFree(s->d_res);
        (void)hipHostFree(s->h_res);
        if (s->owned) (void)hipFree(s->data);
        delete s;
        return VQE_ERR_DEVICE;
    }
    *out = s;
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_state_free(vqe_state* s) {
    if (!s) return VQE_OK;
    (void)hipSetDevice(s->device);
    (void)hipStreamSynchronize(s->stream);
    if (s->owned && s->data) (void)hipFree(s->data);
    if (s->d_part) (void)hipFree(s->d_part);
    if (s->d_res) (void)hipFree(s->d_res);
    if (s->h_res) (void)hipHostFree(s->h_res);
    if (s->d_mats) (void)hipFree(s->d_mats);
    if (s->h_mats) (void)hipHostFree(s->h_mats);
    if (s->mats_ev) (void)hipEventDestroy(s->mats_ev);
    (void)vqe_batch_free(s->mid);
    delete s;
    return VQE_OK;
}

int vqe_state_set_basis(vqe_state* s, uint64_t b) {
    if (int rc = check_state(s, "vqe_state_set_basis")) return rc;
    if (b >= (1ull << s->n)) {
        set_error("vqe_state_set_basis: basis index out of range");
        return VQE_ERR_ARG;
    }
    VQE_HIP(hipSetDevice(s->device));
    VQE_HIP(launch_set_basis(s->dtype, s->data, 1ull << s->n, b, s->stream));
    return VQE_OK;
}

int vqe_state_info(const vqe_state* s, void** device_ptr, int* n_qubits, int* dtype) {
    if (int rc = check_state(s, "vqe_state_info")) return rc;
    if (device_ptr) *device_ptr = s->data;
    if (n_qubits) *n_qubits = s->n;
    if (dtype) *dtype = s->dtype;
    return VQE_OK;
}

int vqe_state_read(const vqe_state* s, uint64_t offset, uint64_t count, void* host_dst) {
    if (int rc = check_state(s, "vqe_state_read")) return rc;
    if (!host_dst && count) {
        set_error("vqe_state_read: null destination");
        return VQE_ERR_ARG;
    }
    if (offset > (1ull << s->n) || count > (1ull << s->n) - offset) {
        set_error("vqe_state_read: range out of bounds");
        return VQE_ERR_ARG;
    }
    const size_t ab = amp_bytes(s->dtype);
    VQE_HIP(hipSetDevice(s->device));
    VQE_HIP(hipMemcpyAsync(host_dst, (const char*)s->data + offset * ab, count * ab, hipMemcpyDeviceToHost, s->stream));
    VQE_HIP(hipStreamSynchronize(s->stream));
    return VQE_OK;
}

int vqe_state_write(vqe_state* s, uint64_t offset, uint64_t count, const void* host_src) {
    if (int rc = check_state(s, "vqe_state_write")) return rc;
    if (!host_src && count) {
        set_error("vqe_state_write: null source");
        return VQE_ERR_ARG;
    }
    if (offset > (1ull << s->n) || count > (1ull << s->n) - offset) {
        set_error("vqe_state_write: range out of bounds");
        return VQE_ERR_ARG;
    }
    const size_t ab = amp_bytes(s->dtype);
    VQE_HIP(hipSetDevice(s->device));
    VQE_HIP(hipMemcpyAsync((char*)s->data + offset * ab, host_src, count * ab, hipMemcpyHostToDevice, s->stream));
    VQE_HIP(hipStreamSynchronize(s->stream));
    return VQE_OK;
}

int vqe_circuit_create(int n_qubits, const vqe_gate* gates, size_t n_gates, vqe_circuit** out) {
    VQE_GUARD_BEGIN
    if (!out || (n_gates && !gates)) {
        set_error("vqe_circuit_create: null argument");
        return VQE_ERR_ARG;
    }
    if (n_qubits < 1 || n_qubits > 40) {
        set_error("vqe_circuit_create: n_qubits must be in [1, 40]");
        return VQE_ERR_ARG;
    }
    std::vector<Gate> gs(n_gates);
    size_t n_params = 0;
    for (size_t i = 0; i < n_gates; ++i) {
        const vqe_gate& g = gates[i];
        if (g.kind > VQE_GATE_DEXC) {
            set_error("vqe_circuit_create: gate " + std::to_string(i) + " has an unknown kind");
            return VQE_ERR_ARG;
        }
        Gate ig{g.kind, g.q0, g.q1, g.param_index, g.angle};
        ig.q2 = g.q2;
        ig.q3 = g.q3;
        int gq[4];
        const int nqg = gate_qubits(ig, gq);
        bool ok = true;
        for (int a = 0; a < nqg; ++a) {
            ok = ok && gq[a] < n_qubits;
            for (int b = 0; b < a; ++b) ok = ok && gq[a] != gq[b];
        }
        if (!ok) {
            set_error("vqe_circuit_create: gate " + std::to_string(i) + " has an invalid or repeated qubit");
            return VQE_ERR_ARG;
        }
        if (g.param_index >= 0 && !(g.kind == VQE_GATE_RY || g.kind == VQE_GATE_RZ || g.kind == VQE_GATE_RX ||
                                    is_excitation(g.kind))) {
            set_error("vqe_circuit_create: gate " + std::to_string(i) + " cannot take a parameter");
            return VQE_ERR_ARG;
        }
        if (g.param_index < -1) {
            set_error("vqe_circuit_create: gate " + std::to_string(i) + " has param_index < -1");
            return VQE_ERR_ARG;
        }
        if (g.param_index < 0 && !std::isfinite(g.angle)) {
            set_error("vqe_circuit_create: gate " + std::to_string(i) + " has a non-finite angle");
            return VQE_ERR_ARG;
        }
        if (nqg == 1) ig.q1 = ig.q0;
        if (nqg < 4) ig.q2 = ig.q3 = 0;
        gs[i] = ig;
        if (g.param_index >= 0) n_params = std::max(n_params, (size_t)g.param_index + 1);
    }
    auto* c = new vqe_circuit();
    c->n = n_qubits;
    c->gates = std::move(gs);
    c->n_params = n_params;
    for (const Gate& g : c->gates) c->has_excitation = c->has_excitation || is_excitation(g.kind);
    for (int v = 0; v < 2; ++v) {
        if (v == 0 && c->has_excitation) continue;  // interpreted kernels have no pair ops
        int rc = build_plan(c, v ? kJitLimits : kInterpLimits, v == 1, c->plan[v]);
        if (rc) {
            free_circuit(c);
            return rc;
        }
    }
    *out = c;
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_circuit_free(vqe_circuit* c) {
    free_circuit(c);
    return VQE_OK;
}

int vqe_circuit_info(const vqe_circuit* c, size_t* n_params, size_t* n_passes) {
    if (!c) {
        set_error("vqe_circuit_info: null circuit");
        return VQE_ERR_ARG;
    }
    if (n_params) *n_params = c->n_params;
    if (n_passes) *n_passes = plan_of(c, jit_mode()).passes.size();
    return VQE_OK;
}

int vqe_circuit_pass(const vqe_circuit* c, int dtype, size_t pass, int* window, int* qubits, size_t* n_gates,
                     int32_t* gate_index, size_t capacity) {
    if (!c || (dtype != VQE_C64 && dtype != VQE_C128)) {
        set_error("vqe_circuit_pass: null circuit or bad dtype");
        return VQE_ERR_ARG;
    }
    const int form = jit_mode();
    if (int rc = check_form(c, form, "vqe_circuit_pass")) return rc;
    const Plan& pl = plan_of(c, form);
    if (pass >= pl.passes.size()) {
        set_error("vqe_circuit_pass: pass index out of range");
        return VQE_ERR_ARG;
    }
    const PlannedPass& p = pl.passes[pass];
    if (window) *window = p.K;
    if (qubits)
        for (int j = 0; j < p.K; ++j) qubits[j] = p.pos[j];
    if (n_gates) *n_gates = p.gates.size();
    if (gate_index) {
        if (capacity < p.gates.size()) {
            set_error("vqe_circuit_pass: gate_index capacity too small");
            return VQE_ERR_ARG;
        }
        for (size_t i = 0; i < p.gates.size(); ++i) gate_index[i] = p.gates[i];
    }
    return VQE_OK;
}

int vqe_apply_circuit(vqe_state* s, const vqe_circuit* c, const double* params, size_t n_params) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(s, "vqe_apply_circuit")) return rc;
    if (!c || c->n != s->n) {
        set_error("vqe_apply_circuit: circuit missing or of a different qubit count");
        return VQE_ERR_ARG;
    }
    if (int rc = check_params(c, params, n_params, "vqe_apply_circuit")) return rc;
    const int form = jit_mode();
    if (int rc = check_form(c, form, "vqe_apply_circuit")) return rc;
    VQE_HIP(hipSetDevice(s->device));
    const std::vector<size_t> nob;
    const std::vector<void*> nock;
    // any state whose norm square is in range
    return s->dtype == VQE_C64 ? forward<float>(s, c, form, params, nob, nock, false, 0x1p64)
                               : forward<double>(s, c, form, params, nob, nock, false, 0x1p512);
    VQE_GUARD_END
}

int vqe_apply_dense(vqe_state* s, const int* qubits, int k, const double* u) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(s, "vqe_apply_dense")) return rc;
    if (!qubits || !u) {
        set_error("vqe_apply_dense: null argument");
        return VQE_ERR_ARG;
    }
    if (k != kDenseK) {
        set_error("vqe_apply_dense: k must be " + std::to_string(kDenseK));
        return VQE_ERR_ARG;
    }
    DenseArgs a{};
    uint64_t seen = 0;
    for (int i = 0; i < k; ++i) {
        if (qubits[i] < 4 || qubits[i] >= s->n || ((seen >> qubits[i]) & 1)) {
            set_error("vqe_apply_dense: qubits must be distinct and in [4, n)");
            return VQE_ERR_ARG;
        }
        seen |= 1ull << qubits[i];
        a.q[i] = (uint32_t)qubits[i];
    }
    for (int i = 0, q = 0; q < s->n; ++q)
        if ((seen >> q) & 1) a.sorted[i++] = (uint32_t)q;
    a.n_tiles = 1ull << (s->n - kDenseK - 4);
    VQE_HIP(hipSetDevice(s->device));
    return s->dtype == VQE_C64 ? apply_dense<float>(s, a, u) : apply_dense<double>(s, a, u);
    VQE_GUARD_END
}

int vqe_hamiltonian_create(int n_qubits, const uint64_t* x, const uint64_t* z, const double* w, size_t n_terms,
                           vqe_hamiltonian** out) {
    VQE_GUARD_BEGIN
    if (!out || (n_terms && (!x || !z || !w))) {
        set_error("vqe_hamiltonian_create: null argument");
        return VQE_ERR_ARG;
    }
    if (n_qubits < 1 || n_qubits > 40) {
        set_error("vqe_hamiltonian_create: n_qubits must be in [1, 40]");
        return VQE_ERR_ARG;
    }
    if (n_terms == 0) {
        set_error("vqe_hamiltonian_create: no terms");
        return VQE_ERR_ARG;
    }
    const uint64_t lim = 1ull << n_qubits;
    for (size_t i = 0; i < n_terms; ++i) {
        if (x[i] >= lim || z[i] >= lim) {
            set_error("vqe_hamiltonian_create: term " + std::to_string(i) + " has a mask bit >= n_qubits");
            return VQE_ERR_ARG;
        }
        if (!std::isfinite(w[i])) {
            set_error("vqe_hamiltonian_create: term " + std::to_string(i) + " has a non-finite weight");
            return VQE_ERR_ARG;
        }
    }
    std::vector<size_t> idx(n_terms);
    std::iota(idx.begin(), idx.end(), 0);
    std::stable_sort(idx.begin(), idx.end(), [&](size_t a, size_t b) {
        return x[a] != x[b] ? x[a] < x[b] : z[a] < z[b];
    });
    auto* h = new vqe_hamiltonian();
    h->n = n_qubits;
    for (size_t k = 0; k < n_terms; ++k) {
        const size_t i = idx[k];
        if (!h->x.empty() && h->x.back() == x[i] && h->z.back() == z[i]) {
            h->w.back() += w[i];
        } else {
            h->x.push_back(x[i]);
            h->z.push_back(z[i]);
            h->w.push_back(w[i]);
        }
    }
    std::vector<TermDesc<float>>& t32 = h->t32;
    std::vector<TermDesc<double>>& t64 = h->t64;
    t32.resize(h->w.size());
    t64.resize(h->w.size());
    for (size_t t = 0; t < h->w.size(); ++t) {
        if (h->x[t] == 0 && h->z[t] == 0) h->identity += h->w[t];
        h->norm1 += std::fabs(h->w[t]);
        if (h->groups.empty() || h->groups.back().x != h->x[t]) {
            GroupDesc g{};
            g.x = h->x[t];
            g.begin = (uint32_t)t;
            g.hbit = h->x[t] ? 63 - __builtin_clzll(h->x[t]) : 0;
            h->groups.push_back(g);
        }
        h->groups.back().end = (uint32_t)t + 1;
        // c = w (-i)^y with y = popcount(x & z) mod 4
        const int y = __builtin_popcountll(h->x[t] & h->z[t]) & 3;
        const double wv = h->w[t];
        const double cre = (y == 0) ? wv : (y == 2 ? -wv : 0.0);
        const double cim = (y == 1) ? -wv : (y == 3 ? wv : 0.0);
        t64[t] = TermDesc<double>{h->z[t], cre, cim};
        t32[t] = TermDesc<float>{h->z[t], (float)cre, (float)cim};
        if (y & 1) h->real_coeffs = false;
    }
    plan_hwin(h);
    if (h->n <= kBatchMaxQubitsC64) {
        plan_small<float>(h, h->t32, h->sm_blocks[0], h->sm_stream[0]);
        plan_small<double>(h, h->t64, h->sm_blocks[1], h->sm_stream[1]);
    }
    *out = h;
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_hamiltonian_free(vqe_hamiltonian* h) {
    if (!h) return VQE_OK;
    free_hamiltonian_tables(h);
    delete h;
    return VQE_OK;
}

int vqe_hamiltonian_plan(const vqe_hamiltonian* h, size_t* n_windows, uint64_t* window_masks, size_t capacity) {
    if (!h || !n_windows) {
        set_error("vqe_hamiltonian_plan: null argument");
        return VQE_ERR_ARG;
    }
    const size_t m = h->hw_lam ? h->hw_wins.size() : 0;
    *n_windows = m;
    if (window_masks) {
        if (capacity < m) {
            set_error("vqe_hamiltonian_plan: window_masks capacity too small");
            return VQE_ERR_ARG;
        }
        for (size_t i = 0; i < m; ++i) {
            uint64_t wm = 0;
            for (int k = 0; k < kHwBits; ++k) wm |= 1ull << h->hw_wins[i].pos[k];
            window_masks[i] = wm;
        }
    }
    return VQE_OK;
}

int vqe_hamiltonian_info(const vqe_hamiltonian* h, size_t* n_terms, size_t* n_groups, double* identity_weight) {
    if (!h) {
        set_error("vqe_hamiltonian_info: null Hamiltonian");
        return VQE_ERR_ARG;
    }
    if (n_terms) *n_terms = h->w.size();
    if (n_groups) *n_groups = h->groups.size();
    if (identity_weight) *identity_weight = h->identity;
    return VQE_OK;
}

int vqe_expect_pauli(vqe_state* s, const vqe_hamiltonian* h, int mode, double* energy, double* norm) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(s, "vqe_expect_pauli")) return rc;
    if (!h || h->n != s->n || !energy) {
        set_error("vqe_expect_pauli: Hamiltonian missing, of a different qubit count, or null energy");
        return VQE_ERR_ARG;
    }
    if (mode != VQE_EXPECT_GROUPED && mode != VQE_EXPECT_PER_TERM) {
        set_error("vqe_expect_pauli: unknown mode");
        return VQE_ERR_ARG;
    }
    VQE_HIP(hipSetDevice(s->device));
    if (int rc = upload_hamiltonian(h)) return rc;
    if (int rc = ensure_part(s)) return rc;
    return s->dtype == VQE_C64 ? expect_impl<float>(s, h, mode, energy, norm)
                               : expect_impl<double>(s, h, mode, energy, norm);
    VQE_GUARD_END
}

int vqe_apply_hamiltonian(vqe_state* psi, vqe_state* lam, const vqe_hamiltonian* h, double* energy, double* norm) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(psi, "vqe_apply_hamiltonian")) return rc;
    if (int rc = check_state(lam, "vqe_apply_hamiltonian")) return rc;
    if (psi == lam || psi->data == lam->data || lam->n != psi->n || lam->dtype != psi->dtype || !h ||
        h->n != psi->n) {
        set_error("vqe_apply_hamiltonian: lam must be a distinct state of the same n and dtype as psi");
        return VQE_ERR_ARG;
    }
    VQE_HIP(hipSetDevice(psi->device));
    int rc = upload_hamiltonian(h);
    if (rc) return rc;
    if ((rc = ensure_part(psi))) return rc;
    rc = ensure_res(psi, 2);
    if (rc) return rc;
    rc = psi->dtype == VQE_C64 ? apply_h<float>(psi, lam->data, h, psi->d_res)
                               : apply_h<double>(psi, lam->data, h, psi->d_res);
    if (rc) return rc;
    VQE_HIP(hipMemcpyAsync(psi->h_res, psi->d_res, 2 * sizeof(double), hipMemcpyDeviceToHost, psi->stream));
    VQE_HIP(hipStreamSynchronize(psi->stream));
    if (energy) *energy = psi->h_res[0] / psi->h_res[1];
    if (norm) *norm = psi->h_res[1];
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_energy_grad(vqe_state* psi, vqe_state* lam, const vqe_circuit* c, const double* params, size_t n_params,
                    const vqe_hamiltonian* h, const vqe_grad_opts* opts, double* energy, double* grad) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(psi, "vqe_energy_grad")) return rc;
    if (!c || c->n != psi->n || !h || h->n != psi->n || !energy || (n_params && !grad)) {
        set_error("vqe_energy_grad: circuit / Hamiltonian missing or of a different qubit count, or null output");
        return VQE_ERR_ARG;
    }
    if (int rc = check_params(c, params, n_params, "vqe_energy_grad")) return rc;
    const int form = jit_mode();
    if (int rc = check_form(c, form, "vqe_energy_grad")) return rc;
    const int method = opts ? opts->method : VQE_GRAD_ADJOINT;
    VQE_HIP(hipSetDevice(psi->device));
    if (int rc = upload_hamiltonian(h)) return rc;
    if (int rc = ensure_part(psi)) return rc;
    if (method == VQE_GRAD_PARAM_SHIFT) {
        const int mode = opts ? opts->expect_mode : VQE_EXPECT_GROUPED;
        if (mode != VQE_EXPECT_GROUPED && mode != VQE_EXPECT_PER_TERM) {
            set_error("vqe_energy_grad: unknown expect_mode");
            return VQE_ERR_ARG;
        }
        return psi->dtype == VQE_C64 ? param_shift_impl<float>(psi, c, form, params, h, mode, energy, grad)
                                     : param_shift_impl<double>(psi, c, form, params, h, mode, energy, grad);
    }
    if (method != VQE_GRAD_ADJOINT) {
        set_error("vqe_energy_grad: unknown method");
        return VQE_ERR_ARG;
    }
    if (int rc = check_state(lam, "vqe_energy_grad")) return rc;
    if (lam == psi || lam->data == psi->data || lam->n != psi->n || lam->dtype != psi->dtype) {
        set_error("vqe_energy_grad: lam must be a distinct state of the same n and dtype as psi");
        return VQE_ERR_ARG;
    }
    if (opts && opts->chunk_passes < 0) {
        set_error("vqe_energy_grad: chunk_passes must be >= 0");
        return VQE_ERR_ARG;
    }
    if (opts && opts->n_ckpt > 0) {
        if (!opts->ckpt) {
            set_error("vqe_energy_grad: n_ckpt > 0 with a null ckpt array");
            return VQE_ERR_ARG;
        }
        for (int k = 0; k < opts->n_ckpt; ++k) {
            const vqe_state* ck = opts->ckpt[k];
            if (!ck || !ck->data || ck->n != psi->n || ck->dtype != psi->dtype || ck->data == psi->data ||
                ck->data == lam->data) {
                set_error("vqe_energy_grad: checkpoint " + std::to_string(k) +
                          " must be a distinct state of the same n and dtype as psi");
                return VQE_ERR_ARG;
            }
            for (int j = 0; j < k; ++j)
                if (opts->ckpt[j]->data == ck->data) {
                    set_error("vqe_energy_grad: checkpoint states must be distinct");
                    return VQE_ERR_ARG;
                }
        }
    }
    // A state that fits LDS runs in one launch, whatever its gates, unless a
    // kernel form was chosen.  12 qubits, 4 layers, complex128: 26 launches of 1 to 8
    // blocks 408 us, against one of one block 188 us.
    if (form == VQE_SPECIALIZE_AUTO && psi->n <= max_small(psi->dtype))
        return psi->dtype == VQE_C64 ? small_grad<float>(psi, lam, c, params, h, opts, energy, grad)
                                     : small_grad<double>(psi, lam, c, params, h, opts, energy, grad);
    // Above that, where specialised kernels are not worth compiling, the batch
    // programs of mid-size items on the caller's states: 2 to 4 passes over
    // 12-qubit windows instead of 10 to 30 over 5 qubits.  4 / 12 layers, interpreted
    // window passes against these: complex64 14 qubits 478 / 1247 us, 209 / 498;
    // 19 qubits 666 / 1784, 326 / 782; complex128 13 qubits 441 / 1179, 249 / 626; 19
    // qubits 752 / 1963, 405 / 1010.
    if (form == VQE_SPECIALIZE_AUTO && psi->n < VQE_SPECIALIZE_AUTO_MIN_QUBITS && !use_tiles(c, form)) {
        if (!psi->mid) {
            psi->mid = new vqe_batch();
            psi->mid->dtype = psi->dtype;
            psi->mid->stream = psi->stream;
            psi->mid->device = psi->device;
        }
        const vqe_batch_item it{c, h, params, n_params, energy, grad};
        const MidOwn own{psi, lam, opts};
        return psi->dtype == VQE_C64 ? mid_impl<float>(psi->mid, &it, {0}, &own) : mid_impl<double>(psi->mid, &it, {0}, &own);
    }
    return psi->dtype == VQE_C64 ? adjoint_impl<float>(psi, lam, c, form, params, h, opts, energy, grad)
                                 : adjoint_impl<double>(psi, lam, c, form, params, h, opts, energy, grad);
    VQE_GUARD_END
}

int vqe_batch_create(int dtype, void* hip_stream, vqe_batch** out) {
    VQE_GUARD_BEGIN
    if (!out || (dtype != VQE_C64 && dtype != VQE_C128)) {
        set_error("vqe_batch_create: null out or bad dtype");
        return VQE_ERR_ARG;
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) {
        set_error("vqe_batch_create: no HIP device");
        return VQE_ERR_DEVICE;
    }
    if (int rc = small_lds_limit()) return rc;
    auto* b = new vqe_batch();
    b->dtype = dtype;
    b->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&b->device) != hipSuccess) {
        delete b;
        set_error("vqe_batch_create: hipGetDevice failed");
        return VQE_ERR_DEVICE;
    }
    *out = b;
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_batch_free(vqe_batch* b) {
    if (!b) return VQE_OK;
    (void)hipSetDevice(b->device);
    (void)hipStreamSynchronize(b->stream);
    if (b->d_buf) (void)hipFree(b->d_buf);
    if (b->h_buf) (void)hipHostFree(b->h_buf);
    if (b->md_buf) (void)hipFree(b->md_buf);
    if (b->mh_buf) (void)hipHostFree(b->mh_buf);
    delete b;
    return VQE_OK;
}

int vqe_batch_energy_grad(vqe_batch* b, size_t n_items, const vqe_batch_item* items) {
    VQE_GUARD_BEGIN
    if (!b || (n_items && !items)) {
        set_error("vqe_batch_energy_grad: null batch or items");
        return VQE_ERR_ARG;
    }
    if (n_items == 0) return VQE_OK;
    if (n_items > (1u << 20)) {
        set_error("vqe_batch_energy_grad: too many items in one batch (limit 2^20)");
        return VQE_ERR_ARG;
    }
    VQE_HIP(hipSetDevice(b->device));
    // Items up to the LDS limit go to the small-state kernel, larger ones up
    // to kMidMaxQubits to the tile passes; every item is checked first.
    std::vector<vqe_batch_item> small;
    std::vector<size_t> mid;
    for (size_t i = 0; i < n_items; ++i) {
        const vqe_batch_item& it = items[i];
        if (!it.circuit || !it.hamiltonian || !it.energy || (it.n_params && (!it.params || !it.grad))) {
            set_error("vqe_batch_energy_grad: item " + std::to_string(i) + " has a null field");
            return VQE_ERR_ARG;
        }
        const int n = it.circuit->n;
        if (n > kMidMaxQubits || it.hamiltonian->n != n) {
            set_error("vqe_batch_energy_grad: item " + std::to_string(i) + " has " + std::to_string(n) +
                      " qubits (limit " + std::to_string(kMidMaxQubits) + ") or a Hamiltonian of another size");
            return VQE_ERR_ARG;
        }
        if (int rc = check_params(it.circuit, it.params, it.n_params, "vqe_batch_energy_grad")) return rc;
        if (n <= max_small(b->dtype)) small.push_back(it);
        else mid.push_back(i);
    }
    if (!small.empty()) {
        const int rc = b->dtype == VQE_C64 ? batch_impl<float>(b, small.size(), small.data())
                                           : batch_impl<double>(b, small.size(), small.data());
        if (rc) return rc;
    }
    if (!mid.empty()) return b->dtype == VQE_C64 ? mid_impl<float>(b, items, mid) : mid_impl<double>(b, items, mid);
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_circuit_prepare(const vqe_circuit* c, int dtype) {
    VQE_GUARD_BEGIN
    if (!c || (dtype != VQE_C64 && dtype != VQE_C128)) {
        set_error("vqe_circuit_prepare: null circuit or bad dtype");
        return VQE_ERR_ARG;
    }
    const int form = jit_mode();
    if (int rc = check_form(c, form, "vqe_circuit_prepare")) return rc;
    const int d = dtype == VQE_C128 ? 1 : 0;
    // the programs of batches and of single evaluations in the default form
    if (form == VQE_SPECIALIZE_AUTO && c->n <= kMidMaxQubits)
        if (int rc = ensure_batch(c, d)) return rc;
    if (use_tiles(c, form)) return ensure_tiles(c, d);
    const Plan& pl = plan_of(c, form);
    if (!pl.jit) return VQE_OK;
    return ensure_jit(c, pl, d);
    VQE_GUARD_END
}

int vqe_set_specialize(int mode) {
    if (mode != VQE_SPECIALIZE_NEVER && mode != VQE_SPECIALIZE_AUTO && mode != VQE_SPECIALIZE_ALWAYS) {
        vqe::set_error("vqe_set_specialize: unknown mode");
        return VQE_ERR_ARG;
    }
    return vqe::jit_set_mode(mode);
}

int vqe_stream_create(const uint32_t* cu_mask, size_t mask_words, void** stream) {
    VQE_GUARD_BEGIN
    if (!stream || (mask_words && !cu_mask)) {
        set_error("vqe_stream_create: null argument");
        return VQE_ERR_ARG;
    }
    hipStream_t st = nullptr;
    if (mask_words == 0) {
        VQE_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
    } else {
        int dev = 0, ncu = 0;
        VQE_HIP(hipGetDevice(&dev));
        VQE_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        size_t on = 0;
        for (size_t i = 0; i < mask_words; ++i)
            for (int b = 0; b < 32; ++b)
                if (((cu_mask[i] >> b) & 1) && (int)(32 * i + b) < ncu) ++on;
        if (on == 0) {
            set_error("vqe_stream_create: the CU mask selects no compute unit of the device");
            return VQE_ERR_ARG;
        }
        VQE_HIP(hipExtStreamCreateWithCUMask(&st, (uint32_t)mask_words, cu_mask));
    }
    *stream = st;
    return VQE_OK;
    VQE_GUARD_END
}

int vqe_stream_destroy(void* stream) {
    if (!stream) return VQE_OK;
    VQE_HIP(hipStreamDestroy((hipStream_t)stream));
    return VQE_OK;
}

int vqe_profile_enable(int on) {
    std::lock_guard<std::mutex> g(g_prof_mu);
    g_prof_on = on != 0;
    return VQE_OK;
}

int vqe_profile_reset(void) {
    std::lock_guard<std::mutex> g(g_prof_mu);
    prof_drain();
    for (auto& t : g_prof_tot) t = ProfTotals{};
    return VQE_OK;
}

int vqe_profile_read(int kind, uint64_t* launches, double* total_ms, double* bytes) {
    if (kind < 0 || kind >= VQE_KERNEL_KINDS) {
        set_error("vqe_profile_read: unknown kernel kind");
        return VQE_ERR_ARG;
    }
    std::lock_guard<std::mutex> g(g_prof_mu);
    prof_drain();
    if (launches) *launches = g_prof_tot[kind].launches;
    if (total_ms) *total_ms = g_prof_tot[kind].ms;
    if (bytes) *bytes = g_prof_tot[kind].bytes;
    return VQE_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- grouped energy without allocation
// Scratch memory of vqe_expect_pauli_noalloc: the per-block partial sums of
// the energy sweep (kEnergyPartBlocks blocks x 2) and the two reduced sums,
// in a fixed device array.  Each device that runs the call holds its own
// copy until the process ends.  Host code never passes the array's name to a
// kernel: it uses the address hipGetSymbolAddress returns on each device.
namespace {
constexpr size_t kScratchPart = 2 * (size_t)kEnergyPartBlocks;
constexpr size_t kScratchDoubles = kScratchPart + 32;  // partials | sums[2] | pad
static_assert(kScratchDoubles * sizeof(double) == VQE_NOALLOC_SCRATCH_BYTES, "scratch size and its public limit differ");
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
// Address of this device's scratch array, looked up once per device with that
// device current.
int scratch_of_device(int dev, double** out) {
    if (dev < 0 || dev >= kScratchDevices) {
        set_error("vqe_expect_pauli_noalloc: device index beyond the scratch table");
        return VQE_ERR_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        double* p = nullptr;
        const hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error(std::string("vqe_expect_pauli_noalloc: hipGetSymbolAddress of the scratch array: ") +
                      hipGetErrorString(e));
            return VQE_ERR_DEVICE;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return VQE_OK;
}
}  // namespace

extern "C" {

int vqe_expect_pauli_noalloc(vqe_state* s, const vqe_hamiltonian* h, double* d_out) {
    VQE_GUARD_BEGIN
    if (int rc = check_state(s, "vqe_expect_pauli_noalloc")) return rc;
    if (!h || h->n != s->n || !d_out) {
        set_error("vqe_expect_pauli_noalloc: Hamiltonian missing, of a different qubit count, or null d_out");
        return VQE_ERR_ARG;
    }
    hipPointerAttribute_t attr{};
    if (hipPointerGetAttributes(&attr, d_out) != hipSuccess || attr.type != hipMemoryTypeDevice ||
        attr.device != s->device) {
        (void)hipGetLastError();
        set_error("vqe_expect_pauli_noalloc: d_out is not device memory of the state's device");
        return VQE_ERR_ARG;
    }
    if (!h->d_ready) {
        set_error("vqe_expect_pauli_noalloc: the Hamiltonian's tables are not on the device yet (any evaluation "
                  "with it, e.g. vqe_expect_pauli, uploads them)");
        return VQE_ERR_STATE;
    }
    const uint32_t blocks = energy_part_blocks(h, s->n);
    if ((size_t)blocks * 2 > kScratchPart) {
        set_error("vqe_expect_pauli_noalloc: the sweep needs " + std::to_string(blocks) +
                  " blocks of partial sums, more than the scratch holds (" + std::to_string(kEnergyPartBlocks) + ")");
        return VQE_ERR_UNSUPPORTED;
    }
    VQE_HIP(hipSetDevice(s->device));
    double* sc = nullptr;
    if (int rc = scratch_of_device(s->device, &sc)) return rc;
    double* sums = sc + kScratchPart;
    int rc = s->dtype == VQE_C64 ? energy_grouped<float>(s, h, sc, sums) : energy_grouped<double>(s, h, sc, sums);
    if (rc) return rc;
    VQE_HIP(launch_energy_ratio(sums, d_out, s->stream));
    return VQE_OK;
    VQE_GUARD_END
}

}  // extern "C"

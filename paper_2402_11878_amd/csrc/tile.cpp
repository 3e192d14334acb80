// Tile passes: the specialised kernels of states of at least kTileMinQubits
// qubits.  A pass reads and writes the state once, like a window pass, but
// its window has 12 or 13 qubits instead of 7: a block of 256 threads keeps
// the coset (2^T amplitudes) of psi, in reverse passes of lam too, in
// registers, 2^R amplitudes per thread and vector, and works through the
// window's gates in stages of R register bits each; between two stages the
// vectors change layout through LDS (one write and one read per amplitude,
// against four or more vector instructions per amplitude and lane transpose
// bit).  The state crosses HBM once per pass, so the pass count is what a
// large state pays for: 10 passes instead of 23 at 32 qubits x 8 layers.
//
// Measured against the 7-qubit window passes (whole call): 30 qubits complex128
// step 572 -> 310 ms (forward passes 6.2-7.5 ms, 4.6-5.5 TB/s; reverse 13.6-20
// ms, 5.0-3.4 TB/s, and 38 ms for the first window with its 184 gates), 28
// qubits complex64 93.9 -> 46.7 ms, 24 qubits complex128 7.09 -> 3.72 ms, 20
// qubits complex64 1.14 -> 0.52 ms.  What bounds a reverse pass: up to about 50
// gates HBM (and address translation where nine window qubits lie above a 2 MiB
// page), beyond that vector issue (75 % busy at 184 gates) and the LDS traffic
// between stages.
//
// What the generated code does about arithmetic, the second cost:
//   * permutation gates (CNOT, X) rename registers at generation time;
//   * RY and RX run unnormalised, R = c [[1, -t], [t, 1]] with t = tan(a/2) and
//     c = cos(a/2): two fused multiply-adds per amplitude instead of four
//     operations (three as shears); the factors c wait until the next
//     multiplication of the whole vector; near half a turn the half turn is made
//     first, by moves behind a branch on the table (the same for the whole launch);
//   * all diagonal gates (RZ, CZ) of a stage that can stand together are one
//     multiplication by a phase from a host-made table of 2^m entries, which
//     also carries the pending factors c;
//   * the Z-gradient terms of such a group come from one product
//     Im(conj(lam) psi) per amplitude and a tree of signed sums;
//   * gradient terms are summed over the lanes of a wave as they appear, two at
//     a time (each exchange halves the number of values), so that no more than
//     six values per thread wait and one lane ends up with each total.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <sstream>

#include "sched.h"

namespace vqe {
namespace {

struct Layout {
    int reg[8];  // tile bit of register bit i
    int thr[8];  // tile bit of thread bit i
};

struct Gen : StageScheduler {
    TileShape sh;
    int NV, N;
    std::ostringstream o;
    std::vector<int> loc;        // variable holding register entry p
    // gradient terms waiting at each level of the lane sums, as variables and their lane -> push map
    struct Node {
        std::string var;
        std::vector<int> lane;
    };
    std::vector<Node> level[7];
    int vars = 0, pushes = 0, chunk = 0;

    std::string R(int v, int p) const { return "r" + std::to_string(v) + "_" + std::to_string(loc[p]); }
    std::string I(int v, int p) const { return "i" + std::to_string(v) + "_" + std::to_string(loc[p]); }

    // ---- ops
    // c [[1, -t], [t, 1]] (RX: -i t for both signs), after a half turn if the
    // gate's flag is set.  Rotations of different bits are emitted together,
    // with one branch around all their half turns.
    struct Turn {
        StageOp k;
        uint32_t off, flag;
    };
    std::vector<Turn> turns;
    void rot(const StageOp& k) override {
        for (const Turn& t : turns)
            if (t.k.bit[0] == k.bit[0]) {
                turn();
                break;
            }
        const uint32_t off = gate_entry(TF_ROT, k.gate, 1), flag = out->n_flags++;
        out->entries.back().flag_word = flag / 32;
        out->entries.back().flag_bit = flag % 32;
        turns.push_back(Turn{k, off, flag});
        pending.push_back(k.gate);
    }
    template <typename F>
    void pairs(const StageOp& k, F emit) {
        const int b = 1 << k.bit[0];
        for (int p = 0; p < N; ++p)
            if (!(p & b))
                for (int v = 0; v < NV; ++v) emit(R(v, p), I(v, p), R(v, p | b), I(v, p | b));
    }
    void turn() {
        if (turns.empty()) return;
        using S = const std::string&;
        std::map<uint32_t, uint32_t> mask;  // flag word -> bits
        for (const Turn& t : turns) mask[t.flag / 32] |= 1u << (t.flag % 32);
        o << "  if (__builtin_expect(0";  // rare: out of the line of the instruction cache
        for (const auto& [w, m] : mask) o << " | flags(half" << w << ", " << m << "u)";
        o << ", 0)) {\n";
        for (const Turn& t : turns) {
            o << "   if (flags(half" << t.flag / 32 << ", " << (1u << (t.flag % 32)) << "u)) {\n";
            pairs(t.k, [&](S xr, S xi, S yr, S yi) {
                if (t.k.kind == K_ROTY)
                    o << "    half_turn(" << xr << ", " << yr << "); half_turn(" << xi << ", " << yi << ");\n";
                else
                    o << "    half_turn(" << yi << ", " << xr << "); half_turn(" << xi << ", " << yr << ");\n";
            });
            o << "   }\n";
        }
        o << "  }\n";
        for (const Turn& t : turns) {
            o << "  { const T t = tab[" << t.off << "];\n";
            pairs(t.k, [&](S xr, S xi, S yr, S yi) {
                o << "    { const T xr = " << xr << ", xi = " << xi << ", yr = " << yr << ", yi = " << yi << ";\n      ";
                if (t.k.kind == K_ROTY)
                    o << xr << " = xr - t * yr; " << xi << " = xi - t * yi; " << yr << " = yr + t * xr; " << yi
                      << " = yi + t * xi; }\n";
                else
                    o << xr << " = xr + t * yi; " << xi << " = xi - t * yr; " << yr << " = yr + t * xi; " << yi
                      << " = yi - t * xr; }\n";
            });
            o << "  }\n";
        }
        turns.clear();
    }

    void scale_by(uint32_t off) override {
        turn();
        o << "  { const T s = tab[" << off << "];\n";
        for (int p = 0; p < N; ++p)
            for (int v = 0; v < NV; ++v) o << "    " << R(v, p) << " *= s; " << I(v, p) << " *= s;\n";
        o << "  }\n";
    }

    void phase_by(uint32_t off, uint32_t mask) override {
        turn();
        const int m = __builtin_popcount(mask);
        for (uint32_t idx = 0; idx < (1u << m); ++idx) {
            o << "  { const T pr = tab[" << off + 2 * idx << "], pi = tab[" << off + 2 * idx + 1 << "];\n";
            for (int p = 0; p < N; ++p) {
                uint32_t at = 0;
                for (int b = 0, k = 0; b < sh.R; ++b)
                    if ((mask >> b) & 1) at |= ((uint32_t)(p >> b) & 1u) << k++;
                if (at != idx) continue;
                for (int v = 0; v < NV; ++v)
                    o << "    { const T ar = " << R(v, p) << ", ai = " << I(v, p) << "; " << R(v, p)
                      << " = pr * ar - pi * ai; " << I(v, p) << " = pr * ai + pi * ar; }\n";
            }
            o << "  }\n";
        }
    }

    // A real 2x2 matrix between two patterns (H; excitations).
    void matrix(const StageOp& k) override {
        turn();
        const uint32_t off = gate_entry(TF_R2, k.gate, 4);
        o << "  { const T ca = tab[" << off << "], cb = tab[" << off + 1 << "], cc = tab[" << off + 2 << "], cd = tab["
          << off + 3 << "];\n";
        uint32_t mask, A, B;
        stage_pattern((*gates)[k.gate], k, mask, A, B);
        for (int p = 0; p < N; ++p) {
            if ((p & (int)mask) != (int)A) continue;
            const int q = p ^ (int)(A ^ B);
            for (int v = 0; v < NV; ++v)
                o << "    { const T ar = " << R(v, p) << ", ai = " << I(v, p) << ", br = " << R(v, q) << ", bi = "
                  << I(v, q) << ";\n      " << R(v, p) << " = ca * ar + cb * br; " << I(v, p)
                  << " = ca * ai + cb * bi; " << R(v, q) << " = cc * ar + cd * br; " << I(v, q)
                  << " = cc * ai + cd * bi; }\n";
        }
        o << "  }\n";
    }

    void rename(const StageOp& k) override {
        turn();
        const int c = k.kind == K_CNOT ? 1 << k.bit[0] : 0, t = 1 << (k.kind == K_CNOT ? k.bit[1] : k.bit[0]);
        for (int p = 0; p < N; ++p)
            if ((p & c) == c && !(p & t)) std::swap(loc[p], loc[p | t]);
    }

    // ---- gradient terms
    std::string fresh() { return "v" + std::to_string(vars++); }

    // Hands over one term (an expression of type T, this thread's share).
    void push(const std::string& expr, int param) {
        const int id = pushes++;
        out->lane_param.resize(std::max<size_t>(out->lane_param.size(), 64 * (size_t)(id / 64 + 1)), -1);
        term_param.push_back(param);
        Node n{fresh(), std::vector<int>(64, id)};
        o << "  double " << n.var << " = (double)(" << expr << ");\n";
        carry(0, n);
        if (pushes % 64 == 0) flush();
    }
    std::vector<int> term_param;

    void carry(int lv, Node n) {
        while (lv < 6 && !level[lv].empty()) {
            n = join(lv, level[lv].back(), n);
            level[lv].pop_back();
            ++lv;
        }
        if (lv == 6) total(n);
        else level[lv].push_back(n);
    }

    // Sum of a (lanes with bit 5 - lv clear) and b (set) over that lane bit.
    Node join(int lv, const Node& a, const Node& b) {
        Node n{fresh(), a.lane};
        for (int l = 0; l < 64; ++l)
            if ((l >> (5 - lv)) & 1) n.lane[l] = b.lane[l];
        o << "  double " << n.var << " = comb<" << 5 - lv << ">(" << a.var << ", " << b.var << ");\n";
        return n;
    }

    void total(const Node& n) {
        o << "  acc" << chunk << " += " << n.var << ";\n";
        std::vector<char> seen(pushes, 0);
        for (int l = 0; l < 64; ++l)
            if (!seen[n.lane[l]]) {
                seen[n.lane[l]] = 1;
                out->lane_param[64 * chunk + l] = term_param[n.lane[l]];
            }
        ++chunk;
    }

    // Brings every waiting term to a total (missing partners: the value itself on both halves).
    void flush() {
        bool any = false;
        for (auto& l : level) any = any || !l.empty();
        if (!any) return;
        Node carry_n;
        bool have = false;
        for (int lv = 0; lv < 6; ++lv) {
            Node* here = level[lv].empty() ? nullptr : &level[lv].back();
            if (!here && !have) continue;
            Node n = here && have ? join(lv, *here, carry_n) : here ? join(lv, *here, *here) : join(lv, carry_n, carry_n);
            level[lv].clear();
            carry_n = n;
            have = true;
        }
        total(carry_n);
    }

    void gradient(const StageOp& k) override {
        turn();
        const Gate& g = (*gates)[k.gate];
        uint32_t mask, A, B;
        stage_pattern((*gates)[k.gate], k, mask, A, B);
        const std::string acc = fresh();
        o << "  T " << acc << " = 0;\n";
        for (int p = 0; p < N; ++p) {
            if ((p & (int)mask) != (int)A) continue;
            const int q = p ^ (int)(A ^ B);
            const std::string pr = R(0, p), pi = I(0, p), qr = R(0, q), qi = I(0, q);
            const std::string lr = R(1, p), li = I(1, p), mr = R(1, q), mi = I(1, q);
            if (g.kind == VQE_GATE_RX)  // Im<lam|X|psi>
                o << "  " << acc << " += " << lr << " * " << qi << "; " << acc << " -= " << li << " * " << qr << "; "
                  << acc << " += " << mr << " * " << pi << "; " << acc << " -= " << mi << " * " << pr << ";\n";
            else  // Im<lam|Y|psi>, and Re<lam|K|psi> with K = |B><A| - |A><B| of an excitation: the same form
                o << "  " << acc << " += " << mr << " * " << pr << "; " << acc << " += " << mi << " * " << pi << "; "
                  << acc << " -= " << lr << " * " << qr << "; " << acc << " -= " << li << " * " << qi << ";\n";
        }
        push(acc, g.pidx);
    }

    // Im<lam|Z_b|psi> for the bits of the given RZ gates: d = Im(conj(lam) psi)
    // per entry once, then for each bit the sum of differences, passing the sums on.
    void gradient_z(const std::vector<StageOp>& ops) override {
        turn();
        std::vector<std::string> d(N);
        for (int p = 0; p < N; ++p) {
            d[p] = fresh();
            o << "  T " << d[p] << " = " << R(1, p) << " * " << I(0, p) << "; " << d[p] << " -= " << I(1, p) << " * "
              << R(0, p) << ";\n";
        }
        uint32_t want = 0;
        for (const StageOp& k : ops) want |= 1u << k.bit[0];
        for (int b = 0; b < sh.R; ++b) {
            const size_t half = d.size() / 2;  // entries are indexed by the bits b and up
            std::vector<std::string> s(half);
            if ((want >> b) & 1) {
                const std::string acc = fresh();
                for (size_t i = 0; i < half; ++i)
                    o << (i ? "  " + acc + " += " : "  T " + acc + " = ") << d[2 * i] << " - " << d[2 * i + 1] << ";\n";
                // every parameterised gate on the bit has this term
                for (const StageOp& k : ops)
                    if (k.bit[0] == b) push(acc, (*gates)[k.gate].pidx);
            }
            if (!(want >> (b + 1))) break;
            for (size_t i = 0; i < half; ++i) {
                s[i] = fresh();
                o << "  T " << s[i] << " = " << d[2 * i] << " + " << d[2 * i + 1] << ";\n";
            }
            d.swap(s);
        }
    }

    // ---- layouts
    bool split = false;  // exchange real and imaginary parts one after the other (half the LDS)
    int elem_bytes() const { return (dbl ? 16 : 8) / (split ? 2 : 1); }
    int bank_bits() const { return dbl ? (split ? 4 : 3) : (split ? 5 : 4); }  // 128 bytes, what LDS serves per clock

    // LDS slot of tile index j: the lowest bank_bits() bits are XORed with all
    // groups of bits above them, so that amplitudes a fixed power of two apart
    // lie in different banks.
    uint32_t slot(uint32_t j) const {
        const int nb = bank_bits();
        uint32_t f = 0;
        for (uint32_t v = j >> nb; v; v >>= nb) f ^= v;
        return j ^ (f & ((1u << nb) - 1));
    }

    // Layout with register bits `regs` and wave bits `wave` (tile bits); the
    // others go to the lanes in ascending order, for loads and stores, or with
    // lowest lane bits that differ modulo bank_bits() (conflict-free in LDS).
    Layout layout(const std::vector<int>& regs, const std::vector<int>& wave, bool memory) const {
        Layout L{};
        std::vector<int> rest;
        for (int b = 0; b < sh.T; ++b)
            if (std::find(regs.begin(), regs.end(), b) == regs.end() &&
                std::find(wave.begin(), wave.end(), b) == wave.end())
                rest.push_back(b);
        if (!memory) {
            const int nb = bank_bits();
            std::vector<int> first;
            uint32_t used = 0;
            for (int b : rest)
                if ((int)first.size() < nb && !((used >> (b % nb)) & 1)) {
                    first.push_back(b);
                    used |= 1u << (b % nb);
                }
            for (int b : rest)
                if (std::find(first.begin(), first.end(), b) == first.end()) first.push_back(b);
            rest = first;
        }
        rest.insert(rest.end(), wave.begin(), wave.end());
        for (int i = 0; i < sh.R; ++i) L.reg[i] = regs[i];
        for (int i = 0; i < sh.T - sh.R; ++i) L.thr[i] = rest[i];
        return L;
    }

    // The thread's byte offset in LDS under layout L, as variable `b0`, and its
    // variants with some of the low slot bits flipped.
    void lds_base(const Layout& L) {
        const int nb = bank_bits(), eb = elem_bytes();
        o << "    u32 t_ = tid; asm volatile(\"\" : \"+v\"(t_));\n    const u32 j = 0";
        const int TB = sh.T - sh.R;
        for (int k = 0; k < TB;) {
            int e = k + 1;
            while (e < TB && L.thr[e] == L.thr[e - 1] + 1) ++e;
            o << " | (((t_ >> " << k << ") & " << ((1u << (e - k)) - 1) << "u) << " << L.thr[k] << ")";
            k = e;
        }
        o << ";\n    const u32 b0 = (j ^ ((0";
        for (int s = nb; s < sh.T; s += nb) o << " ^ (j >> " << s << ")";
        o << ") & " << ((1u << nb) - 1) << "u)) * " << eb << "u;\n";
        std::vector<uint32_t> flips;
        for (int p = 0; p < N; ++p) flips.push_back(reg_slot(L, p) & ((1u << nb) - 1));
        std::sort(flips.begin(), flips.end());
        flips.erase(std::unique(flips.begin(), flips.end()), flips.end());
        for (uint32_t f : flips)
            if (f) o << "    const u32 b" << f << " = b0 ^ " << f * (uint32_t)eb << "u;\n";
    }

    uint32_t reg_slot(const Layout& L, int p) const {
        uint32_t j = 0;
        for (int i = 0; i < sh.R; ++i)
            if ((p >> i) & 1) j |= 1u << L.reg[i];
        return slot(j);
    }

    std::string lds_at(const Layout& L, int p) const {
        const uint32_t s = reg_slot(L, p), m = (1u << bank_bits()) - 1;
        return std::string(split ? "*(T*)" : "*(V*)") + "(lds + b" + std::to_string(s & m) + " + " +
               std::to_string((s & ~m) * (uint32_t)elem_bytes()) + "u)";
    }

    // Changes the layout of every vector through LDS.  If both layouts have
    // the same wave bits, every wave writes and reads the same quarter of the
    // buffer, its own: no barrier.  Otherwise one barrier between writing and
    // reading, and one before the next vector overwrites the buffer.  None is
    // needed before the first write: the reads of the exchange before it lay in
    // this layout's own quarters.  LDS serves a wave's accesses in order, so
    // between a wave's own writes and reads only the compiler has to be held
    // back (wave_sync: lanes exchange data, which it does not see).
    void exchange(const Layout& from, const Layout& to) {
        const int W = sh.T - sh.R;
        const bool own = std::equal(from.thr + 6, from.thr + W, to.thr + 6);
        const std::vector<int> old = loc;
        std::vector<int> ident(N);
        for (int p = 0; p < N; ++p) ident[p] = p;
        bool first = true;
        for (int v = 0; v < NV; ++v) {
            std::vector<std::string> got(N);
            for (int half = 0; half < (split ? 2 : 1); ++half) {
                o << (!own && !first ? "  __syncthreads();\n" : "  wave_sync();\n");
                first = false;
                loc = old;
                o << "  {\n";
                lds_base(from);
                for (int p = 0; p < N; ++p) {
                    o << "    " << lds_at(from, p) << " = ";
                    if (split) o << (half ? I(v, p) : R(v, p)) << ";\n";
                    else o << "V{" << R(v, p) << ", " << I(v, p) << "};\n";
                }
                o << "  }\n" << (own ? "  wave_sync();\n" : "  __syncthreads();\n");
                loc = ident;
                if (split) {
                    for (int p = 0; p < N; ++p) got[p] = fresh(), o << "  T " << got[p] << ";\n";
                    o << "  {\n";
                    lds_base(to);
                    for (int p = 0; p < N; ++p) o << "    " << got[p] << " = " << lds_at(to, p) << ";\n";
                    o << "  }\n";
                    for (int p = 0; p < N; ++p) o << "  " << (half ? I(v, p) : R(v, p)) << " = " << got[p] << ";\n";
                } else {
                    o << "  {\n";
                    lds_base(to);
                    for (int p = 0; p < N; ++p)
                        o << "    { const V w = " << lds_at(to, p) << "; " << R(v, p) << " = w.x; " << I(v, p)
                          << " = w.y; }\n";
                    o << "  }\n";
                }
            }
        }
        loc = ident;
    }

    std::string reg_offset(const Layout& L, int p) const {
        std::string e;
        for (int i = 0; i < sh.R; ++i)
            if ((p >> i) & 1) e += (e.empty() ? "bit[" : " + bit[") + std::to_string(L.reg[i]) + "]";
        return e.empty() ? "0" : e;
    }

    void thread_offset(const char* name, const Layout& L) {
        o << "  u64 " << name << " = 0;\n";
        for (int k = 0; k < sh.T - sh.R; ++k)
            o << "  if ((tid >> " << k << ") & 1) " << name << " += bit[" << L.thr[k] << "];\n";
    }
};

std::string prelude(bool dbl) {
    const char* T = dbl ? "double" : "float";
    std::ostringstream o;
    o << "typedef unsigned long long u64;\ntypedef unsigned int u32;\ntypedef " << T << " T;\n"
      << "struct __attribute__((aligned(" << (dbl ? 16 : 8) << "))) V { T x, y; };\n"
      << "struct TileArgs { u64 n_units; u32 pos[" << kTileMaxBits << "]; u32 first; };\n"
      // not taken out of the loop over cosets, where every test would keep its own registers
      << "__device__ __forceinline__ u32 flags(u32 w, u32 m) { asm volatile(\"\" : \"+s\"(w)); return w & m; }\n"
      // (x, y) -> (-y, x)
      << "__device__ __forceinline__ void half_turn(T& x, T& y) { const T w = x; x = -y; y = w; }\n"
      << "__device__ __forceinline__ void wave_sync() {\n"
      << "  __builtin_amdgcn_fence(__ATOMIC_RELEASE, \"wavefront\");\n  __builtin_amdgcn_wave_barrier();\n"
      << "  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, \"wavefront\");\n}\n"
      // comb<L>(a, b): lanes with bit L clear get the sum of a over that bit, lanes with it set the sum of b.
      // L = 5, 4: one swap per dword exchanges the halves; below, DPP: row_ror:8, row_half_mirror (pairs
      // lane l with l ^ 7: the lower bits are summed later) and quad permutes.
      << "template <int L> __device__ __forceinline__ u32 dpp(u32 v) {\n"
      << "  constexpr int C = L == 3 ? 0x128 : L == 2 ? 0x141 : L == 1 ? 0x4E : 0xB1;\n"
      << "  return (u32)__builtin_amdgcn_update_dpp(0, (int)v, C, 0xF, 0xF, false);\n}\n"
      << "template <int L> __device__ __forceinline__ double comb(double a, double b) {\n"
      << "  const u64 x = __builtin_bit_cast(u64, a), y = __builtin_bit_cast(u64, b);\n"
      << "  if constexpr (L >= 4) {\n"
      << "    const auto l = L == 5 ? __builtin_amdgcn_permlane32_swap((u32)x, (u32)y, false, false)\n"
      << "                          : __builtin_amdgcn_permlane16_swap((u32)x, (u32)y, false, false);\n"
      << "    const auto h = L == 5 ? __builtin_amdgcn_permlane32_swap((u32)(x >> 32), (u32)(y >> 32), false, false)\n"
      << "                          : __builtin_amdgcn_permlane16_swap((u32)(x >> 32), (u32)(y >> 32), false, false);\n"
      << "    return __builtin_bit_cast(double, ((u64)h[0] << 32) | l[0]) +\n"
      << "           __builtin_bit_cast(double, ((u64)h[1] << 32) | l[1]);\n"
      << "  } else {\n"
      << "    const bool hb = (threadIdx.x >> L) & 1;\n"
      << "    const u64 keep = hb ? y : x, send = hb ? x : y;\n"
      << "    const u64 got = ((u64)dpp<L>((u32)(send >> 32)) << 32) | dpp<L>((u32)send);\n"
      << "    return __builtin_bit_cast(double, keep) + __builtin_bit_cast(double, got);\n"
      << "  }\n}\n";
    return o.str();
}

// Factor f and number t of an unnormalised rotation f [[1, -t], [t, 1]]: f =
// cos(a/2) and t = tan(a/2), or where that is beyond `limit` (returns true)
// those of the rotation by a - pi that is left after (x, y) -> (-y, x): f =
// sin(a/2), t = -cot(a/2).
bool rot_numbers(const HalfAngle& h, double sign, double limit, double& f, double& t) {
    const double s = sign * h.s;
    const bool half = std::fabs(s) > limit * std::fabs(h.c);
    f = half ? s : h.c;
    t = half ? -h.c / s : s / h.c;
    return half;
}

}  // namespace

const char* tile_kernel_name(int NV, bool dbl) {
    return NV == 2 ? (dbl ? "vqe_tile_rev_c128" : "vqe_tile_rev_c64") : (dbl ? "vqe_tile_fwd_c128" : "vqe_tile_fwd_c64");
}

bool tile_kernel(bool dbl, const TileShape& sh, const std::vector<Gate>& gates, const PlannedPass& p, int dir,
                 TileKernel& out, std::string& msg) {
    if (p.K != sh.T) {
        msg = "tile pass of the wrong size (internal error)";
        return false;
    }
    int local[64] = {0};
    for (int j = 0; j < p.K; ++j) local[p.pos[j]] = j;
    std::vector<Gate> lg;
    for (int gi : p.gates) {
        Gate g = gates[gi];
        g.q0 = local[g.q0];
        g.q1 = local[g.q1];
        g.q2 = local[g.q2];
        g.q3 = local[g.q3];
        lg.push_back(g);
    }
    // stages: the window's gates by R register bits
    std::vector<PlannedPass> stages;
    const int big = 1 << 20;
    if (!plan_passes(sh.T, lg, PlanLimits{sh.R, big, big, big}, stages, msg)) return false;
    Gen g;
    g.dbl = dbl;
    g.sh = sh;
    g.NV = dir == 1 ? 2 : 1;
    g.N = 1 << sh.R;
    g.gates = &gates;
    g.split = dir == 0;  // forward passes: half the LDS, twice the blocks per CU
    g.out = &out;
    g.loc.resize(g.N);
    for (int i = 0; i < g.N; ++i) g.loc[i] = i;
    out = TileKernel();
    out.n_scalars = kTileFlagBytes / (dbl ? 8 : 4);  // the flags of half turns come first

    if (dir == 1) std::reverse(stages.begin(), stages.end());

    // Layouts: the load, one per stage, the store.  Loads and stores keep the
    // lowest bits in the lanes (runs of 128 or 64 bytes).  The two wave bits of every
    // layout are chosen so that as few layout changes as possible move data
    // between waves (those need barriers): a shortest path over the pairs.
    struct Node {
        uint32_t used;
        bool memory;
    };
    const uint32_t low = (1u << sh.low) - 1;
    std::vector<Node> nodes{{0, true}};
    for (const PlannedPass& s : stages) {
        uint32_t u = 0;
        for (int j = 0; j < s.K; ++j) u |= 1u << s.pos[j];
        nodes.push_back({u, false});
    }
    nodes.push_back({0, true});
    // a stage off the lowest bits takes the layout of the load or store beside it
    if (nodes.size() > 2 && !(nodes[1].used & low)) {
        nodes[1].memory = true;
        nodes.erase(nodes.begin());
    }
    const bool load_is_stage = !stages.empty() && nodes[0].used != 0;
    if (nodes.size() > 1 && !(nodes[nodes.size() - 2].used & low) && !stages.empty()) {
        nodes[nodes.size() - 2].memory = true;
        nodes.pop_back();
    }
    const int wave_bits = sh.T - sh.R - 6;
    std::vector<uint32_t> pairs;
    for (uint32_t m = 0; m < (1u << sh.T); ++m)
        if (__builtin_popcount(m) == wave_bits) pairs.push_back(m);
    auto fits = [&](const Node& nd, uint32_t w) { return !(w & nd.used) && !(nd.memory && (w & low)); };
    std::vector<std::vector<int>> best(nodes.size(), std::vector<int>(pairs.size(), 1 << 20)), from(best);
    for (size_t i = 0; i < nodes.size(); ++i)
        for (size_t w = 0; w < pairs.size(); ++w) {
            if (!fits(nodes[i], pairs[w])) continue;
            if (i == 0) best[i][w] = 0;
            for (size_t v = 0; i > 0 && v < pairs.size(); ++v)
                if (best[i - 1][v] + (v != w) < best[i][w]) {
                    best[i][w] = best[i - 1][v] + (v != w);
                    from[i][w] = (int)v;
                }
        }
    size_t at = std::min_element(best.back().begin(), best.back().end()) - best.back().begin();
    if (best.back()[at] >= (1 << 20)) {
        msg = "tile pass without a layout (internal error)";
        return false;
    }
    std::vector<Layout> layouts(nodes.size());
    std::vector<std::vector<int>> regs(nodes.size());
    for (size_t i = nodes.size(); i-- > 0;) {
        std::vector<int> wave;
        for (int b = 0; b < sh.T; ++b)
            if ((pairs[at] >> b) & 1) wave.push_back(b);
        std::vector<int>& r = regs[i];
        for (int b = 0; b < sh.T; ++b)
            if ((nodes[i].used >> b) & 1) r.push_back(b);
        // filled up with the highest other bits
        for (int b = sh.T - 1; (int)r.size() < sh.R; --b)
            if (!((nodes[i].used >> b) & 1) && !((pairs[at] >> b) & 1)) r.push_back(b);
        std::sort(r.begin(), r.end());
        layouts[i] = g.layout(r, wave, nodes[i].memory);
        at = (size_t)(i ? from[i][at] : 0);
    }
    const Layout Lin = layouts.front(), Lout = layouts.back();

    // body first: it determines the tables and the number of gradient terms
    size_t node = 0;
    auto go_to = [&](size_t next) {
        const Layout &x = layouts[node], &y = layouts[next];
        if (!std::equal(x.reg, x.reg + sh.R, y.reg) || !std::equal(x.thr, x.thr + sh.T - sh.R, y.thr)) g.exchange(x, y);
        node = next;
    };
    for (size_t si = 0; si < stages.size(); ++si) {
        go_to(si + (load_is_stage ? 0 : 1));
        const std::vector<int>& r = regs[node];
        int rbit[32];
        for (int i = 0; i < sh.R; ++i) rbit[r[i]] = i;
        std::vector<StageOp> ops;
        auto add = [&](int li, bool grad) {
            int q[4], bits[4];
            const int nq = gate_qubits(lg[li], q);
            for (int i = 0; i < nq; ++i) bits[i] = rbit[q[i]];
            ops.push_back(stage_op(lg[li], p.gates[li], bits, grad));
        };
        const std::vector<int>& sg = stages[si].gates;
        if (dir == 0) {
            for (int li : sg) add(li, false);
        } else {
            for (size_t i = sg.size(); i-- > 0;) {
                if (lg[sg[i]].pidx >= 0) add(sg[i], true);
                add(sg[i], false);
            }
        }
        g.stage(std::move(ops));
        g.turn();
    }
    g.scale();
    go_to(nodes.size() - 1);
    g.flush();
    const std::string body = g.o.str();
    const int chunks = g.chunk;
    const std::vector<int> end = g.loc;  // variable of every register entry at the store
    g.o.str("");

    std::ostringstream& o = g.o;
    const int NV = g.NV;
    // in and out may be the same state: not __restrict__, or a pass of renames
    // alone could load an amplitude after its place was overwritten
    o << prelude(dbl) << "extern \"C\" __global__ void __launch_bounds__(" << kTileThreads << ", 2)\n"
      << tile_kernel_name(NV, dbl) << "(const TileArgs a, const T* __restrict__ tab, u32 cpt, u32 mlog, u32 gs, u32 L, "
         "const V* in0, V* out0, const V* in1, V* out1, "
         "double* __restrict__ gpart) {\n"
      << "  __shared__ __attribute__((aligned(16))) char lds[" << (g.elem_bytes() << sh.T) << "];\n"
      << "  const u32 tid = threadIdx.x;\n  u64 bit[" << sh.T << "];\n"
      << "#pragma unroll\n  for (int j = 0; j < " << sh.T << "; ++j) bit[j] = 1ull << a.pos[j];\n";
    g.thread_offset("off_in", Lin);
    g.thread_offset("off_out", Lout);
    for (int c = 0; c < chunks; ++c) o << "  double acc" << c << " = 0.0;\n";
    for (uint32_t w = 0; 32 * w < out.n_flags; ++w) o << "  const u32 half" << w << " = ((const u32*)tab)[" << w << "];\n";
    // Work order: blocks are dispatched round-robin over the 8 XCDs; XCD x
    // takes the eighth x of the cosets, and gs consecutive blocks of it walk a
    // contiguous run side by side (neighbouring cosets share pages).
    o << "  for (u32 it = 0; it < cpt; ++it) {\n"
      << "    u64 base;\n"
      << "    if (mlog < 3) base = (u64)blockIdx.x * cpt + it;\n"
      << "    else { const u32 bx = blockIdx.x >> 3; base = ((u64)(blockIdx.x & 7) << (mlog - 3)) + (u64)(bx / gs) * gs * cpt + "
         "(u64)it * gs + bx % gs; }\n"
      << "    if (base >= a.n_units) break;\n"
      << "    const bool origin = base == 0 && tid == 0;\n"
      << "#pragma unroll\n    for (int j = 0; j < " << sh.T
      << "; ++j) { const u64 low = base & (bit[j] - 1); base = ((base ^ low) << 1) | low; }\n";
    for (int i = 0; i < g.N; ++i) g.loc[i] = i;
    for (int v = 0; v < NV; ++v)
        for (int q = 0; q < g.N; ++q)
            o << "    T r" << v << "_" << q << " = 0, i" << v << "_" << q << " = 0;\n";
    if (NV == 1) o << "    if (a.first) { r0_0 = origin ? T(1) : T(0); } else\n";
    o << "    {\n";
    for (int q = 0; q < g.N; ++q)
        for (int v = 0; v < NV; ++v)
            o << "      const V l" << v << "_" << q << " = in" << v << "[base + off_in + (" << g.reg_offset(Lin, q) << ")];\n";
    for (int q = 0; q < g.N; ++q)
        for (int v = 0; v < NV; ++v)
            o << "      r" << v << "_" << q << " = l" << v << "_" << q << ".x; i" << v << "_" << q << " = l" << v << "_" << q
              << ".y;\n";
    o << "    }\n" << body;
    for (int q = 0; q < g.N; ++q)
        for (int v = 0; v < NV; ++v)
            o << "    out" << v << "[base + off_out + (" << g.reg_offset(Lout, q) << ")] = V{r" << v << "_" << end[q]
              << ", i" << v << "_" << end[q] << "};\n";
    // the next coset's first layout writes where other waves may still read, unless the wave bits agree
    if (!std::equal(Lin.thr + 6, Lin.thr + sh.T - sh.R, Lout.thr + 6)) o << "  __syncthreads();\n";
    o << "  }\n";
    if (chunks) {
        o << "  __syncthreads();\n  double* red = (double*)lds;\n";
        for (int c = 0; c < chunks; ++c) o << "  red[(tid >> 6) * " << 64 * chunks << " + " << 64 * c << " + (tid & 63)] = acc" << c << ";\n";
        o << "  __syncthreads();\n  if (tid < " << 64 * chunks << ") {\n    double r = red[tid];\n"
          << "    for (int w = 1; w < " << kTileThreads / 64 << "; ++w) r += red[w * " << 64 * chunks << " + tid];\n"
          << "    gpart[(u64)blockIdx.x * L + tid] = r;\n  }\n";
    }
    o << "}\n";
    out.src = o.str();
    return true;
}

double turn_limit(bool dbl, double norm) {
    const double room = (dbl ? 1000.0 : 120.0) - std::log2(std::max(norm, 1.0));
    return std::max(1.0, std::exp2(std::floor(room / max_pending(dbl))));
}

template <typename T>
void fill_tile_table(const TileKernel& k, const std::vector<Gate>& gates, const HalfAngle* h, double limit, int dir,
                     T* tab) {
    const double sign = dir ? -1.0 : 1.0;
    double f, t;
    if (k.n_flags) std::memset(tab, 0, kTileFlagBytes);
    for (const TileEntry& e : k.entries) {
        T* m = tab + e.off;
        double s = 1.0;
        for (int g : e.rots) {
            rot_numbers(h[g], sign, limit, f, t);
            s *= f;
        }
        switch (e.kind) {
            case TF_ROT: {
                const bool half = rot_numbers(h[e.gate], sign, limit, f, t);
                m[0] = (T)t;
                if (half) {
                    ((uint32_t*)tab)[e.flag_word] |= 1u << e.flag_bit;
                    ((uint32_t*)tab)[e.any_word] |= e.any;
                }
                break;
            }
            case TF_SCALE:
                m[0] = (T)s;
                break;
            case TF_PHASE: {
                // one bit after the other: RZ multiplies by e^{-i th/2} (bit clear) or e^{i th/2} (set)
                double re[32] = {s}, im[32] = {0.0};
                int n = 1;
                for (int b = 0; b < 8; ++b) {
                    if (!((e.mask >> b) & 1)) continue;
                    double zr = 1.0, zi = 0.0;
                    for (size_t d = 0; d < e.diag.size(); ++d) {
                        if (gates[e.diag[d]].kind == VQE_GATE_CZ || e.diag_bits[d] != 1u << b) continue;
                        const double gr = h[e.diag[d]].c, gi = sign * h[e.diag[d]].s, r = zr * gr - zi * gi;
                        zi = zr * gi + zi * gr;
                        zr = r;
                    }
                    for (int i = 0; i < n; ++i) {
                        re[i + n] = re[i] * zr - im[i] * zi;
                        im[i + n] = re[i] * zi + im[i] * zr;
                        const double r = re[i] * zr + im[i] * zi;
                        im[i] = im[i] * zr - re[i] * zi;
                        re[i] = r;
                    }
                    n *= 2;
                }
                for (size_t d = 0; d < e.diag.size(); ++d) {
                    if (gates[e.diag[d]].kind != VQE_GATE_CZ) continue;
                    uint32_t idx = 0;  // the CZ's bits among the table's
                    for (int b = 0, at = 0; b < 8; ++b)
                        if ((e.mask >> b) & 1) idx |= ((e.diag_bits[d] >> b) & 1u) << at++;
                    for (int i = 0; i < n; ++i)
                        if (((uint32_t)i & idx) == idx) {
                            re[i] = -re[i];
                            im[i] = -im[i];
                        }
                }
                for (int i = 0; i < n; ++i) {
                    m[2 * i] = (T)re[i];
                    m[2 * i + 1] = (T)im[i];
                }
                break;
            }
            case TF_R2:
                if (gates[e.gate].kind == VQE_GATE_H) {
                    const double r = 1.0 / std::sqrt(2.0);
                    m[0] = m[1] = m[2] = (T)r;
                    m[3] = (T)-r;
                } else {  // excitations: [[c, -s], [s, c]]
                    m[0] = m[3] = (T)h[e.gate].c;
                    m[1] = (T)(-sign * h[e.gate].s);
                    m[2] = (T)(sign * h[e.gate].s);
                }
                break;
        }
    }
}

template void fill_tile_table<float>(const TileKernel&, const std::vector<Gate>&, const HalfAngle*, double, int, float*);
template void fill_tile_table<double>(const TileKernel&, const std::vector<Gate>&, const HalfAngle*, double, int, double*);

}  // namespace vqe

// Batched evaluations of many independent requests, by an interpreter of batch
// programs (program.cpp).
//
// Small states: one workgroup evaluates one request (energy and adjoint
// gradient of psi(theta) = U(theta)|0...0>, eqs. 6-7) with the whole state held
// in LDS: psi and lam = H psi (2 x 2^n amplitudes, n <= 13 for complex64, n <= 12
// for complex128), so a request touches HBM only for its program, tables and
// results.  Mid-size states: psi and lam stay in device memory and one launch
// applies one pass, a window of kMidWin qubits, of every item; a block stages a
// coset in LDS and runs the pass's program there.
//
// A program is a list of stages.  A stage keeps 4 bits of the tile's index in
// registers: each of the 2^(bits - 4) threads reads its 16 amplitudes (of lam
// too in reverse), runs the stage's ops on them with every register index a
// constant, and writes them back; one barrier per stage instead of one per
// gate.  A stage's ops and numbers come as one block, read from memory while the
// stage before runs and kept in LDS (scalar loads of tables just written by a
// copy miss every cache, about 0.7 us per line).  Gradient terms are summed over
// the wave as they appear, up to four together; every wave keeps its own sum per
// slot, added in wave order at the end.  The thread -> amplitude map and every
// order of summation depend only on the item, so a request's bits do not depend
// on the rest of its batch.
//
// What bounds it: the vector instructions and the latency of the stages of one
// request, which uses one CU at one wave per SIMD (complex64: two at 13 qubits);
// vector instructions issue in 45 % of the kernel's cycles (complex128 35 %).  A
// gate per barrier with the state read and written in LDS for each took, per call:
// 12 qubits x 4 layers complex64 388 us, now 130 (106 in the kernel); 24 requests
// of 8 to 13 qubits 1745 us, now 609; 4 states of 14 to 16 qubits (10-qubit windows
// before) 1160 us, now 683; 12 qubits, excitations, complex128 439 us, now 215.
// Rows without a branch beat a switch per op (156 against 240 us at 12 qubits:
// the arms of a switch cost copies of the 64 registers of psi and lam); rows of
// CNOTs alone leave early (136).
#include <type_traits>

#include "vqe_internal.h"

namespace vqe {
namespace {

template <typename T> struct VecB;
template <> struct VecB<float> { using type = float2; static constexpr int kBank = 4; };
template <> struct VecB<double> { using type = double2; static constexpr int kBank = 3; };

constexpr int kN = 1 << kProgBits;  // amplitudes per thread and vector

// LDS slot of tile index j: the lowest kBank bits (the amplitudes that LDS
// serves per clock) XORed with the groups of bits above, so that amplitudes a
// power of two apart lie in different banks.  Linear over GF(2).
template <typename T>
__device__ __forceinline__ uint32_t slot_of(uint32_t j) {
    constexpr int nb = VecB<T>::kBank;
    const uint32_t f = (j >> nb) ^ (j >> (2 * nb)) ^ (j >> (3 * nb)) ^ (j >> (4 * nb));
    return j ^ (f & ((1u << nb) - 1));
}

__device__ __forceinline__ uint32_t ins0(uint32_t k, uint32_t q) {
    const uint32_t low = k & ((1u << q) - 1);
    return ((k ^ low) << 1) | low;
}

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// Sum over the 64 lanes of a wave in a fixed order, in every lane: swaps of
// the halves and rows, then DPP (row_ror:8, row_half_mirror, quad permutes).
template <int C>
__device__ __forceinline__ double dpp_add(double v) {
    const unsigned long long x = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)x, C, 0xF, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), C, 0xF, 0xF, false);
    return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum(double v) {
    unsigned long long x = __double_as_longlong(v);
    auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
    v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
        __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    x = __double_as_longlong(v);
    l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
    v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
        __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    v = dpp_add<0x128>(v);
    v = dpp_add<0x141>(v);
    v = dpp_add<0x4E>(v);
    return dpp_add<0xB1>(v);
}

// Sums of up to four values over the wave: value k ends in every lane of row k
// (lanes 16 k .. 16 k + 15).  Two exchanges of halves and rows take the four to
// one value per lane, the rest of the sum is that of one value.
__device__ __forceinline__ double row_sums(const double (&g)[4]) {
    auto swap = [](double a, double b, auto f) {
        const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
        const auto l = f((unsigned)x, (unsigned)y);
        const auto h = f((unsigned)(x >> 32), (unsigned)(y >> 32));
        return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
               __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    };
    auto s32 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); };
    auto s16 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); };
    // lanes below 32: values 0 and 1, above: 2 and 3
    double v = swap(swap(g[0], g[2], s32), swap(g[1], g[3], s32), s16);
    v = dpp_add<0x128>(v);
    v = dpp_add<0x141>(v);
    v = dpp_add<0x4E>(v);
    return dpp_add<0xB1>(v);
}

// ------------------------------------------------------------------ ops on 16 register entries
__device__ __forceinline__ void swap_regs(float& a, float& b) { asm("v_swap_b32 %0, %1" : "+v"(a), "+v"(b)); }
__device__ __forceinline__ void swap_regs(double& a, double& b) {
    unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32), yl = (unsigned)y, yh = (unsigned)(y >> 32);
    asm("v_swap_b32 %0, %1" : "+v"(xl), "+v"(yl));
    asm("v_swap_b32 %0, %1" : "+v"(xh), "+v"(yh));
    a = __longlong_as_double((long long)(((unsigned long long)xh << 32) | xl));
    b = __longlong_as_double((long long)(((unsigned long long)yh << 32) | yl));
}

// RY by half a turn, (x, y) -> (-y, x); X: RX, (-i y, -i x).  Only rotations
// beyond turn_limit() take it.
template <int B, bool X, int NV, typename T>
__device__ __forceinline__ void half_turn(T (&re)[NV][kN], T (&im)[NV][kN]) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if (p & (1 << B)) continue;
            const int q = p | (1 << B);
            swap_regs(re[v][p], X ? im[v][q] : re[v][q]);
            swap_regs(im[v][p], X ? re[v][q] : im[v][q]);
            im[v][p] = -im[v][p];
            if (X) im[v][q] = -im[v][q];
            else re[v][p] = -re[v][p];
        }
}

template <int B, int NV, typename T>
__device__ __forceinline__ void rot_y(T (&re)[NV][kN], T (&im)[NV][kN], T t) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if (p & (1 << B)) continue;
            const int q = p | (1 << B);
            const T xr = re[v][p], xi = im[v][p], yr = re[v][q], yi = im[v][q];
            re[v][p] = xr - t * yr;
            im[v][p] = xi - t * yi;
            re[v][q] = yr + t * xr;
            im[v][q] = yi + t * xi;
        }
}

// x - i t y, y - i t x; half: after a half turn
template <int B, int NV, typename T>
__device__ __forceinline__ void rot_x(T (&re)[NV][kN], T (&im)[NV][kN], T t, bool half) {
    if (__builtin_expect(half, 0)) half_turn<B, true, NV, T>(re, im);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if (p & (1 << B)) continue;
            const int q = p | (1 << B);
            const T xr = re[v][p], xi = im[v][p], yr = re[v][q], yi = im[v][q];
            re[v][p] = xr + t * yi;
            im[v][p] = xi - t * yr;
            re[v][q] = yr + t * xi;
            im[v][q] = yi - t * xr;
        }
}

template <int B, int NV, typename T>
__device__ __forceinline__ void mat_r2(T (&re)[NV][kN], T (&im)[NV][kN], T ca, T cb, T cc, T cd) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if (p & (1 << B)) continue;
            const int q = p | (1 << B);
            const T ar = re[v][p], ai = im[v][p], br = re[v][q], bi = im[v][q];
            re[v][p] = ca * ar + cb * br;
            im[v][p] = ca * ai + cb * bi;
            re[v][q] = cc * ar + cd * br;
            im[v][q] = cc * ai + cd * bi;
        }
}

// Swaps the entries with target bit Tg clear and set where bit C is set (C = Tg: all).
template <int C, int Tg, int NV, typename T>
__device__ __forceinline__ void flip(T (&re)[NV][kN], T (&im)[NV][kN]) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if ((p & (1 << Tg)) || (C != Tg && !(p & (1 << C)))) continue;
            swap_regs(re[v][p], re[v][p | (1 << Tg)]);
            swap_regs(im[v][p], im[v][p | (1 << Tg)]);
        }
}

// CNOT or X of code control << 2 | target (equal: X).
template <int NV, typename T>
__device__ __forceinline__ void permute(uint32_t code, T (&re)[NV][kN], T (&im)[NV][kN]) {
    switch (code) {
#define VQE_PERM(C, G) case 4 * C + G: flip<C, G, NV, T>(re, im); break;
        VQE_PERM(0, 0) VQE_PERM(0, 1) VQE_PERM(0, 2) VQE_PERM(0, 3)
        VQE_PERM(1, 0) VQE_PERM(1, 1) VQE_PERM(1, 2) VQE_PERM(1, 3)
        VQE_PERM(2, 0) VQE_PERM(2, 1) VQE_PERM(2, 2) VQE_PERM(2, 3)
        VQE_PERM(3, 0) VQE_PERM(3, 1) VQE_PERM(3, 2)
        default: flip<3, 3, NV, T>(re, im); break;
#undef VQE_PERM
    }
}

// CNOT of control C, target C + 1 if `on`, without a branch.
template <int C, int NV, typename T>
__device__ __forceinline__ void cnot_if(bool on, T (&re)[NV][kN], T (&im)[NV][kN]) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            if (!(p & (1 << C)) || (p & (2 << C))) continue;
            const int q = p | (2 << C);
            const T xr = re[v][p], xi = im[v][p], yr = re[v][q], yi = im[v][q];
            re[v][p] = on ? yr : xr;
            im[v][p] = on ? yi : xi;
            re[v][q] = on ? xr : yr;
            im[v][q] = on ? xi : yi;
        }
}

// Im<lam|Y_B|psi> (Y) or Im<lam|X_B|psi> over the thread's entries, the terms
// of its pairs summed in 64 bits: eight of them in 32 lost bits of terms that
// cancel (24 requests of 8 to 13 qubits, complex64: 617 us per call against 600).
template <int B, bool Y, typename T>
__device__ __forceinline__ double grad_xy(const T (&re)[2][kN], const T (&im)[2][kN]) {
    double acc = 0;
#pragma unroll
    for (int p = 0; p < kN; ++p) {
        if (p & (1 << B)) continue;
        const int q = p | (1 << B);
        if (Y)
            acc += (double)((re[1][q] * re[0][p] + im[1][q] * im[0][p]) - (re[1][p] * re[0][q] + im[1][p] * im[0][q]));
        else
            acc += (double)((re[1][p] * im[0][q] - im[1][p] * re[0][q]) + (re[1][q] * im[0][p] - im[1][q] * re[0][p]));
    }
    return acc;
}

#define VQE_BITS(CALL)                            \
    case 0: { constexpr int B = 0; CALL; } break; \
    case 1: { constexpr int B = 1; CALL; } break; \
    case 2: { constexpr int B = 2; CALL; } break; \
    default: { constexpr int B = 3; CALL; } break;

// A stage's block on its way from memory to LDS: fetch() issues the loads,
// store() writes what arrived.  NT threads.
template <int NT>
struct BlockFetch {
    static constexpr int kPer = (int)((kProgBlock / 16 + NT - 1) / NT);
    using W = uint32_t __attribute__((ext_vector_type(4)));
    W v[kPer];
    __device__ __forceinline__ void fetch(const char* src, uint32_t bytes, uint32_t t, uint32_t nt) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            if (q * nt * 16 >= bytes) break;
            if ((q * nt + t) * 16 < bytes) v[q] = *(const W*)(src + (q * nt + t) * 16);
        }
    }
    __device__ __forceinline__ void store(char* dst, uint32_t bytes, uint32_t t, uint32_t nt) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            if (q * nt * 16 >= bytes) break;
            if ((q * nt + t) * 16 < bytes) *(W*)(dst + (q * nt + t) * 16) = v[q];
        }
    }
};

// The stages [0, n_stages) of a program on a tile of 2^bits amplitudes in LDS
// (lam too for NV = 2), by nt = 2^(bits - 4) threads (at least NTMIN); blk: two
// blocks of kProgBlock bytes in LDS.  Starts and ends with a barrier.
// emit(slot, v): v = the sum over the calling lane's row of lanes, called by one
// lane per slot and wave.
template <typename T, int NV, int NTMIN, typename Emit>
__device__ __forceinline__ void run_program(char* psi, char* lam, char* blk, uint32_t bits, uint32_t t, uint32_t nt,
                                            const ProgStage* __restrict__ stages, uint32_t n_stages,
                                            const char* __restrict__ stream, Emit emit) {
    using V = typename VecB<T>::type;
    constexpr uint32_t A = sizeof(V);
    const uint32_t lane = t & 63;
    BlockFetch<NTMIN> f;
    // The same in every lane, and known to be: a loop or branch on values that
    // the compiler takes for per-lane ones costs copies of all registers.
    struct Stage {
        uint32_t pos, kind, n_ops, off, bytes;
    };
    auto stage_at = [](const void* at) {
        const uint32_t* w = (const uint32_t*)at;
        const uint32_t w1 = uni(w[1]);
        return Stage{uni(w[0]), w1 & 0xffffu, w1 >> 16, uni(w[2]),
                     uni(w[3])};
    };
    n_stages = uni(n_stages);
    bits = uni(bits);
    nt = uni(nt);
    Stage st{};
    if (n_stages) {
        st = stage_at(stages);
        f.fetch(stream + st.off, st.bytes, t, nt);
        f.store(blk, st.bytes, t, nt);
    }
    __syncthreads();
    for (uint32_t si = 0; si < n_stages; ++si) {
        const char* cur = blk + (si & 1) * kProgBlock;
        Stage nx{};
        if (si + 1 < n_stages) {
            nx = stage_at(cur);  // a block starts with the next stage's header
            f.fetch(stream + nx.off, nx.bytes, t, nt);
        }
        if (st.kind == PK_PAIRS) {
            // excitations: pairs (i | A, i | B) over the other bits of i
            for (uint32_t o = 0; o < st.n_ops; ++o) {
                const ProgPair<T>& op = *(const ProgPair<T>*)(cur + 16 + o * sizeof(ProgPair<T>));
                const uint32_t x = uni(op.x), pa = x & 0xffffu, pb = x >> 16;
                const bool grad = NV == 2 && uni(op.grad);
                const T ca = op.s[0], cb = op.s[1], cc = op.s[2], cd = op.s[3];
                const uint32_t sa = slot_of<T>(pa) * A, sb = slot_of<T>(pb) * A;
                double acc = 0;
                for (uint32_t i = t; i < (1u << (bits - __popc(pa | pb))); i += nt) {
                    uint32_t j = i;
                    for (uint32_t m = pa | pb; m; m &= m - 1) j = ins0(j, (uint32_t)__builtin_ctz(m));
                    const uint32_t at = slot_of<T>(j) * A, ia = at ^ sa, ib = at ^ sb;
                    V xa[NV], xb[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        xa[v] = *(const V*)((v ? lam : psi) + ia);
                        xb[v] = *(const V*)((v ? lam : psi) + ib);
                    }
                    if (grad)
                        acc += (double)((xb[NV - 1].x * xa[0].x + xb[NV - 1].y * xa[0].y) -
                                        (xa[NV - 1].x * xb[0].x + xa[NV - 1].y * xb[0].y));
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        V na, nb;
                        na.x = ca * xa[v].x + cb * xb[v].x;
                        na.y = ca * xa[v].y + cb * xb[v].y;
                        nb.x = cc * xa[v].x + cd * xb[v].x;
                        nb.y = cc * xa[v].y + cd * xb[v].y;
                        *(V*)((v ? lam : psi) + ia) = na;
                        *(V*)((v ? lam : psi) + ib) = nb;
                    }
                }
                if (grad) {
                    const double g = wave_sum(acc);
                    if (lane == 0) emit(op.slot, g);
                }
                if (o + 1 < st.n_ops) __syncthreads();
            }
        } else {
            uint32_t j = t, s[kProgBits];
#pragma unroll
            for (int k = 0; k < kProgBits; ++k) {
                const uint32_t q = (st.pos >> (8 * k)) & 255u;
                j = ins0(j, q);
                s[k] = slot_of<T>(1u << q) * A;
            }
            const uint32_t b = slot_of<T>(j) * A;
            auto at = [&](int p) {
                return b ^ ((p & 1) ? s[0] : 0) ^ ((p & 2) ? s[1] : 0) ^ ((p & 4) ? s[2] : 0) ^ ((p & 8) ? s[3] : 0);
            };
            auto load = [&](T (&re)[NV][kN], T (&im)[NV][kN]) {
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int p = 0; p < kN; ++p) {
                        const V x = *(const V*)((v ? lam : psi) + at(p));
                        re[v][p] = x.x;
                        im[v][p] = x.y;
                    }
            };
            auto save = [&](const T (&re)[NV][kN], const T (&im)[NV][kN]) {
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int p = 0; p < kN; ++p) {
                        V x;
                        x.x = re[v][p];
                        x.y = im[v][p];
                        *(V*)((v ? lam : psi) + at(p)) = x;
                    }
            };
            // sums over the wave of the terms g of the bits in mask, to their slots
            auto emit4 = [&](const double (&g)[4], uint32_t mask, uint32_t slot, uint32_t off) {
                const double r = row_sums(g);
                const uint32_t row = lane >> 4;
                if ((lane & 15) == 0 && ((mask >> row) & 1)) emit(slot + ((off >> (8 * row)) & 255u), r);
            };
            if (st.kind == PK_ROWS) {
                // HALF: with the half turns that the rows' flags ask for; a loop of its own, as a branch
                // in the other costs it registers (12 qubits, complex128: 201 us per call, 188 with two loops)
                auto rows = [&](auto HALF) {
                    T re[NV][kN], im[NV][kN];
                    load(re, im);
                    for (uint32_t i = 0; i < st.n_ops; ++i) {
                        const ProgRow<T>& o = *(const ProgRow<T>*)(cur + 16 + i * sizeof(ProgRow<T>));
                        const uint32_t fl = uni(o.flags);
                        auto turns = [&] {
                            if constexpr (decltype(HALF)::value) {
                                if (fl & 0x10000u) half_turn<0, false, NV, T>(re, im);
                                if (fl & 0x20000u) half_turn<1, false, NV, T>(re, im);
                                if (fl & 0x40000u) half_turn<2, false, NV, T>(re, im);
                                if (fl & 0x80000u) half_turn<3, false, NV, T>(re, im);
                            }
                            rot_y<0, NV, T>(re, im, o.t[0]);
                            rot_y<1, NV, T>(re, im, o.t[1]);
                            rot_y<2, NV, T>(re, im, o.t[2]);
                            rot_y<3, NV, T>(re, im, o.t[3]);
                        };
                        auto phases = [&] {
#pragma unroll
                            for (int p = 0; p < kN; ++p) {
                                const T pr = o.ph[2 * p], pi = o.ph[2 * p + 1];
#pragma unroll
                                for (int v = 0; v < NV; ++v) {
                                    const T ar = re[v][p], ai = im[v][p];
                                    re[v][p] = pr * ar - pi * ai;
                                    im[v][p] = pr * ai + pi * ar;
                                }
                            }
                        };
                        if constexpr (NV == 1) {
                            turns();
                            phases();
                            cnot_if<0, NV, T>(fl & 1, re, im);
                            cnot_if<1, NV, T>(fl & 2, re, im);
                            cnot_if<2, NV, T>(fl & 4, re, im);
                        } else {
                            cnot_if<2, NV, T>(fl & 4, re, im);
                            cnot_if<1, NV, T>(fl & 2, re, im);
                            cnot_if<0, NV, T>(fl & 1, re, im);
                            if (!(fl & 16)) continue;  // CNOTs alone
                            phases();
                            // Z: d = Im(conj(lam) psi) once; per bit the sum of differences, the sums passed on
                            double gz[4];
                            {
                                double d[kN];
#pragma unroll
                                for (int p = 0; p < kN; ++p) d[p] = (double)(re[1][p] * im[0][p] - im[1][p] * re[0][p]);
#pragma unroll
                                for (int q = 0; q < kProgBits; ++q) {
                                    double acc = 0;
#pragma unroll
                                    for (int p = 0; p < (kN >> (q + 1)); ++p) {
                                        acc += d[2 * p] - d[2 * p + 1];
                                        d[p] = d[2 * p] + d[2 * p + 1];
                                    }
                                    gz[q] = acc;
                                }
                            }
                            const double gy[4] = {grad_xy<0, true, T>(re, im), grad_xy<1, true, T>(re, im),
                                                  grad_xy<2, true, T>(re, im), grad_xy<3, true, T>(re, im)};
                            turns();
                            emit4(gz, (fl >> 8) & 15u, o.z_slot, o.z_off);
                            emit4(gy, (fl >> 12) & 15u, o.y_slot, o.y_off);
                        }
                    }
                    save(re, im);
                };
                if (__builtin_expect(uni(((const ProgRow<T>*)(cur + 16))->flags) & kRowHalf, 0)) rows(std::true_type{});
                else rows(std::false_type{});
            } else {
                T re[NV][kN], im[NV][kN];
                load(re, im);
                for (uint32_t i = 0; i < st.n_ops; ++i) {
                    const ProgMisc<T>& o = *(const ProgMisc<T>*)(cur + 16 + i * sizeof(ProgMisc<T>));
                    const uint32_t code = uni(o.code), a = (code >> 8) & 0xffu;
                    switch (code & 255u) {
                        case PM_ROTX:
                            switch (a) { VQE_BITS((rot_x<B, NV, T>(re, im, o.t[0], code >> 31))) }
                            break;
                        case PM_R2:
                            switch (a) { VQE_BITS((mat_r2<B, NV, T>(re, im, o.t[0], o.t[1], o.t[2], o.t[3]))) }
                            break;
                        case PM_PERM:
                            permute<NV, T>(a, re, im);
                            break;
                        default:  // PM_GX
                            if constexpr (NV == 2) {
                                double v = 0;
                                switch (a) { VQE_BITS((v = grad_xy<B, false, T>(re, im))) }
                                const double g[4] = {v, 0.0, 0.0, 0.0};
                                emit4(g, 1, o.slot, 0);
                            }
                            break;
                    }
                }
                save(re, im);
            }
        }
        if (si + 1 < n_stages) f.store(blk + ((si + 1) & 1) * kProgBlock, nx.bytes, t, nt);
        st = nx;
        __syncthreads();
    }
}

// ------------------------------------------------------------------ small states
template <typename T> constexpr int small_threads() { return 1 << ((sizeof(T) == 4 ? kBatchMaxQubitsC64 : kBatchMaxQubitsC128) - kProgBits); }

// v with its sign bit xor the highest bit of s.
__device__ __forceinline__ float flip_sign(float v, uint32_t s) { return __uint_as_float(__float_as_uint(v) ^ s); }
__device__ __forceinline__ double flip_sign(double v, uint32_t s) {
    return __hiloint2double((int)((uint32_t)__double2hiint(v) ^ s), __double2loint(v));
}

// lam = H psi for the thread's amplitudes b = t + p 2^(bits - 4): the terms of a
// group go to one bucket per z pattern of the register bits, signed by the
// thread part of their z bits, and D_x for the 16 patterns is the
// Walsh-Hadamard transform of the bucket sums; the terms of small groups are
// added to the 16 directly (12 qubits complex64, 500 groups of 1, 2 and 4 terms:
// 287, 371 and 547 us per call, 575, 601 and 654 with buckets for all).  The tables come block by block
// as a program's do.
template <typename T, bool REAL>
__device__ __forceinline__ void small_hpsi(const BatchDesc<T>& d, const char* psi, char* blk, uint32_t t, uint32_t nt,
                                           T (&lr)[kN], T (&li)[kN]) {
    using V = typename VecB<T>::type;
    constexpr uint32_t A = sizeof(V);
    const uint32_t sh = (uint32_t)d.bits - kProgBits, n_blocks = uni(d.n_blocks);
    const uint32_t b = slot_of<T>(t) * A;
    // largest group summed term by term: 500 groups of four terms, directly and by
    // buckets: complex64 10 qubits 534 and 566 us, 12 qubits 547 and 589, 13 qubits
    // (two waves per SIMD) 681 and 648; complex128 10 qubits 691 and 633
    const uint32_t direct = sizeof(T) == 4 && nt <= 256 ? 4 : 3;
#pragma unroll
    for (int p = 0; p < kN; ++p) lr[p] = li[p] = 0;
    for (uint32_t k = 0; k < n_blocks; ++k) {
        const SmallBlock bk = d.ham[k];
        char* buf = blk + (k & 1) * kProgBlock;  // the block before may still be in use
        {
            BlockFetch<64> f;
            f.fetch(d.ham_stream + uni(bk.off), uni(bk.bytes), t, nt);
            f.store(buf, uni(bk.bytes), t, nt);
        }
        __syncthreads();
        const char *at = buf, *nx = buf;
        SmallGroup head = *(const SmallGroup*)at;
        SmallTerm<T> term = *(const SmallTerm<T>*)(at + sizeof(SmallGroup));
        for (uint32_t g = uni(bk.n_groups); g; --g, at = nx) {
            const uint32_t gx = uni(head.x), n_terms = uni(head.n_terms);
            const SmallGroup G = head;
            const SmallTerm<T> first = term;
            const SmallTerm<T>* tm = (const SmallTerm<T>*)(at + sizeof(SmallGroup));
            // what can be on its way while this group is worked on: its amplitudes, the next header and term
            V x[kN];
            const uint32_t from = b ^ (slot_of<T>(gx) * A);
#pragma unroll
            for (int p = 0; p < kN; ++p) x[p] = *(const V*)(psi + (from ^ (slot_of<T>((uint32_t)p << sh) * A)));
            nx = at + sizeof(SmallGroup) + n_terms * sizeof(SmallTerm<T>);
            head = *(const SmallGroup*)(g > 1 ? nx : at);
            term = *(const SmallTerm<T>*)((g > 1 ? nx : at) + sizeof(SmallGroup));
            T er[kN], ei[kN];
            if (n_terms <= direct) {
                // a term is the same in all 16 patterns but for the signs of its register bits
                auto signs = [&](const SmallTerm<T>& c, T (&sr)[kN], T (&si)[kN]) {
                    const uint32_t neg = (uint32_t)__popc(c.zt & t) << 31, zr = uni(c.zr);
                    sr[0] = flip_sign(c.cre, neg);
                    if (!REAL) si[0] = flip_sign(c.cim, neg);
#pragma unroll
                    for (int q = 0; q < kProgBits; ++q) {
                        const uint32_t nq = (zr >> q) << 31;
#pragma unroll
                        for (int p = 0; p < (1 << q); ++p) {
                            sr[p | (1 << q)] = flip_sign(sr[p], nq);
                            if (!REAL) si[p | (1 << q)] = flip_sign(si[p], nq);
                        }
                    }
                };
                signs(first, er, ei);
                for (uint32_t k = 1; k < n_terms; ++k) {
                    T sr[kN], si[kN];
                    signs(tm[k], sr, si);
#pragma unroll
                    for (int p = 0; p < kN; ++p) {
                        er[p] += sr[p];
                        if (!REAL) ei[p] += si[p];
                    }
                }
            } else {
                const uint32_t w[4] = {uni(G.count[0]), uni(G.count[1]), uni(G.count[2]), uni(G.count[3])};
#pragma unroll
                for (int u = 0; u < kN; ++u) {
                    er[u] = ei[u] = 0;
                    for (uint32_t c = (w[u >> 2] >> (8 * (u & 3))) & 255u; c; --c, ++tm) {
                        const bool neg = __popc(tm->zt & t) & 1;
                        er[u] += neg ? -tm->cre : tm->cre;
                        if (!REAL) ei[u] += neg ? -tm->cim : tm->cim;
                    }
                }
#pragma unroll
                for (int bit = 1; bit < kN; bit <<= 1)
#pragma unroll
                    for (int i = 0; i < kN; ++i) {
                        if (i & bit) continue;
                        const T y = er[i], v = er[i | bit];
                        er[i] = y + v;
                        er[i | bit] = y - v;
                        if (!REAL) {
                            const T yi = ei[i], vi = ei[i | bit];
                            ei[i] = yi + vi;
                            ei[i | bit] = yi - vi;
                        }
                    }
            }
#pragma unroll
            for (int p = 0; p < kN; ++p) {
                lr[p] += er[p] * x[p].x;
                li[p] += er[p] * x[p].y;
                if (!REAL) {
                    lr[p] -= ei[p] * x[p].y;
                    li[p] += ei[p] * x[p].x;
                }
            }
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(small_threads<T>())
batch_kernel(const BatchDesc<T>* __restrict__ items) {
    using V = typename VecB<T>::type;
    constexpr uint32_t A = sizeof(V);
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2][8];
    const BatchDesc<T>& d = items[blockIdx.x];
    const uint32_t dim = 1u << d.bits, nt = dim >> kProgBits, waves = nt >> 6;
    const uint32_t t = threadIdx.x;
    if (t >= nt) return;  // whole waves that the item has no amplitudes for
    char* blk = reinterpret_cast<char*>(smem);
    char* psi = blk + 2 * kProgBlock;
    char* lam = psi + dim * A;
    const uint32_t wave = t >> 6, lane = t & 63;
#pragma unroll
    for (int p = 0; p < kN; ++p) {
        const uint32_t i = t + p * nt;
        V v;
        v.x = i == 0 ? T(1) : T(0);
        v.y = 0;
        *(V*)(psi + slot_of<T>(i) * A) = v;
    }
    for (uint32_t k = 0, s = 0; k <= d.n_ckpt; ++k) {
        const uint32_t end = k < d.n_ckpt ? d.ckpt[k].fwd_end : d.n_fwd;
        run_program<T, 1, 64>(psi, nullptr, blk, (uint32_t)d.bits, t, nt, d.fwd + s, end - s, d.fwd_stream,
                              [](uint32_t, double) {});
        s = end;
        if (k == d.n_ckpt) break;
        for (uint32_t i = t; i < (1u << d.n); i += nt) ((V*)d.ckpt[k].buf)[i] = *(const V*)(psi + slot_of<T>(i) * A);
        __syncthreads();
    }
    // lam = H psi, energy and norm
    double e = 0.0, nn = 0.0;
    {
        T lr[kN], li[kN];
        if (d.real) small_hpsi<T, true>(d, psi, blk, t, nt, lr, li);
        else small_hpsi<T, false>(d, psi, blk, t, nt, lr, li);
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            const uint32_t at = slot_of<T>(t + p * nt) * A;
            const V x = *(const V*)(psi + at);
            V l;
            l.x = lr[p];
            l.y = li[p];
            *(V*)(lam + at) = l;
            e += (double)(x.x * lr[p] + x.y * li[p]);
            nn += (double)(x.x * x.x + x.y * x.y);
        }
    }
    e = wave_sum(e);
    nn = wave_sum(nn);
    if (lane == 0) {
        red[0][wave] = e;
        red[1][wave] = nn;
    }
    __syncthreads();
    double E = red[0][0], nrm = red[1][0];
    for (uint32_t w = 1; w < waves; ++w) {
        E += red[0][w];
        nrm += red[1][w];
    }
    if (t == 0) {
        d.out[0] = E / nrm;
        d.out[1] = nrm;
    }
    double* part = d.part;
    for (uint32_t k = d.n_ckpt, s = 0;; --k) {
        const uint32_t end = k > 0 ? d.ckpt[k - 1].rev_end : d.n_rev;
        run_program<T, 2, 64>(psi, lam, blk, (uint32_t)d.bits, t, nt, d.rev + s, end - s, d.rev_stream,
                              [=](uint32_t sl, double v) { part[8 * sl + wave] = v; });
        s = end;
        if (k == 0) break;
        for (uint32_t i = t; i < (1u << d.n); i += nt) *(V*)(psi + slot_of<T>(i) * A) = ((const V*)d.ckpt[k - 1].buf)[i];
        __syncthreads();
    }
    __threadfence_block();
    __syncthreads();
    for (uint32_t k = t; k < d.n_slots; k += nt) {
        double g = part[8 * k];
        for (uint32_t w = 1; w < waves; ++w) g += part[8 * k + w];
        d.out[2 + k] = g / nrm;
    }
    if (d.psi_out) {
        for (uint32_t i = t; i < (1u << d.n); i += nt) {
            ((V*)d.psi_out)[i] = *(const V*)(psi + slot_of<T>(i) * A);
            ((V*)d.lam_out)[i] = *(const V*)(lam + slot_of<T>(i) * A);
        }
    }
}

// ------------------------------------------------------------------ mid-size items
constexpr int kMT = 1 << (kMidWin - kProgBits);  // threads per block

// Index of the descriptor that owns block b: the last one with blk_begin <= b.
template <typename D>
__device__ uint32_t owner(const D* d, uint32_t n, uint32_t b) {
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (d[m].blk_begin <= b) lo = m;
        else hi = m;
    }
    return lo;
}

template <typename T, bool REV>
__global__ void __launch_bounds__(kMT)
mid_pass_kernel(const MidPass* __restrict__ descs, uint32_t n_desc, double* __restrict__ part) {
    using V = typename VecB<T>::type;
    constexpr uint32_t A = sizeof(V);
    __shared__ __align__(16) char sp[A << kMidWin];
    __shared__ __align__(16) char sl[REV ? A << kMidWin : 16];
    __shared__ __align__(16) char blks[2 * kProgBlock];
    __shared__ double acc[REV ? kMidMaxSlots * (kMT / 64) : 1];
    const MidPass& d = descs[owner(descs, n_desc, blockIdx.x)];
    const uint32_t blk = blockIdx.x - d.blk_begin;
    const uint32_t t = threadIdx.x, wave = t >> 6;
    V* psi = reinterpret_cast<V*>(d.psi);
    V* lam = reinterpret_cast<V*>(d.lam);
    uint64_t off = 0, hi[kProgBits];
#pragma unroll
    for (int k = 0; k < kMidWin - kProgBits; ++k)
        if ((t >> k) & 1) off += 1ull << d.pos[k];
#pragma unroll
    for (int k = 0; k < kProgBits; ++k) hi[k] = 1ull << d.pos[kMidWin - kProgBits + k];
    if (REV)
        for (uint32_t s = t; s < d.n_slots * (kMT / 64); s += kMT) acc[s] = 0.0;
    for (uint64_t c = blk; c < d.n_cosets; c += d.n_blk) {
        uint64_t base = c;
#pragma unroll
        for (int k = 0; k < kMidWin; ++k) {
            const uint64_t low = base & ((1ull << d.pos[k]) - 1);
            base = ((base ^ low) << 1) | low;
        }
        base += off;
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            uint64_t idx = base;
#pragma unroll
            for (int k = 0; k < kProgBits; ++k)
                if ((p >> k) & 1) idx += hi[k];
            const uint32_t at = slot_of<T>(t + p * kMT) * A;
            if (!REV && d.first) {
                V v;
                v.x = idx == 0 ? T(1) : T(0);
                v.y = 0;
                *(V*)(sp + at) = v;
            } else {
                *(V*)(sp + at) = psi[idx];
            }
            if (REV) *(V*)(sl + at) = lam[idx];
        }
        run_program<T, REV ? 2 : 1, kMT>(sp, sl, blks, kMidWin, t, kMT, d.stages, d.n_stages, d.stream,
                                         [&](uint32_t s, double v) {
                                             if (REV) acc[s * (kMT / 64) + wave] += v;
                                         });
#pragma unroll
        for (int p = 0; p < kN; ++p) {
            uint64_t idx = base;
#pragma unroll
            for (int k = 0; k < kProgBits; ++k)
                if ((p >> k) & 1) idx += hi[k];
            const uint32_t at = slot_of<T>(t + p * kMT) * A;
            psi[idx] = *(const V*)(sp + at);
            if (REV) lam[idx] = *(const V*)(sl + at);
        }
        __syncthreads();  // the next coset restages the tiles
    }
    if (!REV) return;
    for (uint32_t s = t; s < d.n_slots; s += kMT) {
        double g = acc[s * (kMT / 64)];
#pragma unroll
        for (int w = 1; w < kMT / 64; ++w) g += acc[s * (kMT / 64) + w];
        part[d.part_off + (uint64_t)s * d.n_blk + blk] = g;
    }
}

constexpr int kHT = 256;  // threads per block of the tile form of H psi and of the reduction

// Block sum of kHT threads in a fixed order (waves, then wave totals in order), in every thread.
__device__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    __syncthreads();  // earlier readers of red are done
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int w = 1; w < kHT / 64; ++w) r += red[w];
    return r;
}

template <typename T>
__global__ void __launch_bounds__(kHT)
mid_hpsi_kernel(const MidHam* __restrict__ descs, uint32_t n_desc, double* __restrict__ part) {
    using V = typename VecB<T>::type;
    __shared__ double red[kHT / 64];
    const MidHam& d = descs[owner(descs, n_desc, blockIdx.x)];
    const uint32_t blk = blockIdx.x - d.blk_begin;
    const int t = threadIdx.x;
    const V* psi = reinterpret_cast<const V*>(d.psi);
    V* lam = reinterpret_cast<V*>(d.lam);
    const TermDesc<T>* terms = reinterpret_cast<const TermDesc<T>*>(d.terms);
    double e_acc = 0.0, n_acc = 0.0;
    for (uint64_t c = blk; c < d.n_tiles; c += d.n_blk) {
#pragma unroll
        for (int r = 0; r < (1 << kMidTileBits) / kHT; ++r) {
            const uint64_t b = (c << kMidTileBits) + t + kHT * r;
            T ar = 0, ai = 0;
            for (uint32_t gq = 0; gq < d.n_groups; ++gq) {
                const GroupDesc G = d.groups[gq];
                T dr = 0, di = 0;
                for (uint32_t k = G.begin; k < G.end; ++k) {
                    const TermDesc<T> tm = terms[k];
                    const bool neg = __popcll(tm.z & b) & 1;
                    dr += neg ? -tm.cre : tm.cre;
                    di += neg ? -tm.cim : tm.cim;
                }
                const V p = psi[b ^ G.x];
                ar += dr * p.x - di * p.y;
                ai += dr * p.y + di * p.x;
            }
            V l;
            l.x = ar;
            l.y = ai;
            lam[b] = l;
            const V p = psi[b];
            e_acc += (double)(p.x * ar + p.y * ai);
            n_acc += (double)(p.x * p.x + p.y * p.y);
        }
    }
    const double e = block_sum(e_acc, red);
    const double nn = block_sum(n_acc, red);
    if (t == 0) {
        part[d.part_off + blk] = e;
        part[d.part_off + d.n_blk + blk] = nn;
    }
}

__global__ void __launch_bounds__(kHT)
mid_reduce_kernel(const MidRed* __restrict__ r, const double* __restrict__ part, double* __restrict__ out) {
    __shared__ double red[kHT / 64];
    const MidRed d = r[blockIdx.x];
    double s = 0.0;
    for (uint32_t i = threadIdx.x; i < d.count; i += kHT) s += part[d.part_off + i];
    const double tot = block_sum(s, red);
    if (threadIdx.x == 0) out[blockIdx.x] = tot;
}

}  // namespace

template <typename T>
hipError_t launch_batch(const BatchDesc<T>* items, uint32_t n_items, int max_bits, hipStream_t st) {
    using V = typename VecB<T>::type;
    const size_t lds = 2 * kProgBlock + 2 * ((size_t)1 << max_bits) * sizeof(V);
    if (lds > (size_t)kBatchLdsBytes || max_bits < kBatchMinBits) return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_kernel<T>, dim3(n_items), dim3(1u << (max_bits - kProgBits)), lds, st, items);
    return hipGetLastError();
}

hipError_t batch_set_lds_limit() {
    hipError_t e = hipFuncSetAttribute((const void*)batch_kernel<float>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kBatchLdsBytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)batch_kernel<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kBatchLdsBytes);
}

template <typename T>
hipError_t launch_mid_pass(const MidPass* d, uint32_t n_desc, uint32_t grid, bool rev, double* part, hipStream_t st) {
    if (rev)
        hipLaunchKernelGGL((mid_pass_kernel<T, true>), dim3(grid), dim3(kMT), 0, st, d, n_desc, part);
    else
        hipLaunchKernelGGL((mid_pass_kernel<T, false>), dim3(grid), dim3(kMT), 0, st, d, n_desc, part);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mid_hpsi(const MidHam* d, uint32_t n_desc, uint32_t grid, double* part, hipStream_t st) {
    hipLaunchKernelGGL(mid_hpsi_kernel<T>, dim3(grid), dim3(kHT), 0, st, d, n_desc, part);
    return hipGetLastError();
}

hipError_t launch_mid_reduce(const MidRed* r, uint32_t n, const double* part, double* out, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(mid_reduce_kernel, dim3(n), dim3(kHT), 0, st, r, part, out);
    return hipGetLastError();
}

template hipError_t launch_mid_pass<float>(const MidPass*, uint32_t, uint32_t, bool, double*, hipStream_t);
template hipError_t launch_mid_pass<double>(const MidPass*, uint32_t, uint32_t, bool, double*, hipStream_t);
template hipError_t launch_mid_hpsi<float>(const MidHam*, uint32_t, uint32_t, double*, hipStream_t);
template hipError_t launch_mid_hpsi<double>(const MidHam*, uint32_t, uint32_t, double*, hipStream_t);
template hipError_t launch_batch<float>(const BatchDesc<float>*, uint32_t, int, hipStream_t);
template hipError_t launch_batch<double>(const BatchDesc<double>*, uint32_t, int, hipStream_t);

}  // namespace vqe

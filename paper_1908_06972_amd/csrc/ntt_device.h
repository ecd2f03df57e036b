// ntt_device.h -- device building blocks of the transforms: butterflies,
// register phases, twiddle sets, LDS exchanges and the X -> X^kappa tile
// gather, shared by the transform passes and conversions (ntt.hip) and the
// fused kernels of key switching (keyswitch.hip).  The decomposition into
// passes, phases and tiles is described in ntt.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pft_device.h"

namespace {

// ---- integer butterflies (51-bit to 60-bit q), 16q < 2^64

// Forward: with x = X (reduced below 2q first if `reduce`) and r = W Y mod q
// up to 4q, X' = x + r and Y' = x - r + 4q, both at most 4q above x; Y may be
// any 64-bit value.
__device__ __forceinline__ void fwd_bfly_int(uint64_t& X, uint64_t& Y, const TwPair& tp, const DevMod& md,
                                             bool reduce) {
    const uint64_t x = reduce ? reduce_int(X, md) : X;
    X = shoup_add4(x, Y, tp.w, tp.wp, md.nq);
    Y = ((x << 1) + 4 * md.q) - X;
}
// Integer forward stages of a pass reduce X only at stages spp with
// (LOG_M - 1 - spp) divisible by 3, counted from the pass's last stage so
// that the last stage reduces: from inputs up to 6q, the (at most two) stages
// before a reducing one leave values up to 10q and 14q, the reducing stage
// brings X below 2q and leaves at most 6q, and so does every pass.
__device__ __forceinline__ constexpr bool int_fwd_reduces(int log_m, int spp) { return (log_m - 1 - spp) % 3 == 0; }

// Inverse (Gentleman-Sande): X' = X + Y, Y' = (X - Y + B q) W up to 4q, for
// X, Y up to B q.  X' is reduced below 2q on the odd stages of a pass and on
// its last stage: from at most 4q an even stage leaves at most 8q (B = 4), an
// odd one at most 4q (B = 8, X + Y at most 16q), and so does every pass.
__device__ __forceinline__ void inv_bfly_int(uint64_t& X, uint64_t& Y, const TwPair& tp, const DevMod& md, int bit,
                                             bool last) {
    const uint64_t u = X + Y;
    const uint64_t d = X + ((bit & 1) ? 8 : 4) * md.q - Y;
    X = (bit & 1) || last ? reduce_int(u, md) : u;
    Y = shoup_add4(0, d, tp.w, tp.wp, md.nq);
}

// ---- fp64 butterflies (q < 2^50): fmulmod / freduce in pft_device.h
// Forward: X is reduced on every third stage of a pass (pass-local stage
// index = 0 mod 3).  With inputs within B q a reducing stage leaves
// (1 + B/4) q and a skipping one (5B/4 + 1/2) q.  A pass starts with a
// reducing stage, so at most two skipping stages follow one another; from
// inputs below 4q the bound settles at 2.1q after a reducing stage and stays
// below 4.5q (|values| < 2^53, and fmulmod's quotient is then off by at most
// 1/2 + 4.5/4, so every step stays exact).
__device__ __forceinline__ void fwd_bfly_fp(uint64_t& X, uint64_t& Y, const TwPair& tp, double q, double qinv,
                                            bool reduce_x) {
#pragma clang fp contract(off)
    const double x = reduce_x ? freduce(as_f(X), q, qinv) : as_f(X);
    const double t = fmulmod(as_f(Y), as_f(tp.w), as_f(tp.wp), q);
    X = as_u(x + t);
    Y = as_u(x - t);
}
// Inverse: X + Y is left unreduced on every third stage of a pass (stages in
// execution order, index = 2 mod 3).  Inputs within B q give X within q/2
// (reduced) or 2B q (not), Y within (1/2 + B/2) q; with two reducing stages
// between skipping ones the bound settles at 1.5q and stays below 4q.
__device__ __forceinline__ void inv_bfly_fp(uint64_t& X, uint64_t& Y, const TwPair& tp, double q, double qinv,
                                            bool reduce_x) {
#pragma clang fp contract(off)
    const double x = as_f(X), y = as_f(Y);
    X = as_u(reduce_x ? freduce(x + y, q, qinv) : x + y);
    Y = as_u(fmulmod(x - y, as_f(tp.w), as_f(tp.wp), q));
}
// Register phase PH of a radix-2^LOG_M pass with E = 2^EB residues per
// thread: stage bits HB down to LB; element e of thread l is index r_of(l, e)
// of its sub-problem (the EB window bits sit at WLO).
template <int LOG_M, int PH, int EB>
struct Phase {
    static constexpr int HB = LOG_M - 1 - EB * PH;                       // highest stage bit of this phase
    static constexpr int LB = (HB - (EB - 1) > 0) ? HB - (EB - 1) : 0;   // lowest stage bit
    static constexpr int WLO = (HB - (EB - 1) >= 0) ? HB - (EB - 1) : 0; // window of the register elements
    __device__ __forceinline__ static uint32_t r_of(uint32_t l, int e) {
        return ((l >> WLO) << (WLO + EB)) | ((uint32_t)e << WLO) | (l & ((1u << WLO) - 1u));
    }
};

// Twiddle index (high << spp) | (r >> (bit + 1)) of the butterfly at stage
// bit `bit` whose upper element is register e (r = r_of(l, e)).  The lane
// bits below the window drop out of the shift; in the phase that holds the
// window's top bits no lane bit is left, so the index is the same for every
// lane of a sub-problem.
template <int LOG_M, int PH, int EB>
__device__ __forceinline__ uint32_t tw_index(uint32_t l, int e, int bit, uint32_t high, int spp) {
    using Ph = Phase<LOG_M, PH, EB>;
    const uint32_t lhi = (Ph::WLO + EB >= LOG_M) ? 0u : (l >> Ph::WLO);
    return (high << spp) | (lhi << (Ph::WLO + EB - bit - 1)) | ((uint32_t)e >> (bit + 1 - Ph::WLO));
}

// Twiddles preloaded per register phase ahead of the exchange before it
// (PhaseTw below) by the transform passes with 8 or 16 residues per thread;
// larger budgets spill or cost waves per SIMD.
constexpr int TW_PRE_PASS3 = 8;
constexpr int TW_PRE_PASS4 = 3;
constexpr int tw_pre_pass(int eb) { return eb == 3 ? TW_PRE_PASS3 : eb == 4 ? TW_PRE_PASS4 : 0; }
// The twiddles of register phase PH for one thread.  At the stage whose
// butterflies span window bit pos, the upper elements e that agree in
// e >> (pos + 1) share one twiddle (tw_index drops the bits below), so the
// stage needs E >> (pos + 1) of them.  The first stages in execution order,
// up to PRE twiddles, are loaded by the constructor: a pass builds the set
// of its next phase before the LDS exchange that precedes that phase, so the
// loads are in flight during the exchange and its barrier (the fences of
// the exchange would keep the compiler from moving them there itself).  The
// later stages load at use.  The inverse transform's final stage with N^-1
// folded in (FOLD, phase 0, top bit) uses none.
template <int LOG_M, int PH, int EB, bool INV, bool FOLD, int PRE = 8>
struct PhaseTw {
    using Ph = Phase<LOG_M, PH, EB>;
    static constexpr int E = 1 << EB;
    static constexpr int P_HI = Ph::HB - Ph::WLO;  // window positions 0 .. P_HI
    static constexpr int MAXPRE = PRE;
    static constexpr int cnt(int pos) { return (INV && FOLD && PH == 0 && pos == P_HI) ? 0 : E >> (pos + 1); }
    struct Layout {
        int base[8];
        bool pre[8];
        int total;
    };
    static constexpr Layout layout() {
        Layout y{};
        int n = 0;
        bool open = true;
        for (int k = 0; k <= P_HI; ++k) {
            const int pos = INV ? k : P_HI - k;
            const int c = cnt(pos);
            if (open && n + c <= MAXPRE) {
                y.base[pos] = n;
                y.pre[pos] = true;
                n += c;
            } else {
                open = false;
                y.base[pos] = 0;
                y.pre[pos] = false;
            }
        }
        y.total = n;
        return y;
    }
    static constexpr Layout LY = layout();
    TwPair t[LY.total > 0 ? LY.total : 1];
    const TwPair* __restrict__ twt;
    uint32_t l, high, s0;

    __device__ __forceinline__ PhaseTw(const TwPair* __restrict__ tw, uint32_t l_, uint32_t high_, uint32_t s0_)
        : twt(tw), l(l_), high(high_), s0(s0_) {
#pragma unroll
        for (int pos = 0; pos <= P_HI; ++pos) {
            if (!LY.pre[pos]) continue;
#pragma unroll
            for (int m = 0; m < cnt(pos); ++m) t[LY.base[pos] + m] = load(pos, m << (pos + 1));
        }
    }
    // uniform base, 32-bit lane offset, constant rest: one address per stage
    __device__ __forceinline__ TwPair load(int pos, int e) const {
        const int bit = pos + Ph::WLO;
        const int spp = LOG_M - 1 - bit;
        const char* base = reinterpret_cast<const char*>(twt + (1u << (s0 + (uint32_t)spp)));
        const uint32_t lane = tw_index<LOG_M, PH, EB>(l, 0, bit, high, spp) * (uint32_t)sizeof(TwPair);
        return reinterpret_cast<const TwPair*>(base + lane)[(uint32_t)e >> (bit + 1 - Ph::WLO)];
    }
    // the twiddle of the butterfly at window bit pos whose upper element is e
    __device__ __forceinline__ TwPair get(int pos, int e) const {
        if (LY.pre[pos]) return t[LY.base[pos] + (e >> (pos + 1))];
        return load(pos, e);
    }
};

// One register phase of G independent tiles: each twiddle is loaded once and
// serves the butterflies of every tile.
// LOW (forward only): the inputs are already reduced (fp64 within q/2 + 1
// or below q; integers below 2q), so the first stage skips its reduction of
// X; the bounds of the later stages are those of reduced inputs.
template <int LOG_M, int PH, int EB, int G, bool INV, bool FP, bool FOLD, int PRE, bool LOW = false>
__device__ __forceinline__ void run_phase_g(uint64_t (&x)[G][1 << EB],
                                            const PhaseTw<LOG_M, PH, EB, INV, FOLD, PRE>& tw, const DevMod& md) {
    static_assert(!LOW || (!INV && PH == 0), "reduced inputs enter the first forward phase");
    using Ph = Phase<LOG_M, PH, EB>;
    constexpr int E = 1 << EB;
    [[maybe_unused]] const uint64_t q = md.q;
    const double qd = md.qd, qinv = md.qinv;
#pragma unroll
    for (int k = 0; k <= Ph::HB - Ph::LB; ++k) {
        const int bit = INV ? Ph::LB + k : Ph::HB - k;
        const int spp = LOG_M - 1 - bit;
        const int pos = bit - Ph::WLO;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e & (1 << pos)) continue;
            const int f = e | (1 << pos);
            if (INV && FOLD && PH == 0 && bit == Ph::HB) {
                // stage 0 with N^-1 folded in (integer path: outputs fully reduced)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint64_t X = x[g][e], Y = x[g][f];
                    if constexpr (FP) {
                        x[g][e] = as_u(fmulmod(as_f(X) + as_f(Y), md.n_inv_d, md.n_inv_q, qd));
                        x[g][f] = as_u(fmulmod(as_f(X) - as_f(Y), md.last_inv_d, md.last_inv_q, qd));
                    } else {
                        // inputs up to 8q; shoup takes any 64-bit value
                        x[g][e] = shoup(X + Y, md.n_inv, md.n_inv_sh, q);
                        x[g][f] = shoup(X + 8 * q - Y, md.last_inv, md.last_inv_sh, q);
                    }
                }
                continue;
            }
            const TwPair tp = tw.get(pos, e);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if constexpr (INV) {
                    if constexpr (FP)
                        inv_bfly_fp(x[g][e], x[g][f], tp, qd, qinv, bit % 3 != 2);
                    else
                        inv_bfly_int(x[g][e], x[g][f], tp, md, bit, bit == LOG_M - 1);
                } else {
                    const bool first = LOW && PH == 0 && spp == 0;  // folded after unrolling
                    if constexpr (FP)
                        fwd_bfly_fp(x[g][e], x[g][f], tp, qd, qinv, spp % 3 == 0 && !first);
                    else
                        fwd_bfly_int(x[g][e], x[g][f], tp, md, int_fwd_reduces(LOG_M, spp) && !first);
                }
            }
        }
    }
}

// One register phase of one tile loading each twiddle at its use (a
// single-phase pass: with no exchange in the way the compiler schedules the
// loads itself).
template <int LOG_M, int PH, int EB, bool INV, bool FP, bool FOLD, bool LOW = false>
__device__ __forceinline__ void run_phase(uint64_t (&x)[1 << EB], uint32_t l, uint32_t high, uint32_t s0,
                                          const TwPair* __restrict__ twt, const DevMod& md) {
    const PhaseTw<LOG_M, PH, EB, INV, FOLD, 0> tw(twt, l, high, s0);
    run_phase_g<LOG_M, PH, EB, 1, INV, FP, FOLD, 0, LOW>(reinterpret_cast<uint64_t(&)[1][1 << EB]>(x), tw, md);
}

// LDS word of element r of sub-problem c: c S + r + P (r >> 4), or, where
// the 8-byte words of a 16-lane group cannot all be spread over distinct
// bank pairs by a padding, c S + (r ^ h(r)) with h(r) = ((r >> XA) & 7) |
// (((r >> XB) & 1) << 3): the low four bits of r are permuted by higher
// ones (a bijection within each sub-problem).  The padded form is affine in
// the register index e of every arrangement (so ds_read/ds_write take
// immediate offsets).  The parameters are chosen per (M, residues per
// thread) by an exhaustive model of the LDS serving 16 lanes x 8 bytes per
// cycle over every access pattern of the pass -- each register phase's
// arrangement under both lane mappings, the staging order and the
// element-pair order of the staged store: with 16 residues per thread every
// row-pass pattern is conflict-free (radix 6 and 7 keep a two-way conflict
// on one), and with 8 the swizzled forms make the row passes of radix 7-12
// conflict-free where any padding leaves two-way conflicts (radix 9 and 10
// keep one two-way conflict pattern as column passes), and with 4 (row passes
// only) those of radix 8-12.
template <int LOG_M, int EB> struct LdsPad;
template <int EB> struct LdsPad<4, EB> { static constexpr uint32_t S = 17, P = 0, XA = 0, XB = 0; };
template <> struct LdsPad<6, 4> { static constexpr uint32_t S = 69, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<6, 3> { static constexpr uint32_t S = 73, P = 2, XA = 0, XB = 0; };
template <> struct LdsPad<7, 4> { static constexpr uint32_t S = 145, P = 2, XA = 0, XB = 0; };
template <> struct LdsPad<7, 3> { static constexpr uint32_t S = 129, P = 0, XA = 4, XB = 4; };
template <> struct LdsPad<8, 2> { static constexpr uint32_t S = 256, P = 0, XA = 2, XB = 5; };
template <> struct LdsPad<9, 2> { static constexpr uint32_t S = 512, P = 0, XA = 2, XB = 5; };
template <> struct LdsPad<10, 2> { static constexpr uint32_t S = 1024, P = 0, XA = 2, XB = 5; };
template <> struct LdsPad<11, 2> { static constexpr uint32_t S = 2048, P = 0, XA = 2, XB = 5; };
template <> struct LdsPad<12, 2> { static constexpr uint32_t S = 4096, P = 0, XA = 2, XB = 5; };
template <int EB> struct LdsPad<8, EB> { static constexpr uint32_t S = 273, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<8, 3> { static constexpr uint32_t S = 257, P = 0, XA = 4, XB = 5; };
template <int EB> struct LdsPad<9, EB> { static constexpr uint32_t S = 546, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<9, 3> { static constexpr uint32_t S = 514, P = 0, XA = 4, XB = 6; };
template <int EB> struct LdsPad<10, EB> { static constexpr uint32_t S = 1092, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<10, 3> { static constexpr uint32_t S = 1026, P = 0, XA = 4, XB = 4; };
template <int EB> struct LdsPad<11, EB> { static constexpr uint32_t S = 2176, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<11, 3> { static constexpr uint32_t S = 2048, P = 0, XA = 4, XB = 5; };
template <int EB> struct LdsPad<12, EB> { static constexpr uint32_t S = 4352, P = 1, XA = 0, XB = 0; };
template <> struct LdsPad<12, 3> { static constexpr uint32_t S = 4096, P = 0, XA = 4, XB = 6; };
// LDS words of a tile of 2^TB elements.
template <int LOG_M, int EB, int TB = 12>
constexpr uint32_t lds_words() { return ((1u << TB) >> LOG_M) * LdsPad<LOG_M, EB>::S; }
template <int LOG_M, int EB>
__device__ __forceinline__ uint32_t lds_at(uint32_t c, uint32_t r) {
    using L = LdsPad<LOG_M, EB>;
    if constexpr (L::XA != 0)
        return c * L::S + (r ^ (((r >> L::XA) & 7u) | (((r >> L::XB) & 1u) << 3)));
    else
        return c * L::S + r + L::P * (r >> 4);
}

template <int LOG_M, int PH, int EB>
__device__ __forceinline__ void lds_read(uint64_t (&x)[1 << EB], const uint64_t* lds, uint32_t c, uint32_t l) {
#pragma unroll
    for (int e = 0; e < (1 << EB); ++e) x[e] = lds[lds_at<LOG_M, EB>(c, Phase<LOG_M, PH, EB>::r_of(l, e))];
}
template <int LOG_M, int PH, int EB>
__device__ __forceinline__ void lds_write(const uint64_t (&x)[1 << EB], uint64_t* lds, uint32_t c, uint32_t l) {
#pragma unroll
    for (int e = 0; e < (1 << EB); ++e) lds[lds_at<LOG_M, EB>(c, Phase<LOG_M, PH, EB>::r_of(l, e))] = x[e];
}

// Where thread-index bit b lands in the word index c M + r of register
// phase PH (COL: c = tid mod C, l = tid / C; otherwise c = tid / T, l =
// tid mod T; r = Phase::r_of(l, e)).
template <int LOG_M, int EB, bool COL, int TB = 12>
constexpr int tid_bit_pos(int ph, int b) {
    constexpr int LT = LOG_M - EB;  // log2 of the threads per sub-problem
    constexpr int LC = TB - LOG_M;  // log2 of the sub-problems per workgroup
    const int hb = LOG_M - 1 - EB * ph;
    const int wlo = hb - (EB - 1) >= 0 ? hb - (EB - 1) : 0;
    int lb = 0;
    if (COL) {
        if (b < LC) return LOG_M + b;
        lb = b - LC;
    } else {
        if (b >= LT) return LOG_M + (b - LT);
        lb = b;
    }
    return lb < wlo ? lb : lb + EB;
}
// Whether the exchange between register phases pa and pb stays inside each
// wave: every wave reads back exactly the words it wrote (its wave-index
// bits land on the same word-index bits in both phases, and its lane bits
// and element window cover the same set).  Such an exchange needs no
// workgroup barrier: a wave's LDS instructions execute in order, so its
// reads see its own earlier writes, and no other wave touches those words.
template <int LOG_M, int EB, bool COL, int TB = 12>
constexpr bool wave_local_exchange(int pa, int pb) {
    constexpr int LNT = TB - EB;  // log2 of the threads per workgroup
    if (LNT <= 6) return true;
    for (int b = 6; b < LNT; ++b)
        if (tid_bit_pos<LOG_M, EB, COL, TB>(pa, b) != tid_bit_pos<LOG_M, EB, COL, TB>(pb, b)) return false;
    auto varying = [](int ph) {
        const int hb = LOG_M - 1 - EB * ph;
        const int wlo = hb - (EB - 1) >= 0 ? hb - (EB - 1) : 0;
        uint32_t m = ((1u << EB) - 1u) << wlo;
        for (int b = 0; b < 6; ++b) m |= 1u << tid_bit_pos<LOG_M, EB, COL, TB>(ph, b);
        return m;
    };
    return varying(pa) == varying(pb);
}
// Orders a wave's LDS writes before its following reads without a
// workgroup barrier (the compiler must not move memory accesses across it).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The register phases of one pass of G tiles in execution order (forward: 0,
// 1, ...; inverse: the reverse), with an LDS exchange between consecutive
// phases, each tile through its own LDS region (one barrier per exchange for
// all of them).  Each thread writes back to the words it read last, so one
// barrier per exchange suffices; an exchange that stays inside each wave
// needs none.
template <int LOG_M, int EB, int G, bool INV, bool FP, bool FOLD, int K, bool COL, int PRE, int TB>
__device__ __forceinline__ void run_phases_g(uint64_t (&x)[G][1 << EB], uint64_t* lds, uint32_t c, uint32_t l,
                                             uint32_t high, uint32_t s0, const TwPair* __restrict__ twt,
                                             const DevMod& md) {
    constexpr int NPH = (LOG_M + EB - 1) / EB;
    constexpr uint32_t W = lds_words<LOG_M, EB, TB>();
    if constexpr (K < NPH) {
        constexpr int PH = INV ? NPH - 1 - K : K;
        // the phase's twiddle loads go out before the exchange
        const PhaseTw<LOG_M, PH, EB, INV, FOLD, PRE> tw(twt, l, high, s0);
        if constexpr (K > 0) {
            constexpr int PREV = INV ? PH + 1 : PH - 1;
#pragma unroll
            for (int g = 0; g < G; ++g) lds_write<LOG_M, PREV, EB>(x[g], lds + g * W, c, l);
            if constexpr (wave_local_exchange<LOG_M, EB, COL, TB>(PREV, PH))
                wave_lds_sync();
            else
                __syncthreads();
#pragma unroll
            for (int g = 0; g < G; ++g) lds_read<LOG_M, PH, EB>(x[g], lds + g * W, c, l);
        }
        run_phase_g<LOG_M, PH, EB, G, INV, FP, FOLD, PRE>(x, tw, md);
        run_phases_g<LOG_M, EB, G, INV, FP, FOLD, K + 1, COL, PRE, TB>(x, lds, c, l, high, s0, twt, md);
    }
}
template <int LOG_M, int EB, bool INV, bool FP, bool FOLD, bool COL = false, int PRE = 0, int TB = 12>
__device__ __forceinline__ void run_phases(uint64_t (&x)[1 << EB], uint64_t* lds, uint32_t c, uint32_t l,
                                           uint32_t high, uint32_t s0, const TwPair* __restrict__ twt,
                                           const DevMod& md) {
    run_phases_g<LOG_M, EB, 1, INV, FP, FOLD, 0, COL, PRE, TB>(reinterpret_cast<uint64_t(&)[1][1 << EB]>(x), lds, c, l,
                                                               high, s0, twt, md);
}

// X -> X^kappa on an NTT-domain row (entry k holds the evaluation at
// psi^(2 brv(k) + 1)) is the gather out[k] = in[sigma(k)] with
// sigma(k) = brv(((2 brv(k) + 1) kappa mod 2N - 1) / 2).  In natural order
// the map is affine modulo N, so the low bits of the image depend only on
// the low bits of the argument; in bit-reversed order the high bits of
// sigma(k) depend only on the high bits of k: every aligned tile of 2^TB
// words of the result comes from one aligned tile of the input.  This stages
// destination tile `tile` of the result in LDS (in the pass's LDS layout):
// the source tile is read coalesced and word k of it is written at
// pi(k) = sigma^-1(k) (kappa_inv in place of kappa), converted to the fp64
// form if to_fp.  Ends with a barrier.
__device__ __forceinline__ uint32_t galois_index(uint32_t k, uint32_t kap, uint32_t log_n) {
    const uint32_t e = 2u * brev_n(k, log_n) + 1u;
    const uint32_t e2 = (e * kap) & ((2u << log_n) - 1u);  // 2N divides 2^32: the low product bits suffice
    return brev_n((e2 - 1u) >> 1, log_n);
}
template <int LOG_M, int EB, int TB = 12>
__device__ __forceinline__ void galois_tile_to_lds(const uint64_t* __restrict__ src, uint32_t tile, uint32_t log_n,
                                                   uint64_t kappa, uint64_t kappa_inv, uint64_t* lds, bool to_fp) {
    constexpr uint32_t NT = (1u << TB) >> EB;
    constexpr int E = 1 << EB;
    constexpr uint32_t M = 1u << LOG_M;
    const uint32_t st = galois_index(tile << TB, (uint32_t)kappa, log_n) >> TB;
    const uint64_t* __restrict__ s = src + ((size_t)st << TB);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const uint32_t idx = threadIdx.x + NT * (uint32_t)k;
        const uint32_t d = galois_index((st << TB) + idx, (uint32_t)kappa_inv, log_n) - (tile << TB);
        const uint64_t v = s[idx];
        lds[lds_at<LOG_M, EB>(d / M, d % M)] = to_fp ? fp_from_u64(v) : v;
    }
    __syncthreads();
}

}  // namespace

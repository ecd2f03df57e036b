// keyswitch.hip -- the fused kernels of hybrid key switching around the base
// conversions: everything between ModUp's rows and the finished ciphertext
// in two launches, and the inverse transforms before them in one.
//
// The conversion kernels (ntt.hip) leave every extended row after the first
// (radix-16 column) pass of its forward transform, so each still needs one
// row pass of LOG_M = log_n - 4 stages, over tiles that no other tile
// touches.  All that follows is tile-local as well: the products with the
// key, ModDown's subtraction, the addends.  So a workgroup takes one tile of
// one row of one item through the whole of it, in registers:
//   * k_ks_inv, the rows of what is switched: the row pass of their inverse
//     transform (ModUp's conversion applies the last pass), from operands
//     that are formed as they are read;
//   * k_ks_rows<.., SPECIAL true>, the K special rows: every digit through
//     the row pass, products with the key summed into two accumulators, and
//     the accumulators through the row pass of the inverse transform that
//     ModDown's conversion needs (it applies the last pass itself);
//   * k_ks_rows<.., SPECIAL false>, the ciphertext rows, once the conversion
//     of the special rows is there: the digits and their products as above,
//     the two converted rows through their row pass, and the output
//     out_b = (acc_b - conv_b) P^-1.  An addend enters the accumulators as P
//     times itself, so the output is (acc_b - conv_b) P^-1 + add_b.
// No accumulator of a ciphertext row, no transformed row and no tensor of a
// product (d0, d1, d2 below) goes to memory.  RESCALE runs on the same
// kernels: its last limb through k_ks_inv, its output rows through k_ks_rows
// without digits.
//
// Two forms of each: 8 residues a thread (EB 3), and 4 (EB 2) where a launch
// cannot fill the chip anyway: a tile's chain of passes then has twice the
// waves, half the instructions per wave, and takes the rows of both
// arithmetic kinds in one launch.
//
// Measured (MI355X).  16 HMULTs at N = 2^16, level 24, four digits: the fp64
// ciphertext rows 880 us (VALU issue 55%, 2.4 GB at 2.8 TB/s: the chain of
// loads, passes and products at two workgroups a compute unit bounds it, and
// neither the next rows' loads nor the key tiles ahead of the pass, which spill
// or cost a workgroup, nor 8-byte twiddles moved it), the special rows 308 (60-bit
// butterflies, VALU issue 85%), the one integer row 222 beside the fp64 rows,
// k_ks_inv 170.  Before, with the key products, the inverse and ModDown's
// passes and the tensor as launches of their own, the whole call took 2045 us;
// 1525 now.  One item at N = 2^15, level 16: k_ks_inv 7.8, special rows 16.4,
// last launch 24.3 us, each a few dependent rounds of memory and of LDS.
#include "ntt_device.h"
#include "pft_device.h"
#include "pft_kernels.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>

namespace {

// Twiddles of the next register phase loaded ahead of an exchange (PhaseTw):
// with 4 residues a thread all of them; with 8 more spill at four waves per
// SIMD.
constexpr int tw_pre_ks(int eb, bool fp, int g) { return eb == 2 ? 3 : fp && g == 2 ? 3 : 1; }

// One tile's work (see the head of this file).  FP (rows with q < 2^50, the
// key holding integer-valued doubles): every product is an fmulmod against
// the quotient w (1/q); a term lies within 0.9q, an addend's P product
// within q, and the accumulators are reduced to within q/2 after the own
// digit and the addends, so with at most 7 further terms they stay below
// 6.8q < 2^53.  Otherwise the Montgomery products with the key (stored times
// 2^64) are summed without REDC's final subtraction (terms below 2q) onto
// accumulators brought below 2q after the own digit and the addends: with at
// most 7 further terms below 16q < 2^64, reduced once at the end.
//
// G digits go through the row pass together (G = 2: each twiddle load and
// each LDS barrier serves two tiles, and their butterflies are independent
// instruction streams); the two converted rows of the output are such a pair
// too.
template <int LOG_M, int EB, int TB, bool FP, int G, bool SPECIAL>
__device__ __forceinline__ void ks_row(const KsRows& a, const KsItem& it, uint64_t* lds, uint32_t z, uint32_t tile, uint32_t entry,
                                       uint32_t t, uint32_t mi, const DevMod& md, const TwPair* __restrict__ tw,
                                       const TwPair* __restrict__ tw_inv, uint32_t log_n) {
    constexpr int M = 1 << LOG_M;
    constexpr int E = 1 << EB;
    constexpr uint32_t NT = (1u << TB) >> EB;
    constexpr int T = M / E;
    constexpr int C = NT / T;
    constexpr int NPH = (LOG_M + EB - 1) / EB;
    using PIN = Phase<LOG_M, 0, EB>;
    using POUT = Phase<LOG_M, NPH - 1, EB>;
    static_assert(PIN::WLO >= 4, "the row pass reads its input directly");
    static_assert(POUT::WLO == 0, "each thread ends with E consecutive words");
    static_assert(G == 1 || G == 2, "one or two tiles per row pass");
    constexpr int PRE = tw_pre_ks(EB, FP, G);
    // integer ciphertext rows of the small form: their sums may be formed in
    // the special rows' launch (early) and be there in the last one (ready)
    constexpr bool SPLIT = EB == 2 && !FP;

    const uint32_t tid = threadIdx.x;
    [[maybe_unused]] const uint64_t q = md.q;
    const double qd = md.qd, qinv = md.qinv;
    const TwPair* __restrict__ twt = tw + ((size_t)mi << log_n);
    const uint32_t s0 = log_n - LOG_M;
    const uint32_t sp0 = tile * (uint32_t)C;
    const uint32_t c = C == 1 ? 0u : tid / T;
    const uint32_t l = C == 1 ? tid : tid % T;
    uint64_t* __restrict__ item = a.base + (size_t)z * a.stride;
    const uint64_t* __restrict__ key = it.key;
    // Rows are addressed as a uniform base and a 32-bit lane offset in bytes.
    // This thread's E consecutive words of a row start at w0, its words in the
    // row pass's input arrangement at r0.
    const uint32_t w0 = (((sp0 + c) << LOG_M) + l * (uint32_t)E) * 8u;
    const uint32_t r0 = (((sp0 + c) << LOG_M) | PIN::r_of(l, 0)) * 8u;
    auto words = [](const uint64_t* p, uint32_t off) {
        return reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(p) + off);
    };

    auto load_vec = [&](const uint64_t* __restrict__ p, uint64_t (&v)[E]) {
        const ulonglong2* __restrict__ pv = reinterpret_cast<const ulonglong2*>(words(p, w0));
#pragma unroll
        for (int e = 0; e < E / 2; ++e) {
            const ulonglong2 u = pv[e];
            v[2 * e] = u.x;
            v[2 * e + 1] = u.y;
        }
    };
    const bool early = SPECIAL && SPLIT && t < a.level;
    const bool ready = !SPECIAL && SPLIT && (entry >> KS_ROW_EARLY) != 0;
    const uint32_t part = SPECIAL ? (entry >> KS_ROW_PART) & 7u : 0u;
    // an early row's part s of polynomial 1
    [[maybe_unused]] auto early1 = [&](uint32_t s) {
        const uint32_t e = (entry >> KS_ROW_EARLY) - 1u;
        return item + a.off_acc + ((size_t)ks_early_row1(a.rows - a.level, a.parts, e, s) << log_n);
    };
    uint64_t acc0[E], acc1[E];  // FP: doubles; otherwise residues
#pragma unroll
    for (int e = 0; e < E; ++e) acc0[e] = acc1[e] = 0;  // also the bits of +0.0
    // acc += x k, one residue
    auto mac1 = [&](uint64_t x, uint64_t k, uint64_t& acc) {
        if constexpr (FP) {
#pragma clang fp contract(off)
            const double w = as_f(k);
            acc = as_u(as_f(acc) + fmulmod(as_f(x), w, w * qinv, qd));
        } else {
            acc = mont_add2(acc, x, k, md);
        }
    };
    // acc_b += x k, k the key tile key_{j,b}[t] of this thread's words
    auto mac = [&](const uint64_t (&x)[E], uint32_t j, int b, uint64_t (&acc)[E]) {
        uint64_t k[E];
        load_vec(key + ((size_t)((2 * j + b) * a.krows + mi) << log_n), k);
#pragma unroll
        for (int e = 0; e < E; ++e) mac1(x[e], k[e], acc[e]);
    };
    auto accumulate = [&](const uint64_t (&x)[E], uint32_t j) {
        mac(x, j, 0, acc0);
        mac(x, j, 1, acc1);
    };
    // a row after the conversion kernel's column pass into x
    auto load_row = [&](const uint64_t* __restrict__ src, uint64_t (&x)[E]) {
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = *words(src + ((size_t)e << PIN::WLO), r0);
    };
    auto ext = [&](uint32_t j) { return item + a.off_ext + ((size_t)(j * a.rows + t) << log_n); };
    auto store_vec = [&](uint64_t* __restrict__ p, const uint64_t (&v)[E]) {
        ulonglong2* __restrict__ pv = reinterpret_cast<ulonglong2*>(const_cast<uint64_t*>(words(p, w0)));
#pragma unroll
        for (int e = 0; e < E / 2; ++e) {
            ulonglong2 u;
            u.x = v[2 * e];
            u.y = v[2 * e + 1];
            pv[e] = u;
        }
    };
    // the row pass's output brought within q/2 (FP; the integer products take any value)
    auto settle = [&](uint64_t (&x)[E]) {
        if constexpr (FP) {
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = as_u(freduce(as_f(x[e]), qd, qinv));
        }
    };
    // One or two rows through the row pass.  The twiddles and their addresses
    // are the same for every row; an opaque zero offset of their base and
    // opaque copies of the lane indices keep the compiler from holding all of
    // them in registers from one row to the next (they are recomputed and
    // reloaded).  The offset, not the pointer, is hidden, so the loads stay
    // global (not flat) loads.
    auto pass_1 = [&](uint64_t (&x)[E]) {
        uint32_t lj = l, cj = c;
        asm volatile("" : "+v"(lj), "+v"(cj));
        run_phases<LOG_M, EB, false, FP, false, false, PRE, TB>(x, lds, cj, lj, sp0 + c, s0, twt, md);
        __syncthreads();  // the next row's exchanges reuse the LDS
    };
    [[maybe_unused]] auto pass_2 = [&](uint64_t (&x)[2][E]) {
        uint32_t lj = l, cj = c;
        asm volatile("" : "+v"(lj), "+v"(cj));
        run_phases_g<LOG_M, EB, 2, false, FP, false, 0, false, PRE, TB>(x, lds, cj, lj, sp0 + c, s0, twt, md);
        __syncthreads();
    };
    auto digit_1 = [&](uint32_t j) {
        uint64_t x[E];
        load_row(ext(j), x);
        pass_1(x);
        settle(x);
        accumulate(x, j);
    };
    [[maybe_unused]] auto digit_2 = [&](uint32_t j1, uint32_t j2) {
        uint64_t x[2][E];
        load_row(ext(j1), x[0]);
        load_row(ext(j2), x[1]);
        pass_2(x);
        settle(x[0]);
        accumulate(x[0], j1);
        settle(x[1]);
        accumulate(x[1], j2);
    };

    uint32_t jo = ~0u;  // the digit whose own rows include t: d itself, no transform needed
    const size_t row0 = (size_t)t << log_n, row1 = (size_t)(a.src_level + t) << log_n;
    if (!SPECIAL && a.mode == KS_RESCALE) {
        // the input's rows in the accumulators' place
        load_vec(it.src + row0, acc0);
        load_vec(it.src + row1, acc1);
        if constexpr (FP) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                acc0[e] = fp_from_u64(acc0[e]);
                acc1[e] = fp_from_u64(acc1[e]);
            }
        }
    } else if constexpr (!SPECIAL) {
        jo = t / a.alpha;
        const TwPair pm = FP ? a.gadget_fp[t] : a.gadget[t];  // P mod q
        // acc_b += P s for s = an addend, canonical (FP: as a double, or a sum of two such or of two products)
        auto add_p = [&](uint64_t s, uint64_t& acc) {
            if constexpr (FP) {
#pragma clang fp contract(off)
                acc = as_u(as_f(acc) + fmulmod(as_f(s), as_f(pm.w), as_f(pm.wp), qd));
            } else {
                acc += shoup_lazy(s, pm.w, pm.wp, q);
            }
        };
        if (a.mode == KS_PRODUCT) {
            // d2 = a1 b1 is switched; d0 = a0 b0 and d1 = a0 b1 + a1 b0 are added
            const uint64_t* __restrict__ A = it.src;
            const uint64_t* __restrict__ B = it.src2;
            const uint64_t* __restrict__ k0 = key + ((size_t)(2 * jo * a.krows + mi) << log_n);
            const uint64_t* __restrict__ k1 = k0 + ((size_t)a.krows << log_n);
            // two words of every operand at a time; the scheduling barrier
            // after each half of them bounds the loads in flight (registers)
#pragma unroll
            for (int e = 0; e < E; e += 2) {
                auto two = [&](const uint64_t* __restrict__ p) {
                    return *reinterpret_cast<const ulonglong2*>(words(p, w0) + e);
                };
                const ulonglong2 va1 = two(A + row1), vb1 = two(B + row1), va0 = two(A + row0), vb0 = two(B + row0),
                                 vk0 = two(k0), vk1 = two(k1);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint64_t a1 = h ? va1.y : va1.x, b1 = h ? vb1.y : vb1.x, a0 = h ? va0.y : va0.x,
                                   b0 = h ? vb0.y : vb0.x, w0k = h ? vk0.y : vk0.x, w1k = h ? vk1.y : vk1.x;
                    if constexpr (FP) {
#pragma clang fp contract(off)
                        const double x1 = as_f(fp_from_u64(a1)), y1 = as_f(fp_from_u64(b1));
                        const double x0 = as_f(fp_from_u64(a0)), y0 = as_f(fp_from_u64(b0));
                        const double y1q = y1 * qinv, y0q = y0 * qinv;
                        const uint64_t d2 = as_u(fmulmod(x1, y1, y1q, qd));
                        mac1(d2, w0k, acc0[e + h]);
                        mac1(d2, w1k, acc1[e + h]);
                        add_p(as_u(fmulmod(x0, y0, y0q, qd)), acc0[e + h]);
                        add_p(as_u(fmulmod(x0, y1, y1q, qd) + fmulmod(x1, y0, y0q, qd)), acc1[e + h]);
                    } else {
                        const uint64_t d2 = mul_barrett(a1, b1, md);
                        mac1(d2, w0k, acc0[e + h]);
                        mac1(d2, w1k, acc1[e + h]);
                        add_p(mul_barrett(a0, b0, md), acc0[e + h]);
                        add_p(mul_barrett(a0, b1, md) + mul_barrett(a1, b0, md), acc1[e + h]);
                    }
                }
                if (!FP || (e & 2) != 0) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            uint64_t x[E];
            if (a.mode == KS_ROTATE) {
                // d = X^kappa image of c1's row t, its tile staged in LDS; the
                // image of c0's row is added
                galois_tile_to_lds<LOG_M, EB, TB>(it.src + row1, tile, log_n, it.gal.kappa, it.gal.kappa_inv, lds, FP);
#pragma unroll
                for (int e = 0; e < E; ++e) x[e] = lds[lds_at<LOG_M, EB>(c, l * (uint32_t)E + (uint32_t)e)];
                __syncthreads();
                accumulate(x, jo);
                galois_tile_to_lds<LOG_M, EB, TB>(it.src + row0, tile, log_n, it.gal.kappa, it.gal.kappa_inv, lds, FP);
#pragma unroll
                for (int e = 0; e < E; ++e)
                    add_p(lds[lds_at<LOG_M, EB>(c, l * (uint32_t)E + (uint32_t)e)], acc0[e]);
                __syncthreads();  // the digits' exchanges reuse the LDS
            } else {
                load_vec(item + a.off_d + row0, x);
                if constexpr (FP) {
#pragma unroll
                    for (int e = 0; e < E; ++e) x[e] = fp_from_u64(x[e]);
                }
                accumulate(x, jo);
            }
            if (a.has_add) {
                const uint64_t* A = it.src2;  // may be the output: each word is read before it is written
                uint64_t s[E];
                load_vec(A + row0, s);
#pragma unroll
                for (int e = 0; e < E; ++e) add_p(FP ? fp_from_u64(s[e]) : s[e], acc0[e]);
                load_vec(A + row1, s);
#pragma unroll
                for (int e = 0; e < E; ++e) add_p(FP ? fp_from_u64(s[e]) : s[e], acc1[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (FP) {
                acc0[e] = as_u(freduce(as_f(acc0[e]), qd, qinv));
                acc1[e] = as_u(freduce(as_f(acc1[e]), qd, qinv));
            } else {
                acc0[e] = reduce_int(acc0[e], md);  // at most three terms below 2q
                acc1[e] = reduce_int(acc1[e], md);
            }
        }
    }
    // every other digit through the row pass, G at a time (uniform control
    // flow: t, level, alpha and beta are the same for the whole workgroup)
    if (early) jo = t / a.alpha;
    const uint32_t j0 = SPECIAL ? part * a.group : 0u;
    const uint32_t j1 = ready ? 0u : SPECIAL ? min(a.beta, j0 + a.group) : a.beta;
    uint32_t pend = ~0u;
    for (uint32_t j = j0; j < j1; ++j) {
        if (j == jo) continue;
        if constexpr (G == 1) {
            digit_1(j);
        } else {
            if (pend == ~0u) {
                pend = j;
                continue;
            }
            digit_2(pend, j);
            pend = ~0u;
        }
    }
    if (pend != ~0u) digit_1(pend);

    if constexpr (SPLIT) {
        if (ready) {  // at most four parts below 2q each onto sums below 2q
            for (uint32_t s = 0; s < a.parts; ++s) {
                uint64_t x[2][E];
                load_vec(ext(s * a.group), x[0]);
                load_vec(early1(s), x[1]);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    acc0[e] += x[0][e];
                    acc1[e] += x[1][e];
                }
            }
        }
        if (early) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                acc0[e] = reduce_int(acc0[e], md);
                acc1[e] = reduce_int(acc1[e], md);
            }
            store_vec(ext(j0), acc0);
            store_vec(early1(part), acc1);
            return;
        }
    }
    if constexpr (SPECIAL) {
        // both accumulators through the row pass of their inverse transform
        const TwPair* __restrict__ twi = tw_inv + ((size_t)mi << log_n);
        uint64_t* o0 = item + a.off_acc + ((size_t)t << log_n);
        uint64_t* o1 = o0 + ((size_t)a.rows << log_n);
        if (a.packed) {  // see KsSplit
            o0 = ext(j0);
            o1 = item + a.off_acc + ((size_t)ks_special_row1(a.rows - a.level, t - a.level, part) << log_n);
        }
        auto put = [&](const uint64_t (&x)[E], uint32_t b) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                *const_cast<uint64_t*>(words((b ? o1 : o0) + ((size_t)e << PIN::WLO), r0)) = x[e];
        };
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (FP) {
                acc0[e] = as_u(freduce(as_f(acc0[e]), qd, qinv));
                acc1[e] = as_u(freduce(as_f(acc1[e]), qd, qinv));
            } else {
                acc0[e] = reduce_int(acc0[e], md);
                acc1[e] = reduce_int(acc1[e], md);
            }
        }
        uint32_t lj = l, cj = c;
        asm volatile("" : "+v"(lj), "+v"(cj));
        if constexpr (G == 2) {
            uint64_t x[2][E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                x[0][e] = acc0[e];
                x[1][e] = acc1[e];
            }
            run_phases_g<LOG_M, EB, 2, true, FP, false, 0, false, PRE, TB>(x, lds, cj, lj, sp0 + cj, s0, twi, md);
            put(x[0], 0);
            put(x[1], 1);
        } else {
            run_phases<LOG_M, EB, true, FP, false, false, PRE, TB>(acc0, lds, cj, lj, sp0 + cj, s0, twi, md);
            put(acc0, 0);
            __syncthreads();
            asm volatile("" : "+v"(lj), "+v"(cj));
            run_phases<LOG_M, EB, true, FP, false, false, PRE, TB>(acc1, lds, cj, lj, sp0 + cj, s0, twi, md);
            put(acc1, 1);
        }
    } else {
        const TwPair pinv = FP ? a.pinv_fp[t] : a.pinv[t];  // P^-1 mod q
        // x: the transformed converted row; the result to row t of polynomial b
        auto finish = [&](const uint64_t (&x)[E], const uint64_t (&acc)[E], uint32_t b) {
            ulonglong2* __restrict__ o = reinterpret_cast<ulonglong2*>(
                const_cast<uint64_t*>(words(it.out + ((size_t)(b * a.level + t) << log_n), w0)));
            uint64_t r[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (FP) {
#pragma clang fp contract(off)
                    // acc within q/2, the converted row within 4.5q
                    const double y = freduce(as_f(acc[e]), qd, qinv) - as_f(x[e]);
                    r[e] = fp_to_u64(as_u(fmulmod(y, as_f(pinv.w), as_f(pinv.wp), qd)), qd, qinv);
                } else {
                    // the converted row up to 6q
                    r[e] = shoup(reduce_int(acc[e], md) + 6 * q - x[e], pinv.w, pinv.wp, q);
                }
            }
#pragma unroll
            for (int e = 0; e < E / 2; ++e) {
                ulonglong2 v;
                v.x = r[2 * e];
                v.y = r[2 * e + 1];
                o[e] = v;
            }
        };
        auto conv = [&](uint32_t b) { return item + a.off_conv + ((size_t)(b * a.level + t) << log_n); };
        if constexpr (G == 2) {
            uint64_t x[2][E];
            load_row(conv(0), x[0]);
            load_row(conv(1), x[1]);
            pass_2(x);
            finish(x[0], acc0, 0);
            finish(x[1], acc1, 1);
        } else {
            uint64_t x[E];
            load_row(conv(0), x);
            pass_1(x);
            finish(x, acc0, 0);
            load_row(conv(1), x);
            pass_1(x);
            finish(x, acc1, 1);
        }
    }
}

// Block order: blocks are issued to the eight XCDs round-robin; block id
// 8 k + x runs item k mod n of the (row, tile) pair 8 floor(k / n) + x, so
// the items sharing one key tile run on one XCD at about the same time and
// the tile comes from HBM about once per launch, then from that XCD's L2.
// Returns false past the last pair.
__device__ __forceinline__ bool ks_block(uint32_t n_items, uint32_t tiles, uint32_t n_rows, uint32_t& z,
                                         uint32_t& tile, uint32_t& r) {
    const uint32_t kx = blockIdx.x >> 3;
    z = kx % n_items;
    const uint32_t pair = (kx / n_items) * 8u + (blockIdx.x & 7u);
    tile = pair % tiles;
    r = pair / tiles;
    return pair < tiles * n_rows;
}

// KIND: the rows of a launch run fp64 (KS_ROWS_FP), integer (KS_ROWS_INT) or
// either (KS_ROWS_ALL) arithmetic.
template <int LOG_M, int EB, int TB, uint32_t KIND, int G, bool SPECIAL>
__global__ __launch_bounds__((1 << TB) >> EB) __attribute__((amdgpu_waves_per_eu(4)))
void k_ks_rows(KsRows a, const DevMod* __restrict__ mods, const TwPair* __restrict__ tw,
               const TwPair* __restrict__ tw_inv, uint32_t log_n) {
    __shared__ uint64_t lds[G * lds_words<LOG_M, EB, TB>()];
    uint32_t z, tile, r;
    if (!ks_block(a.n_items, a.tiles, a.n_rows, z, tile, r)) return;  // whole workgroup, before any barrier
    const KsItem it = a.item[z];
    const uint32_t entry = a.row[r], t = entry & KS_ROW_MASK;
    const uint32_t mi = t < a.level ? t : a.L + (t - a.level);
    const DevMod md = mods[mi];
    if (KIND == KS_ROWS_FP || (KIND == KS_ROWS_ALL && md.fp))
        ks_row<LOG_M, EB, TB, true, G, SPECIAL>(a, it, lds, z, tile, entry, t, mi, md, tw, tw_inv, log_n);
    else
        ks_row<LOG_M, EB, TB, false, G, SPECIAL>(a, it, lds, z, tile, entry, t, mi, md, tw, tw_inv, log_n);
}

// The row pass (the first) of an inverse transform of rows that are read, or
// formed, in the NTT domain; see KsInv.
template <int LOG_M, int EB, int TB>
__global__ __launch_bounds__((1 << TB) >> EB) __attribute__((amdgpu_waves_per_eu(4)))
void k_ks_inv(KsInv a, const DevMod* __restrict__ mods, const TwPair* __restrict__ tw_inv, uint32_t log_n) {
    constexpr int M = 1 << LOG_M;
    constexpr int E = 1 << EB;
    constexpr uint32_t NT = (1u << TB) >> EB;
    constexpr int T = M / E;
    constexpr int C = NT / T;
    using PIN = Phase<LOG_M, 0, EB>;
    __shared__ uint64_t lds[lds_words<LOG_M, EB, TB>()];
    uint32_t z, tile, r;
    if (!ks_block(a.n_items, a.tiles, a.n_rows, z, tile, r)) return;
    const KsInvItem it = a.item[z];
    const uint32_t mi = a.mod0 + r * a.mod_step;
    const DevMod md = mods[mi];
    const TwPair* __restrict__ twi = tw_inv + ((size_t)mi << log_n);
    const uint32_t tid = threadIdx.x;
    const uint32_t sp0 = tile * (uint32_t)C;
    const uint32_t c = C == 1 ? 0u : tid / T;
    const uint32_t l = C == 1 ? tid : tid % T;
    const uint32_t w0 = (((sp0 + c) << LOG_M) + l * (uint32_t)E) * 8u;
    const uint32_t r0 = (((sp0 + c) << LOG_M) | PIN::r_of(l, 0)) * 8u;
    uint64_t* __restrict__ item = a.base + (size_t)z * a.stride;
    const size_t row = (size_t)(a.src_row + r * a.src_step) << log_n;
    auto two = [&](const uint64_t* __restrict__ p, int e) {
        return *reinterpret_cast<const ulonglong2*>(reinterpret_cast<const char*>(p + e) + w0);
    };
    uint64_t x[E];
    if (a.mode == KS_ROTATE) {
        galois_tile_to_lds<LOG_M, EB, TB>(it.src + row, tile, log_n, it.gal.kappa, it.gal.kappa_inv, lds, md.fp != 0);
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = lds[lds_at<LOG_M, EB>(c, l * (uint32_t)E + (uint32_t)e)];
    } else if (a.mode == KS_PRODUCT) {
        const uint64_t *A = it.src + row, *B = it.src2 + row;
#pragma unroll
        for (int e = 0; e < E; e += 2) {
            const ulonglong2 u = two(A, e), v = two(B, e);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint64_t p = h ? u.y : u.x, s = h ? v.y : v.x;
                if (md.fp) {
                    const double y = as_f(fp_from_u64(s));
                    x[e + h] = as_u(fmulmod(as_f(fp_from_u64(p)), y, y * md.qinv, md.qd));  // within 0.9q
                } else {
                    x[e + h] = mul_barrett(p, s, md);
                }
            }
        }
    } else {
        const uint64_t* A = a.mode == KS_WS ? item + a.off_d + row : it.src + row;
#pragma unroll
        for (int e = 0; e < E; e += 2) {
            const ulonglong2 u = two(A, e);
            x[e] = md.fp ? fp_from_u64(u.x) : u.x;
            x[e + 1] = md.fp ? fp_from_u64(u.y) : u.y;
        }
    }
    constexpr int PRE = EB == 2 ? 3 : 8;
    if (md.fp)
        run_phases<LOG_M, EB, true, true, false, false, PRE, TB>(x, lds, c, l, sp0 + c, log_n - LOG_M, twi, md);
    else
        run_phases<LOG_M, EB, true, false, false, false, PRE, TB>(x, lds, c, l, sp0 + c, log_n - LOG_M, twi, md);
    uint64_t* __restrict__ o = item + a.off_out + ((size_t)r << log_n);
#pragma unroll
    for (int e = 0; e < E; ++e)
        *reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(o + ((size_t)e << PIN::WLO)) + r0) = x[e];
}

// Calls f(integral_constant LOG_M, integral_constant TB) for the row pass of
// ring 2^log_n.  A tile is one row-pass problem, at least 1024 words: the
// smallest that fills a pair of wavefronts with 8 residues a thread.
template <class F>
void by_row_pass(uint32_t log_n, F&& f) {
    auto go = [&](auto lm) {
        constexpr int LM = decltype(lm)::value;
        f(lm, std::integral_constant<int, (LM > 10 ? LM : 10)>{});
    };
    switch (log_n - 4) {
        case 8: go(std::integral_constant<int, 8>{}); break;
        case 9: go(std::integral_constant<int, 9>{}); break;
        case 10: go(std::integral_constant<int, 10>{}); break;
        case 11: go(std::integral_constant<int, 11>{}); break;
        case 12: go(std::integral_constant<int, 12>{}); break;
        default: break;
    }
}

}  // namespace

bool ks_rows_supported(uint32_t log_n) {
    const uint32_t r = log_n - 4;
    return r >= 8 && r <= 12;
}

void launch_ks_inv(uint32_t n, KsInv a, const DevTables& t, uint32_t log_n, hipStream_t st, ProfHook* prof) {
    a.n_items = n;
    const bool small = ks_small(n, a.n_rows, log_n);
    if (prof) prof->begin(PK_NTT_INV, st);
    by_row_pass(log_n, [&](auto lm, auto tb) {
        constexpr int LM = decltype(lm)::value, TB = decltype(tb)::value;
        a.tiles = (1u << log_n) >> TB;
        const dim3 grid(8u * n * ((a.tiles * a.n_rows + 7u) / 8u));
        if (small)
            hipLaunchKernelGGL((k_ks_inv<LM, 2, TB>), grid, dim3((1u << TB) >> 2), 0, st, a, t.mods, t.tw_inv, log_n);
        else
            hipLaunchKernelGGL((k_ks_inv<LM, 3, TB>), grid, dim3((1u << TB) >> 3), 0, st, a, t.mods, t.tw_inv, log_n);
    });
    if (prof) {
        const double words = (double)n * a.n_rows * (double)(1u << log_n);
        prof->end(PK_NTT_INV, 8.0 * words * (a.mode == KS_PRODUCT ? 2.0 : 1.0), 0.5 * words * (log_n - 4),
                  8192u + (log_n - 4) + (small ? 64u : 0u), st);
    }
}

void launch_ks_rows(uint32_t n, KsRows a, bool special, const KsConsts& kc, const DevTables& t,
                    const uint32_t* fp_rows, uint32_t log_n, bool pair_digits, hipStream_t st, ProfHook* prof,
                    uint32_t rows_sel, KsSplit split) {
    const uint32_t level = a.level;
    a.n_items = n;
    a.rows = level + kc.K;
    a.alpha = kc.alpha;
    a.beta = a.mode == KS_RESCALE ? 0 : (level + kc.alpha - 1) / kc.alpha;
    a.src_level = a.mode == KS_RESCALE ? level + 1 : level;
    // the integer accumulators hold at most 8 terms below 2q (callers check)
    if (a.beta > 8) {
        fprintf(stderr, "launch_ks_rows: %u digits, at most 8 supported\n", a.beta);
        abort();
    }
    a.L = kc.L;
    a.krows = kc.L + kc.K;
    a.parts = split.parts;
    a.group = split.parts > 1 ? split.group : a.beta;
    a.packed = split.packed() ? 1u : 0u;
    const bool small = ks_small(n, special ? kc.K : level, log_n);
    // the rows of one arithmetic kind (the small form: of both, the longer
    // integer rows first), in chunks that fit the row list
    for (uint32_t kind : {KS_ROWS_FP, KS_ROWS_INT}) {
        if (!(rows_sel & kind) || (small && kind == KS_ROWS_FP && rows_sel == KS_ROWS_ALL)) continue;
        std::vector<uint32_t> rows;
        for (uint32_t k : {KS_ROWS_INT, KS_ROWS_FP}) {
            if (k != kind && !(small && rows_sel == KS_ROWS_ALL)) continue;
            for (uint32_t r = special ? level : 0; r < (special ? a.rows : level); ++r) {
                const uint32_t mi = r < level ? r : kc.L + (r - level);
                if (fp_rows[mi] != (k == KS_ROWS_FP ? 1u : 0u)) continue;
                for (uint32_t s = 0; s < (special ? a.parts : 1u); ++s) rows.push_back(r | s << KS_ROW_PART);
            }
        }
        if (split.early) {
            // last, being shorter than the other rows
            std::vector<uint32_t> ints;
            for (uint32_t r = 0, e = 1; r < level; ++r)
                if (!fp_rows[r]) ints.push_back(r | e++ << KS_ROW_EARLY);
            if (special) {
                for (uint32_t i : ints)
                    for (uint32_t s = 0; s < a.parts; ++s) rows.push_back(i | s << KS_ROW_PART);
            } else {
                rows.erase(rows.begin(), rows.begin() + ints.size());
                rows.insert(rows.end(), ints.begin(), ints.end());
            }
        }
        for (size_t r0 = 0; r0 < rows.size(); r0 += PFT_ROW_LIST) {
            a.n_rows = (uint32_t)std::min<size_t>(PFT_ROW_LIST, rows.size() - r0);
            std::copy_n(rows.begin() + r0, a.n_rows, a.row);
            const bool g2 = small || (kind == KS_ROWS_FP && pair_digits && !special);
            if (prof) prof->begin(PK_KEY_INNER, st);
            by_row_pass(log_n, [&](auto lm, auto tb) {
                constexpr int LM = decltype(lm)::value, TB = decltype(tb)::value;
                a.tiles = (1u << log_n) >> TB;
                const dim3 grid(8u * n * ((a.tiles * a.n_rows + 7u) / 8u));
                auto run = [&](auto ebc, auto kindc, auto gc, auto spc) {
                    constexpr int EB = decltype(ebc)::value;
                    hipLaunchKernelGGL(
                        (k_ks_rows<LM, EB, TB, decltype(kindc)::value, decltype(gc)::value, decltype(spc)::value>),
                        grid, dim3((1u << TB) >> EB), 0, st, a, t.mods, t.tw_fwd, t.tw_inv, log_n);
                };
                using e2 = std::integral_constant<int, 2>;
                using e3 = std::integral_constant<int, 3>;
                using g_1 = std::integral_constant<int, 1>;
                using g_2 = std::integral_constant<int, 2>;
                using fp = std::integral_constant<uint32_t, KS_ROWS_FP>;
                using in = std::integral_constant<uint32_t, KS_ROWS_INT>;
                using all = std::integral_constant<uint32_t, KS_ROWS_ALL>;
                if (small)
                    special ? run(e2{}, all{}, g_2{}, std::true_type{}) : run(e2{}, all{}, g_2{}, std::false_type{});
                else if (special)
                    kind == KS_ROWS_FP ? run(e3{}, fp{}, g_1{}, std::true_type{})
                                       : run(e3{}, in{}, g_1{}, std::true_type{});
                else if (g2)
                    run(e3{}, fp{}, g_2{}, std::false_type{});
                else
                    kind == KS_ROWS_FP ? run(e3{}, fp{}, g_1{}, std::false_type{})
                                       : run(e3{}, in{}, g_1{}, std::false_type{});
            });
            if (prof) {
                // method bytes: the operands and the finished rows per item, the
                // key rows once (extended and converted rows are pass boundaries);
                // work: the row passes' butterflies and the products
                const double N = (double)(1u << log_n), lm = (double)(log_n - 4);
                const double in = special ? 0.0 : a.mode == KS_PRODUCT ? 4.0 : a.mode == KS_WS ? 1.0 : 2.0;
                const double io = in + (special ? 0.0 : 2.0 + (a.has_add ? 2.0 : 0.0));
                // a special row once for all its parts, an early row with the last launch
                const double m = (double)std::count_if(a.row, a.row + a.n_rows, [&](uint32_t e) {
                    return !special || (e >> KS_ROW_PART) == 0;
                });
                prof->end(PK_KEY_INNER, 8.0 * N * m * (n * io + 2.0 * a.beta),
                          N * n * m * (0.5 * lm * (a.beta + (special ? 2.0 : 1.0)) + 2.0 * a.beta),
                          1024u + (log_n - 4) + (small ? 512u : kind == KS_ROWS_FP ? 64u : 0u) + (g2 ? 128u : 0u) +
                              (special ? 256u : 0u),
                          st);
            }
        }
    }
}

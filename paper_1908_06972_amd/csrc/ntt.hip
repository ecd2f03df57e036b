// ntt.hip -- negacyclic NTT / inverse NTT per RNS limb for gfx950.
//
// Forward: A[k] = sum_j a_j psi^((2 brv(k) + 1) j) (evaluation of a(X) at the
// odd powers of the primitive 2N-th root psi, bit-reversed order).  It is
// computed by log2(N) radix-2 stages; stage s (0-based) pairs index j with
// j + N/2^(s+1) and uses the twiddle psi^brv(2^s + (j >> (log2 N - s))).
// The inverse runs the stages backwards with Gentleman-Sande butterflies and
// psi^-brv(.) twiddles, and folds N^-1 into its last stage.
//
// Decomposition.  A pass executes a window of LOG_M consecutive stages.  The
// elements touched by those stages split into independent sub-problems of
// M = 2^LOG_M elements (fixed high index bits above the window, fixed low
// bits below it).  A 256-thread workgroup owns 4096 elements: C = 4096/M
// sub-problems, 16 elements per thread held in registers.  Inside a pass the
// stages run in phases of up to 4 (radix-16 in registers); between phases the
// elements are exchanged through LDS.  Global memory is read and written in
// a coalesced order through LDS (consecutive lanes touch consecutive
// addresses: along the sub-problem index when low bits exist, else along
// the sub-problem itself).  The split of the stages into passes is a
// schedule (ntt_candidates below lists them per N; the first is the default,
// e.g. one pass of 12 stages at N = 2^12 and 8 + 8 at N = 2^16); a
// context's autotuner or a tuning table picks one per direction and batch
// size (the large-ring workload uses 4 + 12 for its forward transforms).
// Arithmetic, chosen per limb (uniform within a workgroup):
//   * q < 2^50: fp64.  A residue fits the 53-bit significand, and MI355X issues
//     fp64 FMA at the full VALU rate, so an exact product modulo q costs six
//     fp64 instructions instead of some twenty 32-bit integer ones (bounds at
//     fmulmod below).
//   * otherwise (q < 2^60): 64-bit integer Shoup butterflies kept lazily
//     reduced (forward up to 14q inside a pass and 6q between passes,
//     inverse up to 8q and 4q).
// Inputs below 4q are accepted; outputs of a full transform are in [0, q).
#include "bconv_device.h"
#include "ntt_device.h"
#include "pft_device.h"
#include "pft_kernels.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>

namespace {

// One pass over stages s0 .. s0 + LOG_M - 1 of a 4096-element tile.
// COL (stages below log_n - LOG_M leave low index bits: the M elements of a
// sub-problem are 2^lbits apart): consecutive lanes take consecutive
// sub-problems, so every register arrangement is a coalesced global access
// and the pass loads and stores directly.  Row passes (lbits = 0, each
// sub-problem contiguous): consecutive lanes walk along a sub-problem.  With
// STAGE, a side whose arrangement gives runs shorter than 16 words goes
// through LDS in address order; without, it is accessed directly, and the
// arrangement in which each thread owns 16 consecutive words (the window's
// lowest stages) moves 16 bytes per lane per access.
// Limbs with DevMod::fp run the fp64 butterflies: the first pass of a
// transform converts its u64 input, later passes exchange the doubles through
// HBM, and the final pass writes canonical u64.  Integer limbs keep u64.
template <int LOG_M, int EB, bool INV, bool COL, bool FINAL, bool STAGE, bool EPI>
__global__ __launch_bounds__(4096 >> EB) void k_ntt_pass(PolyBatch b, const DevMod* __restrict__ mods,
                                                         const TwPair* __restrict__ tw, uint32_t log_n, uint32_t s0,
                                                         uint32_t first_pass, NttEpilogue ep) {
    constexpr int M = 1 << LOG_M;
    constexpr int E = 1 << EB;          // residues per thread
    constexpr uint32_t NT = 4096 >> EB;  // threads per workgroup
    constexpr int T = M / E;             // threads per sub-problem
    constexpr int C = NT / T;            // sub-problems per workgroup
    constexpr int NPH = (LOG_M + EB - 1) / EB;
    constexpr int PH_IN = INV ? NPH - 1 : 0;
    constexpr int PH_OUT = INV ? 0 : NPH - 1;
    using PIN = Phase<LOG_M, PH_IN, EB>;
    using POUT = Phase<LOG_M, PH_OUT, EB>;
    constexpr bool DIRECT_IN = COL || !STAGE || PIN::WLO >= 4;
    constexpr bool DIRECT_OUT = COL || !STAGE || POUT::WLO >= 4;
    // a row-pass arrangement where thread l owns words E l .. E l + E - 1
    constexpr bool VEC_IN = !COL && PIN::WLO == 0;
    constexpr bool VEC_OUT = !COL && POUT::WLO == 0;
    __shared__ uint64_t lds[lds_words<LOG_M, EB>()];

    const uint32_t tid = threadIdx.x;
    const uint32_t job = blockIdx.y;
    const uint32_t limb = job / b.n_polys;
    const uint32_t poly = job - limb * b.n_polys;
    const uint32_t row = pb_row(b, poly, limb);
    const uint32_t mi = pb_mod(b, row);
    uint64_t* __restrict__ data = b.ptr[poly] + ((size_t)row << log_n);
    const DevMod md = mods[mi];
    const bool fp = md.fp != 0;
    const TwPair* __restrict__ twt = tw + ((size_t)mi << log_n);

    // a row pass has no index bits below its window (s0 + LOG_M = log_n)
    const uint32_t lbits = COL ? log_n - s0 - LOG_M : 0u;
    const uint32_t lmask = (1u << lbits) - 1u;
    const uint32_t sp0 = blockIdx.x * C;
    const uint32_t c = C == 1 ? 0u : (COL ? tid % C : tid / T);
    const uint32_t l = C == 1 ? tid : (COL ? tid / C : tid % T);
    const uint32_t high = (sp0 + c) >> lbits;
    // index in the row of element r of the workgroup's sub-problem cc
    auto gidx = [&](uint32_t cc, uint32_t r) -> uint32_t {
        const uint32_t sp = sp0 + cc;
        return ((((sp >> lbits) << LOG_M) | r) << lbits) | (sp & lmask);
    };
    // word i of a row: a uniform base and a 32-bit lane offset in bytes
    auto word = [](auto* p, uint32_t i) {
        using W = std::remove_pointer_t<decltype(p)>;
        using B = std::conditional_t<std::is_const_v<W>, const char, char>;
        return reinterpret_cast<W*>(reinterpret_cast<B*>(p) + i * 8u);
    };

    uint64_t x[E];
    const bool convert_in = fp && first_pass;
    const uint64_t* src = first_pass ? data + b.src_delta : data;  // may alias data (in place)
    if constexpr (DIRECT_IN && VEC_IN) {
        const ulonglong2* __restrict__ srcv = reinterpret_cast<const ulonglong2*>(word(src, gidx(c, (uint32_t)E * l)));
#pragma unroll
        for (int e = 0; e < E / 2; ++e) {
            const ulonglong2 v = srcv[e];
            x[2 * e] = convert_in ? fp_from_u64(v.x) : v.x;
            x[2 * e + 1] = convert_in ? fp_from_u64(v.y) : v.y;
        }
    } else if constexpr (DIRECT_IN) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint64_t v = *word(src + ((size_t)((uint32_t)e << PIN::WLO) << lbits), gidx(c, PIN::r_of(l, 0)));
            x[e] = convert_in ? fp_from_u64(v) : v;
        }
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const uint32_t idx = tid + NT * k;
            const uint32_t cc = idx / M, r = idx % M;
            const uint64_t v = *word(src, gidx(cc, r));
            lds[lds_at<LOG_M, EB>(cc, r)] = convert_in ? fp_from_u64(v) : v;
        }
        __syncthreads();
        lds_read<LOG_M, PH_IN, EB>(x, lds, c, l);
    }

    // the final inverse pass (s0 = 0) folds N^-1 into stage 0
    if (fp)
        run_phases<LOG_M, EB, INV, true, FINAL, COL, tw_pre_pass(EB)>(x, lds, c, l, high, s0, twt, md);
    else
        run_phases<LOG_M, EB, INV, false, FINAL, COL, tw_pre_pass(EB)>(x, lds, c, l, high, s0, twt, md);

    const uint64_t q = md.q;
    const double qd = md.qd, qinv = md.qinv;
    auto finish = [&](uint64_t v) -> uint64_t {
        if constexpr (FINAL) {
            if (fp) {
                v = fp_to_u64(v, qd, qinv);
            } else if constexpr (!INV) {
                v = reduce_int(v, md);
                v = v >= q ? v - q : v;
            }
        }
        return v;
    };
    // ModDown / RESCALE epilogue operands (uniform per workgroup)
    [[maybe_unused]] const uint32_t bsel = poly & 1u;
    [[maybe_unused]] uint64_t* __restrict__ out_row =
        EPI ? ep.out[poly >> 1] + ((size_t)(bsel * ep.level + row) << log_n) : nullptr;
    [[maybe_unused]] const TwPair pinv = EPI ? (fp ? ep.pinv_fp[row] : ep.pinv[row]) : TwPair{0, 0};
    [[maybe_unused]] const uint64_t* __restrict__ acc_src = nullptr;
    [[maybe_unused]] const uint64_t* __restrict__ add_src = nullptr;
    [[maybe_unused]] const uint64_t* add2_src = nullptr;  // may be out_row: read before it is written
    if constexpr (EPI) {
        acc_src = ep.d_acc[bsel] == PFT_EPI_ITEM_ACC
                      ? ep.acc_item[poly >> 1] + ((size_t)(bsel * ep.acc_level + row) << log_n)
                      : data + ep.d_acc[bsel];
        if (ep.d_add[bsel] != PFT_EPI_NO_ADD) add_src = data + ep.d_add[bsel];
        if (ep.has_add) add2_src = ep.src[poly >> 1] + ((size_t)(bsel * ep.level + row) << log_n);
    }
    // Epilogue stores of the E elements pos(k) with register forms val(k)
    // (integer-valued doubles within 4.5q for fp64 limbs; finish() reduces
    // integer limbs).  Every load of a chunk is issued before the first
    // result is formed, so their latencies overlap.
    // PAIRS: positions come in adjacent pairs (pos(2m + 1) = pos(2m) + 1 with
    // pos(2m) even), moved as 16-byte accesses.
    [[maybe_unused]] auto epi_store = [&](auto pos, auto val, auto pairs) {
        constexpr bool PAIRS = decltype(pairs)::value;
        constexpr int CH = E < 8 ? E : 8;
        auto ld = [&](const uint64_t* __restrict__ p, const uint32_t (&jj)[CH], uint64_t (&v)[CH]) {
            if constexpr (PAIRS) {
#pragma unroll
                for (int k = 0; k < CH; k += 2) {
                    const ulonglong2 t = *reinterpret_cast<const ulonglong2*>(word(p, jj[k]));
                    v[k] = t.x;
                    v[k + 1] = t.y;
                }
            } else {
#pragma unroll
                for (int k = 0; k < CH; ++k) v[k] = *word(p, jj[k]);
            }
        };
#pragma unroll
        for (int k0 = 0; k0 < E; k0 += CH) {
            uint32_t jj[CH];
            uint64_t a[CH], u[CH], w[CH], r[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) jj[k] = pos(k0 + k);
            ld(acc_src, jj, a);
            if (add_src) ld(add_src, jj, u);
            if (add2_src) ld(add2_src, jj, w);
            if (fp) {
#pragma unroll
                for (int k = 0; k < CH; ++k) {
#pragma clang fp contract(off)
                    // (acc - conv) P^-1 with |acc - conv| < 5.5q: within 2q; the
                    // addends (< q each) keep it within 5q before the final reduction
                    double y = fmulmod(as_f(fp_from_u64(a[k])) - as_f(val(k0 + k)), as_f(pinv.w), as_f(pinv.wp), qd);
                    if (add_src) y += as_f(fp_from_u64(u[k]));
                    if (add2_src) y += as_f(fp_from_u64(w[k]));
                    r[k] = fp_to_u64(as_u(y), qd, qinv);
                }
            } else {
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    uint64_t v = shoup(a[k] + q - finish(val(k0 + k)), pinv.w, pinv.wp, q);
                    if (add_src) v = add_mod(v, u[k], q);
                    if (add2_src) v = add_mod(v, w[k], q);
                    r[k] = v;
                }
            }
            if constexpr (PAIRS) {
#pragma unroll
                for (int k = 0; k < CH; k += 2) {
                    ulonglong2 t;
                    t.x = r[k];
                    t.y = r[k + 1];
                    *reinterpret_cast<ulonglong2*>(word(out_row, jj[k])) = t;
                }
            } else {
#pragma unroll
                for (int k = 0; k < CH; ++k) *word(out_row, jj[k]) = r[k];
            }
        }
    };
    if constexpr (DIRECT_OUT && VEC_OUT && !EPI) {
        ulonglong2* __restrict__ dst = reinterpret_cast<ulonglong2*>(word(data, gidx(c, (uint32_t)E * l)));
#pragma unroll
        for (int e = 0; e < E / 2; ++e) {
            ulonglong2 v;
            v.x = finish(x[2 * e]);
            v.y = finish(x[2 * e + 1]);
            dst[e] = v;
        }
    } else if constexpr (DIRECT_OUT) {
        if constexpr (EPI)
            epi_store([&](int e) { return (uint32_t)gidx(c, POUT::r_of(l, e)); }, [&](int e) { return x[e]; },
                      std::false_type{});
        else
#pragma unroll
            for (int e = 0; e < E; ++e)
                *word(data + ((size_t)((uint32_t)e << POUT::WLO) << lbits), gidx(c, POUT::r_of(l, 0))) = finish(x[e]);
    } else {
        lds_write<LOG_M, PH_OUT, EB>(x, lds, c, l);
        __syncthreads();
        auto at = [&](int k) {
            const uint32_t idx = tid + NT * k;
            return std::pair<uint32_t, uint32_t>(idx / M, idx % M);
        };
        if constexpr (EPI) {
            // element pairs 2 (tid + NT m) and its successor: adjacent in the
            // row (a row pass has no index bits below its window)
            auto at2 = [&](int k) {
                const uint32_t idx = 2u * (tid + NT * (uint32_t)(k >> 1)) + (uint32_t)(k & 1);
                return std::pair<uint32_t, uint32_t>(idx / M, idx % M);
            };
            if constexpr (!COL) {
                epi_store([&](int k) { const auto p = at2(k); return (uint32_t)gidx(p.first, p.second); },
                          [&](int k) { const auto p = at2(k); return lds[lds_at<LOG_M, EB>(p.first, p.second)]; },
                          std::true_type{});
            } else {
                epi_store([&](int k) { const auto p = at(k); return (uint32_t)gidx(p.first, p.second); },
                          [&](int k) { const auto p = at(k); return lds[lds_at<LOG_M, EB>(p.first, p.second)]; },
                          std::false_type{});
            }
        } else if constexpr (!COL) {
            // adjacent element pairs of the row as 16-byte stores
#pragma unroll
            for (int m = 0; m < E / 2; ++m) {
                const uint32_t idx = 2u * (tid + NT * (uint32_t)m);
                const uint32_t cc = idx / M, r = idx % M;
                ulonglong2 v;
                v.x = finish(lds[lds_at<LOG_M, EB>(cc, r)]);
                v.y = finish(lds[lds_at<LOG_M, EB>(cc, r + 1)]);
                *reinterpret_cast<ulonglong2*>(word(data, gidx(cc, r))) = v;
            }
        } else {
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const auto p = at(k);
                *word(data, gidx(p.first, p.second)) = finish(lds[lds_at<LOG_M, EB>(p.first, p.second)]);
            }
        }
    }
}

template <int LOG_M, int EB, bool INV, bool COL, bool FINAL>
void launch_k(const PolyBatch& b, const DevTables& t, uint32_t log_n, uint32_t s0, uint32_t first_pass, bool stage,
              const NttEpilogue* epi, hipStream_t st) {
    const dim3 grid((1u << log_n) / 4096u, b.n_polys * b.n_limbs);
    const TwPair* tw = INV ? t.tw_inv : t.tw_fwd;
    const NttEpilogue ep = epi ? *epi : NttEpilogue{};
    if constexpr (!INV && !COL && FINAL) {
        // the epilogue reads acc and the addend and writes out beside the
        // transformed value: always through the coalesced staged store
        if (epi) {
            hipLaunchKernelGGL((k_ntt_pass<LOG_M, EB, INV, COL, FINAL, true, true>), grid, dim3(4096 >> EB), 0, st, b,
                               t.mods, tw, log_n, s0, first_pass, ep);
            return;
        }
    }
    if (COL || stage)
        hipLaunchKernelGGL((k_ntt_pass<LOG_M, EB, INV, COL, FINAL, true, false>), grid, dim3(4096 >> EB), 0, st, b,
                           t.mods, tw, log_n, s0, first_pass, ep);
    else if constexpr (!COL)
        hipLaunchKernelGGL((k_ntt_pass<LOG_M, EB, INV, COL, FINAL, false, false>), grid, dim3(4096 >> EB), 0, st, b,
                           t.mods, tw, log_n, s0, first_pass, ep);
}

// One pass.  A column pass (low index bits remain below the window) needs at
// least 16 sub-problems per workgroup for coalescing, so radices above 8 only
// run as the last window.  Going forward the last window is the final pass;
// going back the s0 = 0 window is.
template <int LOG_M, bool INV>
void launch_pass(const PolyBatch& b, const DevTables& t, uint32_t log_n, uint32_t s0, bool final_pass, bool stage,
                 bool e8, const NttEpilogue* epi, hipStream_t st, ProfHook* g_prof) {
    const int kid = INV ? PK_NTT_INV : PK_NTT_FWD;
    const uint32_t first_pass = INV ? (s0 + LOG_M == log_n) : (s0 == 0);
    const bool col = s0 + LOG_M < log_n;
    const bool staged = col || stage || (epi && !INV && final_pass);
    if (g_prof) g_prof->begin(kid);
    auto go = [&](auto eb) {
        constexpr int EB = decltype(eb)::value;
        if (col) {
            if constexpr (LOG_M <= 8) launch_k<LOG_M, EB, INV, true, INV>(b, t, log_n, s0, first_pass, true, nullptr, st);
        } else if (final_pass) {
            if constexpr (!INV || LOG_M == 12)
                launch_k<LOG_M, EB, INV, false, true>(b, t, log_n, s0, first_pass, stage, epi, st);
        } else {
            if constexpr (INV) launch_k<LOG_M, EB, INV, false, false>(b, t, log_n, s0, first_pass, stage, epi, st);
        }
    };
    if (e8)
        go(std::integral_constant<int, 3>{});
    else
        go(std::integral_constant<int, 4>{});
    if (g_prof) {
        const double elems = (double)b.n_polys * b.n_limbs * (double)(1u << log_n);
        // method bytes: the transform's input (read by its first pass) and
        // output (written by its final pass), 8 bytes per residue each; the
        // words between two passes are the layout's cost, not the method's.
        // N/2 butterflies per stage.
        const bool fused = epi && !INV && final_pass && !col;
        const uint32_t variant = 1u + (LOG_M | (col ? 32u : 0u) | (final_pass ? 64u : 0u) | (staged ? 128u : 0u) |
                                       (e8 ? 256u : 0u) | (fused ? 512u : 0u));
        // the ModDown epilogue reads acc (and the addends) and writes out in
        // place of the transform's own store
        double extra = 0.0;  // addends: half of the rows (one polynomial) each
        if (fused) {
            for (int bb = 0; bb < 2; ++bb)
                extra += (epi->d_add[bb] != PFT_EPI_NO_ADD ? 4.0 : 0.0) + (epi->has_add ? 4.0 : 0.0);
        }
        const double in_b = first_pass ? 8.0 : 0.0, out_b = final_pass ? 8.0 : 0.0;
        const double bytes = elems * (in_b + (fused ? 16.0 + extra : out_b));
        g_prof->end(kid, bytes, 0.5 * elems * LOG_M, variant);
    }
}

// A base conversion of hybrid key switching fused with the first pass
// (stages 0-3, a radix-16 column pass) of the forward transform of every row
// it produces.  ModUp (DOWN false): digit j = blockIdx.y of item z =
// blockIdx.z, inputs the digit's rows of d, targets every row outside the
// digit (q-limbs and special primes), output ext_j.  ModDown (DOWN true):
// polynomial b = blockIdx.y, inputs the K special rows of acc_b, targets the
// q-limbs 0..level-1, output conv_b.
//
// A workgroup converts the 512 coefficients u0 + u + t N/16 (u < 32, t < 16)
// of 32 columns.  First a half-wave per input row takes its columns' 16
// values, forms their digits and leaves them in LDS as the matrix operand of
// block t (columns u).  Then each wave takes tiles of four target rows: per
// block t the same exact contraction on the matrix cores and fold as the
// stand-alone conversion kernels.  The 32 columns of an accumulator tile are
// the 32 columns u, so a lane ends with all 16 values t of its column for two
// targets, in registers, and takes them through the four stages exactly as
// the first transform pass does (on fp64 rows the fold's reduced double is
// already the butterflies' input form), storing that pass's output form; the
// transform continues with its second pass.  The tiles hold rows of one
// arithmetic kind, so a wave never runs both; no target goes through LDS.
//
// IFUSE: the input rows come from an inverse transform whose final pass (a
// radix-16 column pass, stages 3-0 with N^-1 folded in) has not run; it is
// applied to the 16 values of each column first.
//
// Bound by the VALU: the integer butterflies of 60-bit rows, the fold, the
// inputs' products.  16 items at N = 2^16, level 24: ModUp's 338 us and
// ModDown's 171 (500 and 231 when the folded values went through LDS to
// another thread's column and a wave's tile mixed the arithmetic kinds).
//
// SMALL (with IFUSE): the form of launches that leave compute units with one
// or two workgroups, where the length of a wave's chain counts: four threads
// share a column's inverse pass (the sums of ModDown's parts too), and two
// waves a tile of targets.
constexpr uint32_t BCONV_COLS = 32;
template <uint32_t NKB, bool DOWN, bool IFUSE, bool SMALL>
__global__ __launch_bounds__(SMALL ? 1024 : 512) __attribute__((amdgpu_waves_per_eu(4))) void k_bconv_col_b(
    WsRef ws, BconvIn src, uint64_t off_out, uint32_t level, KsConsts kc, const DevMod* __restrict__ mods,
    const TwPair* __restrict__ tw, const TwPair* __restrict__ tw_inv, uint32_t log_n) {
    __shared__ uint64_t s_dig[2 * NKB * 16 * BCONV_COLS];  // [input row][t][u]
    extern __shared__ uint4 s_dyn[];  // fold constants by slot, then 16 twiddles by slot
    const uint32_t max_tiles = DOWN ? kc.down_rt : kc.up_rt;
    BconvRed* s_red = reinterpret_cast<BconvRed*>(s_dyn);
    TwPair* s_tw = reinterpret_cast<TwPair*>(s_red + 4 * max_tiles);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, half = lane >> 5, wave = tid >> 6;
    const uint32_t S = 1u << (log_n - 4);
    const uint32_t u = lane & 31u, col = blockIdx.x * BCONV_COLS + u;
    const uint32_t j = blockIdx.y;  // digit (ModUp) or polynomial (ModDown)
    const uint32_t rows = level + kc.K;
    // ModUp: the digit's limbs [i0, i0 + na) are the inputs
    const uint32_t i0 = DOWN ? level : j * kc.alpha;
    const uint32_t na = DOWN ? kc.K : min(i0 + kc.alpha, level) - i0;
    const size_t lj = (size_t)(level - 1) * kc.dnum + j;
    uint64_t* item = ws.base + (size_t)blockIdx.z * ws.stride;
    // ModDown: the special rows themselves; ModUp: d's rows
    const uint64_t* __restrict__ in = item + src.off[DOWN ? j : 0];
    uint64_t* __restrict__ out = item + off_out + ((size_t)j * (DOWN ? level : rows) << log_n);
    auto mod_of = [&](uint32_t t) { return DOWN || t < level ? t : kc.L + (t - level); };
    // fold constants and first twiddles of every slot
    const uint8_t* __restrict__ tgt = DOWN ? kc.down_tgt : kc.up_tgt + lj * kc.up_rt * 4;
    auto row_of = [&](uint32_t t) { return DOWN && t >= level ? PFT_NO_ROW : t; };
    stage_red(kc, s_red, tgt, 4 * max_tiles, row_of, mod_of);
    for (uint32_t i = tid; i < 64 * max_tiles; i += blockDim.x) {
        const uint32_t t = row_of(tgt[i >> 4]);
        if (t != PFT_NO_ROW) s_tw[i] = tw[((size_t)mod_of(t) << log_n) + (i & 15u)];
    }
    // the input rows' digits
    auto word = [&](const uint64_t* __restrict__ p, uint32_t ii, uint32_t e) {
        const uint32_t off = (((DOWN ? ii : i0 + ii) << log_n) + col) * 8u;
        return *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(p + (size_t)e * S) + off);
    };
    auto slot = [&](uint32_t ii, uint32_t e) -> uint64_t& { return s_dig[(ii * 16u + e) * BCONV_COLS + u]; };
    if constexpr (SMALL) {
        // four residues of a column a thread: stages 3 and 2 over residues
        // 4 c .. 4 c + 3, through LDS, stages 1 and 0 over c, c + 4, ..
        for (uint32_t w = tid >> 5; w < 4 * na; w += blockDim.x >> 5) {
            const uint32_t ii = w >> 2, c = w & 3u;
            const uint32_t mi = DOWN ? kc.L + ii : i0 + ii;
            const DevMod md = mods[mi];
            const TwPair* __restrict__ twt = tw_inv + ((size_t)mi << log_n);
            uint64_t x[4];
            if (DOWN && src.parts > 1) {
                // two to four terms, every load in flight at once.  Integer
                // terms are below 4q, their sum below 16q.  An fp64 term
                // may be past 2q (a row pass of 9 or 12 stages ends on one
                // that does not reduce; within 3q by the butterflies'
                // bounds): two of them stay below 2^53, four may not, where
                // doubles are no longer exact, so each pair is brought
                // within q/2 before they meet.
                uint64_t y[4][4];
#pragma unroll
                for (uint32_t s = 0; s < 4; ++s)
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e)
                        y[s][e] = word(in + min(s, src.parts - 1) * src.step[j], ii, 4 * c + e);
                if (md.fp) {
#pragma clang fp contract(off)
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) {
                        const double t2 = src.parts > 2 ? as_f(y[2][e]) : 0.0, t3 = src.parts > 3 ? as_f(y[3][e]) : 0.0;
                        x[e] = as_u(freduce(as_f(y[0][e]) + as_f(y[1][e]), md.qd, md.qinv) +
                                    freduce(t2 + t3, md.qd, md.qinv));
                    }
                } else {
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) {
                        uint64_t v = y[0][e];
#pragma unroll
                        for (uint32_t s = 1; s < 4; ++s) v = s < src.parts ? v + y[s][e] : v;
                        x[e] = reduce_int(v, md);
                    }
                }
            } else {
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) x[e] = word(in, ii, 4 * c + e);
            }
            if (md.fp)
                run_phase<4, 1, 2, true, true, true>(x, c, 0u, 0u, twt, md);
            else
                run_phase<4, 1, 2, true, false, true>(x, c, 0u, 0u, twt, md);
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) slot(ii, 4 * c + e) = x[e];
        }
        __syncthreads();
        for (uint32_t w = tid >> 5; w < 8 * NKB; w += blockDim.x >> 5) {
            const uint32_t ii = w >> 2, c = w & 3u;
            uint64_t x[4] = {};
            if (ii < na) {
                const uint32_t mi = DOWN ? kc.L + ii : i0 + ii;
                const DevMod md = mods[mi];
                const TwPair* __restrict__ twt = tw_inv + ((size_t)mi << log_n);
                const TwPair hv = DOWN ? kc.down_phatinv[ii] : kc.modup_hatinv[lj * kc.alpha + ii];
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) x[e] = slot(ii, 4 * e + c);
                if (md.fp) {
                    run_phase<4, 0, 2, true, true, true>(x, c, 0u, 0u, twt, md);
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) x[e] = fp_to_u64(x[e], md.qd, md.qinv);
                } else {
                    run_phase<4, 0, 2, true, false, true>(x, c, 0u, 0u, twt, md);
                }
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) x[e] = (uint64_t)split_digits(shoup(x[e], hv.w, hv.wp, md.q));
            }
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) slot(ii, 4 * e + c) = x[e];
        }
    }
    for (uint32_t ii = tid >> 5; !SMALL && ii < 2 * NKB; ii += blockDim.x >> 5) {
        uint64_t x[16];
        if (ii < na) {
            const uint32_t mi = DOWN ? kc.L + ii : i0 + ii;
            const DevMod md = mods[mi];
            const TwPair hv = DOWN ? kc.down_phatinv[ii] : kc.modup_hatinv[lj * kc.alpha + ii];
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = word(in, ii, e);
            if constexpr (IFUSE) {
                const TwPair* __restrict__ twt = tw_inv + ((size_t)mi << log_n);
                if (md.fp) {
                    run_phase<4, 0, 4, true, true, true>(x, 0u, 0u, 0u, twt, md);
#pragma unroll
                    for (int e = 0; e < 16; ++e) x[e] = fp_to_u64(x[e], md.qd, md.qinv);
                } else {
                    run_phase<4, 0, 4, true, false, true>(x, 0u, 0u, 0u, twt, md);
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = (uint64_t)split_digits(shoup(x[e], hv.w, hv.wp, md.q));
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = 0;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) slot(ii, e) = x[e];
    }
    __syncthreads();
    const uint32_t kbs = DOWN ? kc.down_kb : kc.up_kb;
    const uint64_t* __restrict__ aop =
        (DOWN ? kc.down_aop : kc.up_aop + lj * kc.up_rt * kc.up_kb * 64) + lane;
    const uint64_t* dig = s_dig + half * 16u * BCONV_COLS + u;  // input rows 2 kb + half
    // targets V0 .. V1 - 1 of this lane's two of tile g
    auto tile = [&](uint32_t g, auto fpc, auto v0c, auto v1c) {
        constexpr bool FP = decltype(fpc)::value;
        constexpr int V0 = decltype(v0c)::value, V1 = decltype(v1c)::value;
        const BconvRed* rc = s_red + 4 * g + 2 * half;
        long av[NKB];
#pragma unroll
        for (uint32_t kb = 0; kb < NKB; ++kb) av[kb] = (long)aop[(g * kbs + kb) * 64];
        uint64_t x[V1 - V0][16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            v16i acc = {};
#pragma unroll
            for (uint32_t kb = 0; kb < NKB; ++kb)
                acc = __builtin_amdgcn_mfma_i32_32x32x16_i8(av[kb], (long)dig[(kb * 32u + t) * BCONV_COLS], acc, 0, 0, 0);
            int z[8];
            if constexpr (V0 == 0) {
                tile_digits<0>(acc, z);
                x[0][t] = fold_digits<FP, true>(z, rc[0]);
            }
            if constexpr (V1 == 2) {
                tile_digits<1>(acc, z);
                x[1 - V0][t] = fold_digits<FP, true>(z, rc[1]);
            }
            // keeps the folds here: moved down to the conditional stores they
            // would hold all 16 accumulator tiles
            if constexpr (V1 - V0 == 2)
                asm volatile("" : "+v"(x[0][t]), "+v"(x[1][t]));
            else
                asm volatile("" : "+v"(x[0][t]));
        }
#pragma unroll
        for (int v = V0; v < V1; ++v) {
            const uint32_t row = rc[v].row;
            if (row == PFT_NO_ROW) continue;
            DevMod md;
            md.q = rc[v].m;
            md.nq = rc[v].negm;
            md.rinv = rc[v].rinv;
            md.rsh = rc[v].rsh;
            md.qd = rc[v].md;
            md.qinv = rc[v].minv;
            // the fold's values are reduced (within q/2 + 1, or below q)
            run_phase<4, 0, 4, false, FP, false, true>(x[v - V0], 0u, 0u, 0u, s_tw + (4 * g + 2 * half + v) * 16, md);
            const uint32_t off = ((row << log_n) + col) * 8u;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                *reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(out + (size_t)e * S) + off) = x[v - V0][e];
        }
    };
    using i0_ = std::integral_constant<int, 0>;
    using i1_ = std::integral_constant<int, 1>;
    using i2_ = std::integral_constant<int, 2>;
    for (uint32_t k = wave; k < (SMALL ? 2 : 1) * max_tiles; k += blockDim.x >> 6) {
        const uint32_t g = SMALL ? k >> 1 : k;
        // a tile's first row is there and has the kind of the others
        const uint32_t row = __builtin_amdgcn_readfirstlane(s_red[4 * g].row);
        if (row == PFT_NO_ROW) break;
        auto run = [&](auto fpc) {
            if constexpr (!SMALL)
                tile(g, fpc, i0_{}, i2_{});
            else if (k & 1u)
                tile(g, fpc, i1_{}, i2_{});
            else
                tile(g, fpc, i0_{}, i1_{});
        };
        if (__builtin_amdgcn_readfirstlane(s_red[4 * g].fp))
            run(std::true_type{});
        else
            run(std::false_type{});
    }
}

// RESCALE's expansion fused with the transforms around it.  last_b
// (polynomial b's limb level-1) has had the row pass of its inverse transform;
// a thread takes its column u through the last pass (stages 3-0 with N^-1
// folded in), and from the 16 coefficients c forms ((c + h) mod q_last) - h
// mod q_k (h = (q_last - 1)/2 rounding, 0 floor; q_last < q_k) for its rows k
// and takes them through the first forward pass (stages 0-3; fp64 rows
// converted on entry); row k of tmp_b continues at the second pass.  Wave w of
// a workgroup takes rows w and w + 4 of its RESCALE_ROWS: a wave's row is
// uniform, so its twiddles come through the scalar cache.
constexpr uint32_t RESCALE_ROWS = 8;
__global__ __launch_bounds__(256) void k_rescale_col_b(WsRef ws, uint64_t off_last, uint64_t off_tmp, uint32_t level,
                                                       uint32_t mode, const DevMod* __restrict__ mods,
                                                       const TwPair* __restrict__ tw,
                                                       const TwPair* __restrict__ tw_inv, uint32_t log_n) {
    const uint32_t S = 1u << (log_n - 4);
    const uint32_t u = (blockIdx.x * 64u + (threadIdx.x & 63u)) * 8u;  // bytes
    const uint32_t nl = level - 1;
    const uint32_t groups = (nl + RESCALE_ROWS - 1) / RESCALE_ROWS;
    const uint32_t b = blockIdx.y / groups, g = blockIdx.y - b * groups;
    uint32_t k = g * RESCALE_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k >= nl) return;  // no barrier in this kernel
    uint64_t* item = ws.base + (size_t)blockIdx.z * ws.stride;
    const uint64_t* __restrict__ last = item + off_last + ((size_t)b << log_n);
    const DevMod ml = mods[level - 1];
    uint64_t r[16];
#pragma unroll
    for (int e = 0; e < 16; ++e)
        r[e] = *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(last + (size_t)e * S) + u);
    const TwPair* __restrict__ twl = tw_inv + ((size_t)(level - 1) << log_n);
    if (ml.fp) {
        run_phase<4, 0, 4, true, true, true>(r, 0u, 0u, 0u, twl, ml);
#pragma unroll
        for (int e = 0; e < 16; ++e) r[e] = fp_to_u64(r[e], ml.qd, ml.qinv);
    } else {
        run_phase<4, 0, 4, true, false, true>(r, 0u, 0u, 0u, twl, ml);
    }
    const uint64_t h = mode == 0 ? (ml.q - 1) / 2 : 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        r[e] += h;
        r[e] = r[e] >= ml.q ? r[e] - ml.q : r[e];
    }
    for (; k < min(nl, (g + 1) * RESCALE_ROWS); k += 4) {
        const DevMod md = mods[k];
        const TwPair* __restrict__ twt = tw + ((size_t)k << log_n);
        uint64_t x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = r[e] >= h ? r[e] - h : r[e] + md.q - h;
        if (md.fp) {
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = fp_from_u64(x[e]);
            run_phase<4, 0, 4, false, true, false, true>(x, 0u, 0u, 0u, twt, md);  // canonical inputs
        } else {
            run_phase<4, 0, 4, false, false, false, true>(x, 0u, 0u, 0u, twt, md);
        }
        uint64_t* __restrict__ orow = item + off_tmp + ((size_t)(b * nl + k) << log_n);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            *reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(orow + (size_t)e * S) + u) = x[e];
    }
}

template <bool INV>
void launch_radix(uint32_t radix, const PolyBatch& b, const DevTables& t, uint32_t log_n, uint32_t s0, bool fin,
                  bool stage, bool e8, const NttEpilogue* epi, hipStream_t st, ProfHook* prof) {
    switch (radix) {
        case 4: launch_pass<4, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 6: launch_pass<6, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 7: launch_pass<7, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 8: launch_pass<8, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 9: launch_pass<9, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 10: launch_pass<10, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 11: launch_pass<11, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        case 12: launch_pass<12, INV>(b, t, log_n, s0, fin, stage, e8, epi, st, prof); break;
        default: break;
    }
}

}  // namespace

bool ntt_supported(uint32_t log_n) { return log_n >= 12 && log_n <= 16; }

// Candidate schedules per log2 N, the default first: every radix split
// below, each with the row pass staged through LDS and direct, and each with
// 16 and with 8 residues per thread.  Windows are
// listed in forward order (stages 0.. first); every candidate has at most two
// passes, so each moves every residue through HBM at most twice.
int ntt_candidates(uint32_t log_n, NttSchedule* out, int max_out) {
    static const uint8_t c12[][2] = {{12, 0}, {8, 4}, {6, 6}, {4, 8}};
    static const uint8_t c13[][2] = {{7, 6}, {6, 7}, {4, 9}};
    static const uint8_t c14[][2] = {{7, 7}, {8, 6}, {6, 8}, {4, 10}};
    static const uint8_t c15[][2] = {{8, 7}, {7, 8}, {6, 9}, {4, 11}};
    static const uint8_t c16[][2] = {{8, 8}, {7, 9}, {6, 10}, {4, 12}};
    const uint8_t(*c)[2] = nullptr;
    int n = 0;
    switch (log_n) {
        case 12: c = c12; n = 4; break;
        case 13: c = c13; n = 3; break;
        case 14: c = c14; n = 4; break;
        case 15: c = c15; n = 4; break;
        case 16: c = c16; n = 4; break;
        default: return 0;
    }
    int k = 0;
    for (int e8 = 0; e8 < 2; ++e8)
        for (int direct = 0; direct < 2; ++direct)
            for (int i = 0; i < n; ++i) {
                if (k >= max_out) return k;
                NttSchedule s{};
                s.n_passes = c[i][1] ? 2 : 1;
                s.radix[0] = c[i][0];
                s.radix[1] = c[i][1];
                s.flags = (direct ? NTT_DIRECT_ROWS : 0u) | (e8 ? NTT_E8 : 0u);
                out[k++] = s;
            }
    return k;
}

bool ntt_schedule_valid(uint32_t log_n, const NttSchedule& s) {
    NttSchedule c[32];
    const int n = ntt_candidates(log_n, c, 32);
    for (int i = 0; i < n; ++i)
        if (c[i].n_passes == s.n_passes && c[i].radix[0] == s.radix[0] && c[i].radix[1] == s.radix[1] &&
            c[i].flags == s.flags)
            return true;
    return false;
}

// fold constants and 16 twiddles for every slot
static uint32_t bconv_col_dyn_lds(uint32_t tiles) {
    return 4 * tiles * (uint32_t)(sizeof(BconvRed) + 16 * sizeof(TwPair));
}
// A workgroup may take a compute unit's whole 160 KB.  The largest, 12 inputs
// and 72 slots, takes 70.5: two still share a compute unit, as the registers
// allow for any size.
bool bconv_col_supported(uint32_t log_n, uint32_t nkb, uint32_t tiles) {
    return log_n >= 9 && nkb <= 6 && 2 * nkb * 16 * BCONV_COLS * 8 + bconv_col_dyn_lds(tiles) <= 160 * 1024;
}

// Up to two workgroups of 32 columns a compute unit, the eight-wave form with
// four threads a column: one item at N = 2^15, level 16 (256 and 128
// workgroups) 18.0 -> 16.1 us for ModUp's and 16.0 -> 14.6 for ModDown's.
// With more of them the threads that only one of the two phases has work for
// cost more than the shorter chain gives.  The line at 128, 256, 512, 1024 and
// 2048 workgroups: one bag-of-words document at N = 2^15 2704, 2604, 2578, 2578
// and 2577 us, six documents' predict step 4879, 4878, 4827, 4837 and 4863, five
// rotations at N = 2^16 351 up to 1024 and 358.  Parts are summed by that form.
constexpr uint64_t BCONV_SMALL_BLOCKS = 512;
static bool bconv_col_small(uint32_t log_n, uint32_t groups, uint32_t n, uint32_t parts) {
    return parts > 1 || (((uint64_t)n * groups << log_n) / (16 * BCONV_COLS)) <= BCONV_SMALL_BLOCKS;
}
uint32_t bconv_col_variant(uint32_t log_n, uint32_t nkb, uint32_t groups, uint32_t n, uint32_t parts, bool ifuse) {
    return 64u + nkb + (ifuse ? 16u : 0u) + (ifuse && bconv_col_small(log_n, groups, n, parts) ? 32u : 0u);
}
template <bool DOWN, bool IFUSE>
static void launch_bconv_col(uint32_t nkb, dim3 grid, hipStream_t st, WsRef ws, const BconvIn& in, uint64_t off_out,
                             uint32_t level, const KsConsts& kc, const DevTables& t, uint32_t log_n) {
    const uint32_t tiles = DOWN ? kc.down_rt : kc.up_rt, lds = bconv_col_dyn_lds(tiles);
    const bool small = bconv_col_small(log_n, grid.y, grid.z, in.parts);
    // four waves take about two tiles each; where that leaves compute units
    // without a second workgroup, eight waves a workgroup take one each, and
    // sixteen where a workgroup has a compute unit to itself and more than
    // eight tiles (one HMULT at N = 2^12, 36 limbs in three digits, 13 tiles:
    // 74.9 -> 65.7 us; 68.2 through separate launches)
    const bool alone = IFUSE && small && tiles > 8 && grid.x * grid.y * grid.z <= 256;
    const uint32_t threads = alone ? 1024 : small ? 512 : 256;
#define PFT_BCONV_COL(K)                                                                                     \
    case K:                                                                                                  \
        if (IFUSE && small)                                                                                  \
            hipLaunchKernelGGL((k_bconv_col_b<K, DOWN, IFUSE, IFUSE>), grid, dim3(threads), lds, st, ws, in, \
                               off_out, level, kc, t.mods, t.tw_fwd, t.tw_inv, log_n);                       \
        else                                                                                                 \
            hipLaunchKernelGGL((k_bconv_col_b<K, DOWN, IFUSE, false>), grid, dim3(threads), lds, st, ws, in, \
                               off_out, level, kc, t.mods, t.tw_fwd, t.tw_inv, log_n);                       \
        break;
    switch (nkb) {
        PFT_BCONV_COL(1)
        PFT_BCONV_COL(2)
        PFT_BCONV_COL(3)
        PFT_BCONV_COL(4)
        PFT_BCONV_COL(5)
        PFT_BCONV_COL(6)
        default: break;
    }
#undef PFT_BCONV_COL
}

void launch_modup_col_b(uint32_t n, WsRef ws, uint64_t off_d, uint64_t off_ext, uint32_t level, const KsConsts& kc,
                        const DevTables& t, uint32_t log_n, bool ifuse, hipStream_t st) {
    const uint32_t beta = (level + kc.alpha - 1) / kc.alpha;
    const uint32_t nkb = (std::min(kc.alpha, level) + 1) / 2;
    const dim3 grid((1u << log_n) / (16 * BCONV_COLS), beta, n);
    const BconvIn in{{off_d, off_d}, {0, 0}, 1};
    if (ifuse)
        launch_bconv_col<false, true>(nkb, grid, st, ws, in, off_ext, level, kc, t, log_n);
    else
        launch_bconv_col<false, false>(nkb, grid, st, ws, in, off_ext, level, kc, t, log_n);
}

void launch_moddown_col_b(uint32_t n, WsRef ws, const BconvIn& in, uint64_t off_conv, uint32_t level,
                          const KsConsts& kc, const DevTables& t, uint32_t log_n, bool ifuse, hipStream_t st) {
    const dim3 grid((1u << log_n) / (16 * BCONV_COLS), 2, n);
    if (ifuse)
        launch_bconv_col<true, true>((kc.K + 1) / 2, grid, st, ws, in, off_conv, level, kc, t, log_n);
    else
        launch_bconv_col<true, false>((kc.K + 1) / 2, grid, st, ws, in, off_conv, level, kc, t, log_n);
}

void launch_rescale_col_b(uint32_t n, WsRef ws, uint64_t off_last, uint64_t off_tmp, uint32_t level, uint32_t mode,
                          const DevTables& t, uint32_t log_n, hipStream_t st) {
    const uint32_t groups = (level - 1 + RESCALE_ROWS - 1) / RESCALE_ROWS;
    hipLaunchKernelGGL(k_rescale_col_b, dim3((1u << log_n) / 1024, 2 * groups, n), dim3(256), 0, st, ws, off_last,
                       off_tmp, level, mode, t.mods, t.tw_fwd, t.tw_inv, log_n);
}

void launch_ntt(const PolyBatch& b, const DevTables& t, uint32_t log_n, bool inverse, const NttSchedule& s,
                hipStream_t st, ProfHook* prof, const NttEpilogue* epi, uint32_t first) {
    if (b.n_polys == 0 || b.n_limbs == 0 || s.n_passes == 0 || s.n_passes > 3) return;
    uint32_t s0[4];
    uint32_t acc = 0;
    for (uint32_t p = 0; p < s.n_passes; ++p) {
        s0[p] = acc;
        acc += s.radix[p];
    }
    if (acc != log_n) return;
    const bool stage = (s.flags & NTT_DIRECT_ROWS) == 0;
    const bool e8 = (s.flags & NTT_E8) != 0;
    if (!inverse) {
        for (uint32_t p = first; p < s.n_passes; ++p)
            launch_radix<false>(s.radix[p], b, t, log_n, s0[p], p + 1 == s.n_passes, stage, e8,
                                p + 1 == s.n_passes ? epi : nullptr, st, prof);
    } else {
        for (uint32_t p = s.n_passes; p-- > first;)
            launch_radix<true>(s.radix[p], b, t, log_n, s0[p], p == 0, stage, e8, nullptr, st, prof);
    }
}

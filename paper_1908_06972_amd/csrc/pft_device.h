// pft_device.h -- device-side data structures and 64-bit modular arithmetic
// for gfx950.  Residues are uint64 below primes q < 2^60.
//
// Three reductions are used, chosen per operand kind:
//   * Shoup (constant multiplier w with w' = floor(w 2^64 / q)): twiddles and
//     per-prime constants; result in [0, 2q) before the optional final
//     subtraction.
//   * Montgomery REDC (R = 2^64) for sums of products whose constant factor
//     was stored pre-multiplied by R: base-conversion matrices, switching keys.
//   * Barrett (mu = floor(2^(2b)/q), b = bit length of q) for products of two
//     variable residues (the HMUL tensor, NTT-domain plaintext products).
// All three are built from 64x64 products that the compiler lowers to
// v_mul_lo_u32 / v_mul_hi_u32 / v_mad_u64_u32, which issue at full rate on
// gfx950.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define PFT_MAX_POLYS 128  // polynomials per NTT launch
#define PFT_MAX_ITEMS 64   // ciphertexts per batched launch
#define PFT_SMALL_POLYS 8  // operands of the small elementwise kernels

struct DevMod {
    uint64_t q;
    uint64_t two_q;
    uint64_t mu;          // floor(2^(2b) / q)
    uint64_t mont_neg_qinv;  // -q^-1 mod 2^64
    uint64_t n_inv, n_inv_sh;      // N^-1 mod q and its Shoup companion
    uint64_t last_inv, last_inv_sh; // psi^-brv(1) * N^-1: fused last inverse stage
    uint32_t bits;
    uint32_t fp;          // 1 if q < 2^50: the NTT runs its butterflies in fp64
    uint64_t nq;          // 2^64 - q
    uint32_t rinv, rsh;   // floor(2^(bits+31) / q) and bits - 33, bits >= 51 (reduce_int)
    // fp64 forms for the NTT when fp != 0: q, 1/q, and each constant c with
    // its quotient c/q, all rounded to nearest (c < q < 2^50 is exact).
    double qd, qinv;
    double n_inv_d, n_inv_q;
    double last_inv_d, last_inv_q;
};

// One twiddle.  Integer limbs: w and its Shoup companion floor(w 2^64 / q).
// fp64 limbs (DevMod::fp): the bit patterns of the doubles w and w/q.
struct TwPair {
    uint64_t w;
    uint64_t wp;
};

// A set of RNS polynomials processed by one NTT launch.  Limb i (0 <= i <
// n_limbs) of polynomial p sits at row r = i + (i >= gap_at[p] ? gap_len[p] : 0)
// of ptr[p] (rows are N words apart); row r is reduced modulo modulus index
// r < split ? off0 + r : off1 + (r - split).  The first pass of a transform
// reads each row from src_delta words past it (0: in place) and writes it in
// place.
struct PolyBatch {
    uint64_t* ptr[PFT_MAX_POLYS];
    uint8_t gap_at[PFT_MAX_POLYS];
    uint8_t gap_len[PFT_MAX_POLYS];
    uint32_t n_polys;
    uint32_t n_limbs;
    uint32_t split, off0, off1;
    int64_t src_delta;
};

__device__ __forceinline__ uint32_t pb_row(const PolyBatch& b, uint32_t p, uint32_t i) {
    return i + (i >= b.gap_at[p] ? (uint32_t)b.gap_len[p] : 0u);
}
__device__ __forceinline__ uint32_t pb_mod(const PolyBatch& b, uint32_t row) {
    return row < b.split ? b.off0 + row : b.off1 + (row - b.split);
}

// Up to eight polynomials of n_limbs consecutive rows starting at row
// `first`, same modulus rule as PolyBatch (small elementwise launches).
struct SmallBatch {
    uint64_t* ptr[PFT_SMALL_POLYS];
    uint32_t n_polys;
    uint32_t n_limbs;
    uint32_t first;
    uint32_t split, off0, off1;
};
__device__ __forceinline__ uint32_t sb_mod(const SmallBatch& b, uint32_t row) {
    return row < b.split ? b.off0 + row : b.off1 + (row - b.split);
}

// Per-ciphertext device pointers of a batched launch.
struct ItemPtrs {
    uint64_t* p[PFT_MAX_ITEMS];
};

__device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) { return __umul64hi(a, b); }

// a*w mod q in [0, 2q) for any a < 2^64 (Shoup).
__device__ __forceinline__ uint64_t shoup_lazy(uint64_t a, uint64_t w, uint64_t wp, uint64_t q) {
    return a * w - mulhi64(a, wp) * q;
}
__device__ __forceinline__ uint64_t shoup(uint64_t a, uint64_t w, uint64_t wp, uint64_t q) {
    uint64_t r = shoup_lazy(a, w, wp, q);
    return r >= q ? r - q : r;
}

// ---- 64-bit products as chains of v_mad_u64_u32 (32 x 32 + 64, full rate)
// Written out by hand: from __umul64hi and 64-bit operators the compiler
// spends more instructions on zero-extending the halves (moves) and on
// carries (subtractions with borrow, each waiting on the mask) than on the
// products.
__device__ __forceinline__ uint64_t mad32(uint32_t a, uint32_t b, uint64_t c) { return (uint64_t)a * b + c; }
__device__ __forceinline__ uint32_t lo32(uint64_t v) { return (uint32_t)v; }
__device__ __forceinline__ uint32_t hi32(uint64_t v) { return (uint32_t)(v >> 32); }
// p + h modulo 2^64 in one instruction (a 64-bit add would need h zero-extended to a register pair)
__device__ __forceinline__ uint64_t add32(uint64_t p, uint32_t h) {
    uint64_t r;
    asm("v_mad_u64_u32 %0, vcc, %1, 1, %2" : "=v"(r) : "v"(h), "v"(p) : "vcc");
    return r;
}
// c + a b + k n modulo 2^64
__device__ __forceinline__ uint64_t mad64x2(uint64_t c, uint64_t a, uint64_t b, uint64_t k, uint64_t n) {
    c = mad32(lo32(k), lo32(n), mad32(lo32(a), lo32(b), c));
    const uint32_t hi = hi32(c) + lo32(a) * hi32(b) + hi32(a) * lo32(b) + lo32(k) * hi32(n) + hi32(k) * lo32(n);
    return ((uint64_t)hi << 32) | lo32(c);
}
// x + r modulo 2^64 with r = a w mod q + e q in [0, 4q), any a < 2^64, w < q
// with wp = floor(w 2^64 / q), nq = 2^64 - q: the quotient is Shoup's with
// the low halves' product and the low parts of the cross products dropped
// (at most 3 below floor(a w / q)).  13 instructions.
__device__ __forceinline__ uint64_t shoup_add4(uint64_t x, uint64_t a, uint64_t w, uint64_t wp, uint64_t nq) {
    const uint64_t k = add32(add32(mad32(hi32(a), hi32(wp), 0), __umulhi(hi32(a), lo32(wp))),
                             __umulhi(lo32(a), hi32(wp)));
    return mad64x2(x, a, w, k, nq);
}
// x - k q in [0, 2q) for any x < 2^64, q of at least 51 bits: k = floor of
// (x's high half times rinv) 2^-(bits-1) never exceeds x / q and is less than
// 1 + 2^-16 below it.  Five instructions against ten for two conditional
// subtractions.
__device__ __forceinline__ uint64_t reduce_int(uint64_t x, const DevMod& m) {
    const uint32_t k = __umulhi(hi32(x), m.rinv) >> m.rsh;
    const uint64_t c = mad32(k, lo32(m.nq), x);
    return ((uint64_t)(hi32(c) + k * hi32(m.nq)) << 32) | lo32(c);
}
// acc + (x k + m q) 2^-64, m = -x k q^-1 mod 2^64: x k 2^-64 mod q in [0, 2q)
// added to acc, for any x < 2^64 and k < q (Montgomery's reduction without
// its final subtraction).
__device__ __forceinline__ uint64_t mont_add2(uint64_t acc, uint64_t x, uint64_t k, const DevMod& md) {
    const uint64_t a = mad32(lo32(x), lo32(k), 0);
    const uint64_t b = add32(mad32(hi32(x), lo32(k), 0), hi32(a));
    const uint64_t c = add32(mad32(lo32(x), hi32(k), 0), lo32(b));
    const uint32_t l0 = lo32(a), l1 = lo32(c);  // x k = d 2^64 + l1 2^32 + l0
    const uint64_t d = add32(add32(mad32(hi32(x), hi32(k), acc), hi32(b)), hi32(c));
    const uint64_t n = md.mont_neg_qinv, q = md.q;
    const uint64_t m0 = mad32(l0, lo32(n), 0);
    const uint32_t ml = lo32(m0), mh = hi32(m0) + l0 * hi32(n) + l1 * lo32(n);
    const uint64_t f = add32(mad32(mh, lo32(q), 0), __umulhi(ml, lo32(q)));
    const uint64_t g = add32(mad32(ml, hi32(q), 0), lo32(f));
    const uint64_t h = add32(add32(mad32(mh, hi32(q), d), hi32(f)), hi32(g));
    return add32(h, (l0 | l1) != 0 ? 1u : 0u);
}

// ---- fp64 arithmetic for primes q < 2^50 (the NTT butterflies, base-conversion folds)
//
// A residue is held as an integer-valued double of either sign; every value
// stays an integer below 2^53 in magnitude, so sums and differences are exact.
// fmulmod(a, w) returns a w - k q with k = rint(fl(a fl(w/q))): the product
// a w is split exactly into hi + lo (hi = fl(a w), lo = fma(a, w, -hi)); then
// fma(-k, q, hi) is exact because the true value is an integer of magnitude
// below 2^53, and adding lo is exact for the same reason.  The quotient is off
// from a w / q by at most 1/2 + |a| 2^-52 (two roundings), so with |a| <= c q
// and q < 2^50 the result lies within (1/2 + c/4) q of zero.  freduce(x) =
// x - rint(x/q) q lies within q/2 (+ a vanishing error) for the magnitudes
// used here.  Forward butterfly with X reduced: inputs within B q give outputs
// within (1 + B/4) q; inverse with X + Y reduced: within max(1/2, 1/2 + B/2) q.
// The lazy schedules of the NTT keep every magnitude below 4.5q < 2^53.
__device__ __forceinline__ double as_f(uint64_t v) { return __builtin_bit_cast(double, v); }
__device__ __forceinline__ uint64_t as_u(double v) { return __builtin_bit_cast(uint64_t, v); }

__device__ __forceinline__ double fmulmod(double a, double w, double wq, double q) {
#pragma clang fp contract(off)
    const double hi = a * w;
    const double lo = __builtin_fma(a, w, -hi);
    const double k = __builtin_rint(a * wq);
    return __builtin_fma(-k, q, hi) + lo;
}
__device__ __forceinline__ double freduce(double x, double q, double qinv) {
#pragma clang fp contract(off)
    return __builtin_fma(-__builtin_rint(x * qinv), q, x);
}

// u64 below 2^52 -> double: the bits of 2^52 + v, minus 2^52.
__device__ __forceinline__ uint64_t fp_from_u64(uint64_t v) {
#pragma clang fp contract(off)
    return as_u(as_f(v | 0x4330000000000000ull) - 4503599627370496.0);
}
// double residue -> canonical u64 in [0, q): reduce to within q/2, lift the
// negative half by q, then read the mantissa of 2^52 + r.
__device__ __forceinline__ uint64_t fp_to_u64(uint64_t v, double q, double qinv) {
#pragma clang fp contract(off)
    double r = freduce(as_f(v), q, qinv);
    r = r < 0.0 ? r + q : r;
    return as_u(r + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
}

// (hi:lo) * 2^-64 mod q for hi:lo < q * 2^64; result in [0, q).
__device__ __forceinline__ uint64_t mont_redc(uint64_t lo, uint64_t hi, uint64_t q, uint64_t neg_qinv) {
    uint64_t m = lo * neg_qinv;
    uint64_t r = hi + mulhi64(m, q) + (lo != 0 ? 1u : 0u);
    return r >= q ? r - q : r;
}

// 128-bit accumulator helpers
struct Acc128 {
    uint64_t lo, hi;
};
__device__ __forceinline__ void mac128(Acc128& acc, uint64_t a, uint64_t b) {
    uint64_t lo = a * b;
    uint64_t hi = mulhi64(a, b);
    acc.lo += lo;
    acc.hi += hi + (acc.lo < lo ? 1u : 0u);
}

// a*b mod q for a, b < q (Barrett, HAC 14.42 with base 2).
__device__ __forceinline__ uint64_t mul_barrett(uint64_t a, uint64_t b, const DevMod& m) {
    uint64_t lo = a * b, hi = mulhi64(a, b);
    uint32_t bits = m.bits;
    uint64_t x1 = (lo >> (bits - 1)) | (hi << (65 - bits));
    uint64_t plo = x1 * m.mu, phi = mulhi64(x1, m.mu);
    uint64_t qh = (plo >> (bits + 1)) | (phi << (63 - bits));
    uint64_t r = lo - qh * m.q;
    if (r >= m.q) r -= m.q;
    if (r >= m.q) r -= m.q;
    return r;
}

__device__ __forceinline__ uint64_t add_mod(uint64_t a, uint64_t b, uint64_t q) {
    uint64_t r = a + b;
    return r >= q ? r - q : r;
}
__device__ __forceinline__ uint64_t sub_mod(uint64_t a, uint64_t b, uint64_t q) {
    return a >= b ? a - b : a + q - b;
}

// index of the bit-reversal of k over log_n bits
__device__ __forceinline__ uint32_t brev_n(uint32_t k, uint32_t log_n) {
    return __brev(k) >> (32 - log_n);
}

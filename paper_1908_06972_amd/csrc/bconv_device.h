// bconv_device.h -- device helpers of the exact base conversion on the
// matrix cores (ModUp / ModDown of hybrid key switching), shared by the
// conversion kernels and the ModUp kernel fused with the first transform pass.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pft_device.h"
#include "pft_kernels.h"

namespace {

// ---- base conversion on the matrix cores -------------------------------
// The contraction y_t = sum_i x_i h_{i,t} mod m_t in signed base-256 digits
// (operand tables and the exactness bound are built on the host):
// Z_{t,b} = sum_{i,a} x_{i,a} v_{(i,a),t,b} by v_mfma_i32_32x32x16_i8 with the
// constant digits as A (32 rows = 4 targets x 8 digits b) and the input
// digits as B (32 columns = 32 coefficients, k = 8 i_local + a), then
// y_t = sum_b 256^b Z_{t,b} mod m_t on the VALU.
typedef int v16i __attribute__((ext_vector_type(16)));

// balanced base-256 digits of v < 2^60 as packed int8: v + 0x80..80 carries
// exactly as the balanced digits do, and each biased byte minus 128 is the
// digit (the same bits as the byte XOR 0x80)
__device__ __forceinline__ long split_digits(uint64_t v) {
    return (long)((v + 0x8080808080808080ull) ^ 0x8080808080808080ull);
}

// sum_b 256^b Z_b mod m for the 8 digit sums of one target (|Z_b| < 2^21).
// lo = sum_{b<4} 256^b Z_b and hi = sum_{b>=4} 256^(b-4) Z_b are integers
// below 2^46 in magnitude, exact in fp64; the value is lo + 2^32 hi.
//  m < 2^50: its quotient k = rint((lo + 2^32 hi) / m), below 2^28 in
//    magnitude and taken from a sum and a product rounded to 53 bits, is
//    exact to 1/2 + 2^-24; 2^32 hi - k m is an integer below 2^50, so fma
//    gives it exactly, and adding lo leaves the remainder within
//    (1/2 + 2^-24) m of zero.  (Z_7 = 0: the constants are below 2^50.)
//  m >= 2^50: the quotient k = round((lo + 2^32 hi) / m) has |k| < 2^29 and
//    comes from fp64 (error below 2^-21); the remainder is formed exactly in
//    integers mod 2^64 as (lo + 2^32 hi + 2^30 m) - (k + 2^30) m, which lies
//    within (1/2 + 2^-21) m of zero, then one conditional add of m.
// RAW: for m < 2^50 return the bits of the remainder itself (an integer of
// magnitude at most m/2 + 1), the input form of the fp64 transform passes,
// instead of the canonical u64.
template <bool FP, bool RAW>
__device__ __forceinline__ uint64_t fold_digits(const int (&z)[8], const BconvRed& rc) {
#pragma clang fp contract(off)
    const double lo = __builtin_fma((double)(z[3] * 256 + z[2]), 65536.0, (double)(z[1] * 256 + z[0]));
    if constexpr (FP) {
        const double hi = __builtin_fma((double)z[6], 65536.0, (double)(z[5] * 256 + z[4]));
        const double k = __builtin_rint(__builtin_fma(hi, 0x1p32, lo) * rc.minv);
        double y = __builtin_fma(-k, rc.md, hi * 0x1p32) + lo;
        if (RAW) return as_u(y);
        y = y < 0.0 ? y + rc.md : y;  // [0, m)
        return as_u(y + 0x1p52) ^ 0x4330000000000000ull;
    } else {
        const double hi = __builtin_fma((double)(z[7] * 256 + z[6]), 65536.0, (double)(z[5] * 256 + z[4]));
        const double s = __builtin_fma(hi, 0x1p32, lo);
        const uint32_t k = (uint32_t)__builtin_fma(s, rc.minv, 0x1p30 + 0.5);  // floor: k + 2^30
        // two's complement of an integer |v| < 2^51 in the low bits of v + 1.5 2^52
        const uint64_t lo64 = as_u(lo + 0x1.8p52) - 0x4338000000000000ull;
        const uint32_t hi32 = (uint32_t)as_u(hi + 0x1.8p52);
        const uint64_t r = lo64 + ((uint64_t)hi32 << 32) + rc.cq0 + (uint64_t)k * rc.negm;
        return (int64_t)r < 0 ? r + rc.m : r;
    }
}

// the two targets of this lane in accumulator tile acc: u = 0, 1
template <int U>
__device__ __forceinline__ void tile_digits(const v16i& acc, int (&z)[8]) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        z[b] = acc[4 * U + b];
        z[4 + b] = acc[8 + 4 * U + b];
    }
}

// The fold constants of n slots (targets in tile order) into LDS, each with
// its target row, so that a slot's reads are short-latency.  row_of(tgt) is
// the target row of a list entry or PFT_NO_ROW, mod_of(row) its modulus index.
template <class R, class M>
__device__ __forceinline__ void stage_red(const KsConsts& kc, BconvRed* s_red, const uint8_t* __restrict__ tgt,
                                          uint32_t n, R&& row_of, M&& mod_of) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t row = row_of(tgt[i]);
        BconvRed r = kc.red[row == PFT_NO_ROW ? 0u : mod_of(row)];
        r.row = row;
        s_red[i] = r;
    }
}

}  // namespace

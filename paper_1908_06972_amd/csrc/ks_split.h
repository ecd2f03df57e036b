// ks_split.h -- how the launches of a key switch that cannot fill the chip
// are split, and where the split sums lie.  Plain C++, so that the rule and
// the layout can be checked without a GPU; the kernels address the rows
// through the same functions.
#pragma once
#include <stdint.h>

#include <algorithm>

// Launches of at most this many words (rows times N, all items) take the
// 4-residue forms: below the line the 8-residue forms' waves (8 per SIMD, in
// two rounds at their registers) do not hide the passes' latency, far above it
// they read each twiddle half as often.  Launches of 2^22.4 to 2^22.6 words
// with the line at 2^22 and at 2^23: four HMULTs at N = 2^16, level 24, 466 and
// 443 us, eight at level 12 401 and 373, 24 at N = 2^15, level 8, 381 and 356;
// five rotations at N = 2^16, level 17, 355 either way, but 401 with the
// 8-residue form where the helper stream has the hardware queue of the
// context's own.  At 2^24 a chain of 16 products at N = 2^16 takes 27.87 ms,
// 27.35 at 2^23, and 16 HMULTs at level 24 1693 us with 4 residues, 1565 with 8.
#define KS_SMALL_WORDS (1ull << 23)
inline bool ks_small(uint32_t n, uint32_t rows, uint32_t log_n) {
    return ((uint64_t)n * rows << log_n) <= KS_SMALL_WORDS;
}

// How a key switch whose launches cannot fill the chip spreads its integer
// rows (ks_split).  parts > 1: each special row is taken by `parts`
// workgroups a tile, each with `group` digits, whose sums go through the
// inverse row pass by themselves; ModDown's conversion adds the parts.  early:
// the digits of the integer ciphertext rows (but their own) are taken in the
// special rows' launch, in the same parts, and the last launch adds their
// sums.  In either case (packed) the sums lie in rows that the fused path has
// no other use for: part s of row t's polynomial 0 over row t of the group's
// first digit, s group (ext, which only that workgroup reads), of its
// polynomial 1 at the row of acc ([2 (level + K)] rows) that ks_special_row1
// or ks_early_row1 gives.  Otherwise a special row's sums lie in its own rows
// of acc.
struct KsSplit {
    uint32_t parts, group;
    bool early;
    constexpr bool packed() const { return parts > 1 || early; }
};
// polynomial 1 of special row k (0..K-1), and of the integer ciphertext row
// that is the e-th of them
constexpr uint32_t ks_special_row1(uint32_t K, uint32_t k, uint32_t s) { return s * K + k; }
constexpr uint32_t ks_early_row1(uint32_t K, uint32_t parts, uint32_t e, uint32_t s) { return parts * (K + e) + s; }

// ints: integer rows (q >= 2^50) among the `level` ciphertext rows.
//
// parts: a tile of a special row costs a workgroup ceil(beta / parts) digits'
// passes and two of the inverse (splitting repeats the latter), a round of
// workgroups being one per compute unit (two of the 1024-word tiles' four
// waves).  At N = 2^15, level 16, one item (64 tiles of 60-bit rows, four
// digits) the launch takes 15.6 us in four parts, 23.3 in one, and ModDown's
// conversion 16.0 instead of 14.1; one HMULT at N = 2^16, level 24 (96 tiles,
// two parts) 172 -> 161 us.
// early: where the last launch is a single round, its few integer rows are
// what it ends with: 28.7 -> 24.1 us at N = 2^15, level 16, the special rows'
// launch 15.6 -> 17.5.  With more rounds they hide (six items: 5028 us without,
// 5065 with, for a predict step).
inline KsSplit ks_split(uint32_t n, uint32_t level, uint32_t alpha, uint32_t K, uint32_t ints, uint32_t log_n) {
    const uint32_t beta = (level + alpha - 1) / alpha;
    KsSplit s{1, beta, false};
    if (beta < 2 || !ks_small(n, std::max(level, K), log_n)) return s;
    const uint32_t tile_log = std::max(log_n - 4, 10u), slots = tile_log == 10 ? 512 : 256;
    auto rounds = [&](uint64_t rows) { return (uint32_t)((((n * rows) << log_n >> tile_log) + slots - 1) / slots); };
    s.early = ints > 0 && ints <= K && rounds(level) == 1;
    if (!s.early) ints = 0;
    uint32_t best = ~0u;
    for (uint32_t parts = 1; parts <= std::min(beta, 4u); ++parts) {
        const uint32_t group = (beta + parts - 1) / parts;
        // every part has a digit, and polynomial 1's parts fit acc
        if ((parts - 1) * group >= beta || parts * (K + ints) > 2 * (level + K)) continue;
        const uint32_t cost = rounds(K * parts) * (group + 2);
        if (cost < best) {
            best = cost;
            s.parts = parts;
            s.group = group;
        }
    }
    return s;
}

"""The split rule and the row layout of a key switch's small launches
(csrc/ks_split.h, plain C++) compiled for the host with g++."""

import ctypes
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <set>
#include <tuple>
#include <vector>
#include "ks_split.h"

extern "C" uint32_t split(uint32_t n, uint32_t level, uint32_t alpha, uint32_t K, uint32_t ints, uint32_t log_n) {
    const KsSplit s = ks_split(n, level, alpha, K, ints, log_n);
    return s.parts | s.group << 8 | (s.early ? 1u : 0u) << 16;
}

// Marks every row that a launch's workgroups store a sum in; false where two
// of them share a row or one lies outside its area.
static bool disjoint(uint32_t level, uint32_t alpha, uint32_t K, uint32_t ints, const KsSplit& s) {
    const uint32_t rows = level + K, beta = (level + alpha - 1) / alpha, group = s.parts > 1 ? s.group : beta;
    std::vector<char> ext(beta * rows, 0), acc(2 * rows, 0);
    auto take = [](std::vector<char>& v, uint32_t r) {
        if (r >= v.size() || v[r]) return false;
        return v[r] = 1, true;
    };
    bool ok = true;
    for (uint32_t p = 0; p < s.parts; ++p) {
        for (uint32_t k = 0; k < K; ++k) {
            ok &= s.packed() ? take(ext, p * group * rows + level + k) : take(acc, level + k);
            ok &= take(acc, s.packed() ? ks_special_row1(K, k, p) : rows + level + k);
        }
        for (uint32_t e = 0; s.early && e < ints; ++e) {  // whichever rows these are
            ok &= take(ext, p * group * rows + e);
            ok &= take(acc, ks_early_row1(K, s.parts, e, p));
        }
    }
    return ok;
}

// Every parameter set's shapes of one ring: the number of distinct layouts,
// of those with early rows and one part, and of those that overlap.
extern "C" void walk(uint32_t log_n, uint32_t* out) {
    std::set<std::tuple<uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, bool>> seen;
    out[0] = out[1] = out[2] = 0;
    for (uint32_t alpha = 1; alpha <= 12; ++alpha)
        for (uint32_t K = 1; K <= 12; ++K)
            for (uint32_t level = 1; level + K <= 64 && (level + alpha - 1) / alpha <= 8; ++level)
                for (uint32_t ints = 0; ints <= level; ++ints)
                    for (uint32_t n = 1; n <= 64; ++n) {
                        const KsSplit s = ks_split(n, level, alpha, K, ints, log_n);
                        if (!seen.insert({alpha, K, level, ints, s.parts, s.group, s.early}).second) continue;
                        ++out[0];
                        out[1] += s.early && s.parts == 1;
                        out[2] += !disjoint(level, alpha, K, ints, s);
                    }
}
"""

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "s.cpp"), os.path.join(d, "s.so")
            with open(src, "w") as f:
                f.write(SOURCE)
            subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I",
                                   os.path.join(ROOT, "paper_1908_06972_amd", "csrc"), src, "-o", so])
            _lib = ctypes.CDLL(so)
    return _lib


def split(n, level, alpha, K, ints, log_n):
    """(parts, digits a part, early) of a key switch of n items."""
    v = lib().split(n, level, alpha, K, ints, log_n)
    return v & 255, v >> 8 & 255, bool(v >> 16)


def walk(log_n):
    out = (ctypes.c_uint32 * 3)()
    lib().walk(log_n, out)
    return tuple(out)

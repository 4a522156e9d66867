"""The quotient of a field difference by a grid spacing, which the float32
path forms from the spacing's reciprocal, is the correctly rounded x / d: the
library's own inline functions, compiled for the host, against the division.
"""
import ctypes
import os
import subprocess

import pytest

from paper_2510_22221_amd import build as B

SRC = r"""
#include "mpx_internal.h"
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
static uint64_t s;
static uint64_t rnd() { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
static float flt(int lo, int hi) { // random significand and sign, exponent in [lo, hi]
    const float m = 1.0f + (float)(rnd() >> 41) * 0x1p-23f;
    return std::ldexp(rnd() & 1 ? m : -m, lo + (int)(rnd() % (uint64_t)(hi - lo + 1)));
}
static bool wrong(double x, double d) {
    double rd, rdl;
    mpx::spacing_parts(d, rd, rdl);
    return mpx::spacing_quotient(x, d, rd, rdl) != x / d;
}
// differences of floats near each other and far apart, over the whole range of
// exponents; spacings with random significands, from 2^-50 to 2^20
extern "C" long long mismatches(long long n, uint64_t seed) {
    s = seed;
    long long bad = 0;
    for (long long t = 0; t < n; t++) {
        const double d = (1.0 + (double)(rnd() >> 12) * 0x1p-52) * std::ldexp(1.0, -50 + (int)(rnd() % 71));
        const float a = flt(-149, 127), b = t & 1 ? a * (1.0f + (float)(rnd() % 64) * 0x1p-23f) : flt(-149, 127);
        if (!std::isfinite(b)) continue;
        const double x = (double)a - (double)b;
        bad += wrong(x, d);
    }
    // the ends of the range of x, by spacings that give a chosen quotient and
    // their neighbours
    const float ends[] = {0x1p-149f, 3 * 0x1p-149f, 0x1p-126f, 1.0f, std::numeric_limits<float>::max()};
    for (float a : ends)
        for (int q = 0; q < 2000; q++) {
            const double mid = (1.0 + (double)(rnd() >> 12) * 0x1p-52) * std::ldexp(1.0, (int)(rnd() % 40) - 20);
            double d = (double)a / mid;
            d = std::ldexp(d, -std::ilogb(d) - 20);
            for (double e : {d, std::nextafter(d, 0.0), std::nextafter(d, 1.0)}) bad += wrong(a, e) + wrong(-a, e);
        }
    return bad;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("spacing")
    src, so = d / "spacing.hip", d / "spacing.so"
    src.write_text(SRC)
    subprocess.check_call([B.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-mfma", "-fPIC",
                           "-shared", "-ffp-contract=off", "-I", B.CSRC, "-o", str(so), str(src)])
    L = ctypes.CDLL(os.fspath(so))
    L.mismatches.restype = ctypes.c_longlong
    L.mismatches.argtypes = [ctypes.c_longlong, ctypes.c_uint64]
    return L


@pytest.mark.parametrize("seed", [1, 22221])
def test_quotient_is_correctly_rounded(lib, seed):
    assert lib.mismatches(10_000_000, seed) == 0

"""csrc/bounds.h compiled for the host: the formulas themselves, not copies of them."""
import ctypes
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1901_00275_amd", "csrc")

SOURCE = r"""
#include "bounds.h"
// The last turns of a workgroup whose lists hold `total` points: 0 if the places handed out are exactly those up to
// `total` and the loop ends, else what went wrong.
extern "C" int last_turns(long long total)
{
    const sw_place_t t = (sw_place_t)total;
    const long long first = total / SW_TURN > 2 ? (total / SW_TURN - 2) * SW_TURN : 0;
    long long next = first;
    int turns = 0;
    for (sw_place_t turn = (sw_place_t)first; turn < t; turn += SW_TURN) {
        if (++turns > 4) return 1;
        for (int wave = 0; wave < SW_NT / 64; ++wave) {
            const sw_place_t base = sw_wave_base(turn, wave);
            for (int u = 0; u < SW_U; ++u)
                for (int lane = 0; lane < 64; ++lane) {
                    const sw_place_t p = sw_place(base, u, lane);
                    if (p < t && (long long)p != next++) return 2;
                }
        }
    }
    return next == total ? 0 : 3;
}
extern "C" float slack(float R2, float Y2, float Q2, float e2, float L, int D, int m)
{
    return scan_wide_slack(R2, Y2, Q2, e2, L, D, m);
}
extern "C" float half_band(float xn, float res, float rho, float big, float dmin, float band_dist, int D)
{
    return nn_half_band(xn, res, rho, big, dmin, band_dist, D);
}
extern "C" int exponent_of(float mx) { return half_exponent(mx); }
extern "C" int gap(void) { return HALF_GAP; }
extern "C" float rel_max(void) { return HALF_REL_MAX; }
extern "C" int idx_bits(int tiles) { return half_idx_bits(tiles); }
extern "C" float band_dist(int bits) { return half_band_dist(bits); }
"""

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "bounds.cpp"), os.path.join(d, "bounds.so")
            with open(src, "w") as f:
                f.write(SOURCE)
            subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
            _lib = ctypes.CDLL(so)
        f, i = ctypes.c_float, ctypes.c_int
        _lib.last_turns.argtypes = [ctypes.c_longlong]
        _lib.slack.restype, _lib.slack.argtypes = f, [f] * 5 + [i] * 2
        _lib.half_band.restype, _lib.half_band.argtypes = f, [f] * 6 + [i]
        _lib.exponent_of.argtypes = [f]
        _lib.rel_max.restype = f
        _lib.band_dist.restype, _lib.band_dist.argtypes = f, [i]
    return _lib

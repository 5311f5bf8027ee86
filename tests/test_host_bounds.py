"""Arithmetic that kernels rely on (csrc/bounds.h), compiled for the host and checked there."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1901_00275_amd", "csrc")

PLACES = r"""
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
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    src, so = d / "places.cpp", d / "places.so"
    src.write_text(PLACES)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


# an index holds up to 2^31 - 1 points: the places behind its last turn need 32 bits
@pytest.mark.parametrize("total", [1, 2047, 2048, 2049, 10_000, 2**31 - 4097, 2**31 - 2049, 2**31 - 2048, 2**31 - 2047, 2**31 - 1])
def test_places_up_to_the_largest_index(host, total):
    host.last_turns.argtypes = [ctypes.c_longlong]
    assert host.last_turns(total) == 0

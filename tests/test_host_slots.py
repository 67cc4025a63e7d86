"""The slots that a device-resident step loop enqueues between two looks of the
host: all of a chunk where the steps left are many, up to the largest count that
a caller can give, and no more than the steps need near the end."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def slots_for(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "s.cpp").write_text('#include "af_slots.hpp"\n'
                             'extern "C" long f(long l, int r, long c)'
                             ' { return afi::slots_for(l, r, c); }\n')
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2609_29081_amd", "csrc"), str(d / "s.cpp"), "-o",
                    str(d / "s.so")], check=True)
    f = C.CDLL(str(d / "s.so")).f
    f.argtypes, f.restype = [C.c_long, C.c_int, C.c_long], C.c_long
    return f


@pytest.mark.parametrize("chunk", [1, 4, 8])
@pytest.mark.parametrize("rounds", [1, 2, 3, 4, 1000, (1 << 31) - 1])
def test_slots(slots_for, rounds, chunk):
    for left in (0, 1, 2, 3, 4, 5, 31, 32, 33, 10 ** 6, (1 << 63) - 2, (1 << 63) - 1):
        assert slots_for(left, rounds, chunk) == max(1, min(chunk, -(-left // rounds)))

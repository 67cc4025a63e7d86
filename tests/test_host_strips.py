"""The cut of a single 2D grid into strips, on the host: the few row counts that
the library looks at against a look at every one (the fewest row steps in all,
of equal ones the least ranges), for grids of all shapes and devices of several
sizes; and that it costs a launch little."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = r"""
#include <algorithm>
#include "af_strips.hpp"
using namespace afi;
extern "C" void fast(int n1x, int n2y, int cus, long most, int* out) {
  const StripShape b = strip_shape(n1x, n2y, cus, most);
  out[0] = b.nx; out[1] = b.ny; out[2] = b.H;
}
extern "C" void every(int n1x, int n2y, int cus, long most, int* out) {
  StripShape b{};
  long best = 0;
  for (int ny = 1; ny <= n2y; ++ny) {
    const StripShape t = strips_with(n1x, n2y, (n2y + ny - 1) / ny);
    const long wgs = (long)t.nx * t.ny;
    if (ny > 1 && wgs > std::min(8L * cus, most)) break;
    const long steps = (wgs + cus - 1) / cus * (t.H + 5);
    if (ny == 1 || steps < best) { b = t; best = steps; }
  }
  out[0] = b.nx; out[1] = b.ny; out[2] = b.H;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("strips")
    src = d / "s.cpp"
    src.write_text(CODE)
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2609_29081_amd", "csrc"), str(src), "-o",
                    str(d / "s.so")], check=True)
    return C.CDLL(str(d / "s.so"))


def shapes():
    rng = random.Random(1)
    for n1x in list(range(4, 70)) + [119, 120, 121, 400, 1000, 1001, 2048, 61441, 1 << 20]:
        for n2y in (4, 5, 31, 255, 256, 257, 500, 501, 1024, 1025, 2000, 5000):
            yield n1x, n2y
    for _ in range(3000):
        yield int(4 * 10 ** rng.uniform(0, 3.5)), int(4 * 10 ** rng.uniform(0, 3.5))


@pytest.mark.parametrize("cus,most", [(256, 1024), (304, 1024), (80, 1024), (1, 1024), (2048, 1024)])
def test_the_cut_is_the_best_of_all(lib, cus, most):
    a, b = (C.c_int * 3)(), (C.c_int * 3)()
    for n1x, n2y in shapes():
        lib.fast(n1x, n2y, cus, C.c_long(most), a)
        lib.every(n1x, n2y, cus, C.c_long(most), b)
        assert list(a) == list(b), (n1x, n2y, cus)
        assert a[0] * a[1] <= max(most, a[0])


def test_the_cut_costs_a_launch_little(lib):
    """this is asked for at every launch; looking at every row count took 35 us
    at 57 x 2000"""
    import time
    a = (C.c_int * 3)()

    def us(f):
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            for _ in range(200):
                f(58, 2001, 256, C.c_long(1024), a)
            best = min(best, (time.perf_counter() - t) / 200 * 1e6)
        return best
    few, all_of_them = us(lib.fast), us(lib.every)
    print(f"{few:.2f} us, every row count {all_of_them:.2f} us")
    assert few < all_of_them / 2

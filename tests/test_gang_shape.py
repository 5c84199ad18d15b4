"""Blocks per CG system of a batched launch (csrc/qdot_gang_shape.hpp), on the
host: a gang waits for all of its blocks, so the shape has to follow the
blocks that the launch really has on the chip."""
import ctypes as C
import os
import subprocess

import pytest

import paper_2105_00115_amd as q

CSRC = os.path.join(os.path.dirname(os.path.abspath(q.__file__)), "csrc")
SOURCE = """
#include "qdot_gang_shape.hpp"
extern "C" void shape(const long long *n, int S, long long rows, int most, long long resident,
                      long long chunk, int *sizes)
{
    const qd::GangShape g =
        qd::gang_shape([&](int s) { return n[s]; }, S, qd::GangShape{rows, most}, resident, chunk);
    for (int s = 0; s < S; s++) sizes[s] = g.size(n[s]);
}
extern "C" int launches() { return qd::GANG_LAUNCHES; }
"""
CHUNK = 1024


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    src, out = d / "shape.cpp", d / "shape.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(out)], check=True)
    return C.CDLL(str(out))


def _sizes(lib, n, rows, most, resident):
    arr, out = (C.c_longlong * len(n))(*n), (C.c_int * len(n))()
    lib.shape(arr, len(n), C.c_longlong(rows), most, C.c_longlong(resident),
              C.c_longlong(CHUNK), out)
    return list(out)


BATCHES = [[1], [1025], [500_000], [1 << 20], [2_000_000_000], [32 * 32] * 24, [512 * 512] * 24,
           [4096] * 1000, [262_144, 100, 65_537, 1_000_000], [700_000] * 3]


@pytest.mark.parametrize("resident", [1, 100, 256, 512, 768])
@pytest.mark.parametrize("rows,most", [(1024, 512), (8192, 16), (8192, 512), (16384, 1),
                                       (1 << 20, 300)])
def test_no_gang_waits_for_blocks_that_cannot_be_resident(lib, resident, rows, most):
    for n in BATCHES:
        sizes = _sizes(lib, n, rows, most, resident)
        tuned = [max(1, min(most, resident, -(-m // rows))) for m in n]
        assert max(sizes) <= resident
        # never fewer blocks than the tuned shape gives, and more only while
        # all gangs are resident together
        assert all(s >= t for s, t in zip(sizes, tuned))
        assert sizes == tuned or sum(sizes) <= resident
        # enough launches at once never fill the chip with gangs that wait
        assert max(sizes) <= max(resident // lib.launches(), *tuned, 1, min(most, resident))


def test_a_grid_of_one_block_per_cu_is_followed(lib):
    """500 000 rows with gangs of up to 512 allowed: 256 resident blocks give
    a gang of at most 256 (the two blocks per CU that the kernel could hold
    are not in the grid), and the tuned 8192 rows give 62."""
    assert _sizes(lib, [500_000], 8192, 512, 256)[0] <= 256
    assert _sizes(lib, [500_000], 8192, 512, 512)[0] == 489
    assert _sizes(lib, [500_000], 8192, 16, 256) == [32]
    assert _sizes(lib, [500_000], 8192, 16, 512) == [64]

"""The choice between the two bf16 GEMM kernels (tiles.hpp), compiled for the
host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2205_01848_amd", "csrc")
CUS = 256


def tiles_lib(tmp):
    """mid_pays and mid_time as C functions."""
    src, lib = os.path.join(tmp, "t.cpp"), os.path.join(tmp, "t.so")
    with open(src, "w") as f:
        f.write('''#include "tiles.hpp"
extern "C" int pays(int E, int64_t R, int N, int K, int gated, int act, int km, int64_t pa, int64_t pb, int cus) {
  return moe::mid_pays({E, R, N, K, gated != 0, act != 0, km != 0, pa, pb}, cus);
}
''')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib],
                   check=True)
    L = ctypes.CDLL(lib)
    i, l = ctypes.c_int, ctypes.c_int64
    L.pays.argtypes = [i, l, i, i, i, i, i, l, l, i]
    return L


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return tiles_lib(str(tmp_path_factory.mktemp("tiles")))


def products(d, f, swiglu):
    """(N, K, gated, act, K-major, A pitch, B pitch) of H, Y, dA and dX."""
    F = 2 * f if swiglu else f
    return [(f, d, swiglu, 1, 0, 2 * d, 2 * d), (d, f, 0, 0, 0, 2 * f, 2 * f),
            (f, d, 0, 1, 1, 2 * d, 2 * f), (d, F, 0, 0, 1, 2 * F, 2 * d)]


@pytest.mark.parametrize("d,f,swiglu", [(512, 2048, False), (1024, 4096, True), (4096, 14336, True),
                                        (64, 128, False), (1000, 2504, False)])
@pytest.mark.parametrize("E,R", [(1, 1), (1, 64), (1, 127), (1, 128), (2, 5), (8, 8), (8, 64)])
def test_few_rows_take_the_smaller_tiles(lib, E, R, d, f, swiglu):
    """A handful of rows per expert fills one 256-row tile per expert to a
    small part: the 256x256 kernel takes two to four times as long."""
    for p in products(d, f, swiglu):
        assert lib.pays(E, R, *map(int, p), CUS), p


@pytest.mark.parametrize("E,rows,d,f,swiglu", [(8, 16384, 4096, 14336, True), (32, 2048, 2048, 8192, False),
                                               (64, 2048, 4096, 4096, False)])
def test_large_products_keep_the_large_tiles(lib, E, rows, d, f, swiglu):
    for p in products(d, f, swiglu)[:2]:
        assert not lib.pays(E, E * rows, *map(int, p), CUS), p


@pytest.mark.parametrize("E,rows,d,f", [(32, 512, 1024, 4096), (64, 512, 1024, 4096), (16, 512, 2048, 2048)])
def test_filled_whole_tiles_keep_the_large_tiles(lib, E, rows, d, f):
    """Static capacities of whole 256-row tiles (the padded baseline among
    them) leave no ragged tile to save: Y and dX took 1.4 times as long on the
    smaller ones."""
    for p in products(d, f, False)[1::2]:
        assert not lib.pays(E, E * rows, *map(int, p), CUS), p

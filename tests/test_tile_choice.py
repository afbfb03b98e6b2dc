"""The choice between the two bf16 GEMM kernels (tiles.hpp), compiled for the
host."""
import pytest

import tiles_util as T


@pytest.mark.parametrize("d,f,swiglu", [(512, 2048, False), (1024, 4096, True), (4096, 14336, True),
                                        (64, 128, False), (1000, 2504, False)])
@pytest.mark.parametrize("E,R", [(1, 1), (1, 64), (1, 127), (1, 128), (2, 5), (8, 8), (8, 64)])
def test_few_rows_take_the_smaller_tiles(E, R, d, f, swiglu):
    """A handful of rows per expert fills one 256-row tile per expert to a
    small part: the 256x256 kernel takes two to four times as long."""
    for p in T.products(d, f, swiglu):
        assert T.pays(E, R, p), p


@pytest.mark.parametrize("E,rows,d,f,swiglu", [(8, 16384, 4096, 14336, True), (32, 2048, 2048, 8192, False),
                                               (64, 2048, 4096, 4096, False)])
def test_large_products_keep_the_large_tiles(E, rows, d, f, swiglu):
    for p in T.products(d, f, swiglu):
        for R in (E * rows, E * rows + 5, E * rows * 21 // 20):
            assert not T.pays(E, R, p), (p, R)


@pytest.mark.parametrize("E,rows,d,f", [(32, 512, 1024, 4096), (64, 512, 1024, 4096), (16, 512, 2048, 2048)])
def test_filled_whole_tiles_keep_the_large_tiles(E, rows, d, f):
    """Static capacities of whole 256-row tiles (the padded baseline among
    them) leave no ragged tile to save: Y and dX took 1.4 times as long on the
    smaller ones."""
    for p in T.products(d, f, False)[1::2]:
        assert not T.pays(E, E * rows, p), p


@pytest.mark.parametrize("E,rows,d,f", [(4, 2048, 1024, 4096), (8, 1024, 1024, 4096), (16, 1024, 2048, 2048),
                                        (32, 1024, 1024, 4096)])
def test_half_filled_whole_tiles_take_the_smaller_tiles(E, rows, d, f):
    """A static capacity of twice a layer's picks holds about half its rows:
    read as filled, H or Y kept the 256x256 kernel and took 1.5 to 1.8 times as
    long."""
    took = [T.pays(E, E * rows, p, most=E * rows // 2) and not T.pays(E, E * rows, p)
            for p in T.products(d, f, False)[:2]]
    assert any(took)
    # picks that can fill the capacity change nothing
    for p in T.products(d, f, False)[:2]:
        assert T.pays(E, E * rows, p, most=E * rows) == T.pays(E, E * rows, p)

"""Tile choice and grids of the GEMMs (host code of the library)."""
import ctypes as C

import pytest

from _cases import gemm_plan


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


@pytest.mark.parametrize("rows", [1, 33, 16384, 65536 * 32, 65536 * 32 + 1, 7500000])
def test_f32_grid_within_the_device_limits(rows):
    """Up to the rows that 288 GB hold (about 37 KB of workspace each)."""
    from paper_2608_29809_amd import abi
    f = abi.LIB._ZN2rc13gemm_f32_gridEiii
    f.restype, f.argtypes = _Dim3, [C.c_int] * 3
    for N, bn in ((1152, 32), (1152, 64), (4608, 32), (4608, 64)):
        g = f(rows, N, bn)
        assert g.x * 32 >= rows > (g.x - 1) * 32 and g.y * bn == N and g.z == 1
        assert g.x * 256 < 2 ** 31 and g.y <= 65536


def test_plan_is_steady_in_the_row_count():
    """A plan holds for a run of row counts: a tile more or less of one of the
    candidates may change it, a single row may not change it back and forth."""
    for N, K, epi in ((3456, 1152, "qkv"), (1152, 1152, "resid"), (1152, 1152, "store"), (4608, 1152, "gelu"),
                      (1152, 4608, "resid")):
        last, start = None, 1
        for M in range(1, 16385):
            p = gemm_plan(M, N, K, epi)[4]
            if p != last:
                assert last is None or M - start >= 32, (N, K, epi, start, M, last, p)
                last, start = p, M


def test_a_short_sum_keeps_the_small_tiles():
    """Narrow outputs of up to 2458 rows take the small tiles at every depth of
    the sum up to the model's width, where they measured faster; from a depth
    of 512 on, 4096 rows take the large ones."""
    for K in (64, 128, 256, 512, 768, 1024, 1152):
        for M in (256, 723, 1100, 1639, 2458):
            assert not gemm_plan(M, 1152, K, "resid")[0], (M, K)
        if K >= 512:
            assert gemm_plan(4096, 1152, K, "resid")[0], K

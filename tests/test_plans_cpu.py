"""The tile choice of the bf16 GEMMs (host code of the library)."""
from _cases import gemm_plan


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

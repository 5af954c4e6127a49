"""Slabs of short GEMM sums: taken while a workgroup's shorter sum saves more
time than the slabs take to write and read.  16-bit storage, whose terms are the
cheaper, keeps large outputs over 2^9 and 2^10 terms whole; the same shapes in
complex64, and small outputs in either, are split."""
import pytest

from paper_2111_01066_amd import tnrcs


@pytest.mark.parametrize("nM,nN,nK,half,c64", [(13, 7, 9, 1, 2), (11, 9, 9, 1, 2), (14, 6, 9, 1, 2), (12, 6, 9, 1, 2),
                                               (11, 11, 9, 1, 2), (11, 11, 10, 1, 2), (14, 7, 11, 2, 4), (11, 7, 9, 2, 2),
                                               (10, 6, 9, 2, 2), (6, 6, 9, 2, 2), (8, 8, 10, 4, 4), (7, 7, 11, 8, 8)])
@pytest.mark.parametrize("low", [True, False])
def test_slabs(nM, nN, nK, half, c64, low):
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    for dtype, slabs in (("f16s", half), ("bf16s", half), ("c64", c64)):
        pp = tnrcs.PairPlan(m + k if low else k + m, n + k, m + n, dtype=dtype, dry_run=True)
        g = [o for o in pp.json()["ops"] if o["kind"] == 1]
        pp.close()
        in_place = g[0]["ga"] == 1
        # (A in place: not split from one workgroup per CU below 2^11 terms)
        want = 1 if in_place and nK < 11 and nM + nN - 14 >= 8 else slabs
        assert [o["split_k"] for o in g] == [want]

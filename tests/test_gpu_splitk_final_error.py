"""Rounding of the split-K final sum: the partial sums of all blocks meet in
FP32, one of them 2^24 and the others 1 (each block holds one product that is
not zero), so that every addition of a single 1 to the large one is lost.  A
sum of depth d of non-negative terms is off by at most d 2^-24 of its value;
the depth is that of 256 chains of at most 4 partials and a tree over them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402

DEPTH = 4 + 8


# in place: both operands read in chunks of 2^8 terms, which 512 blocks take in
# turn; otherwise 1024 blocks of 256 threads with 2 consecutive terms each
@pytest.mark.parametrize("nM,nN,in_place", [(3, 3, True), (2, 2, True), (3, 3, False), (2, 2, False), (0, 0, False),
                                            (4, 4, False), (5, 3, False)])
def test_partials_do_not_chain(nM, nN, in_place):
    print(f"split-K final sum {nM} {nN} in place {in_place}", flush=True)
    nK = 20
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    la = k + m if in_place else m + k
    pp = tnrcs.PairPlan(la, n + k, m + n)
    js = pp.json()
    assert js["steps"][0]["cls"] == 4 and len(js["ops"]) == 1
    n_blocks, step = (512, 1 << 8) if in_place else (1024, 1 << 9)
    a = np.zeros((1 << nK, 1 << nM), dtype=np.complex64)
    a[[b * step for b in range(n_blocks)]] = 1.0
    a[0] = 2.0 ** 24
    A = torch.from_numpy(np.ascontiguousarray(a if in_place else a.T).reshape(-1)).cuda()
    B = torch.ones(1 << (nN + nK), dtype=torch.complex64, device="cuda")
    C = torch.empty(1 << (nM + nN), dtype=torch.complex64, device="cuda")
    pp.run(A, B, C)
    torch.cuda.synchronize()
    pp.close()
    ref = 2.0 ** 24 + n_blocks - 1
    assert np.abs(C.cpu().numpy() - ref).max() <= DEPTH * 2.0 ** -24 * ref

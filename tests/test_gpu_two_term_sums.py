"""Gathered contractions of two terms into few outputs: rounded as one chain of
multiply-adds (which is emulated here), since adding two separately
rounded products has a relative error 1.028 times as large (2^17 outputs)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402


def _fma(a, b, c):  # the product is exact in FP64
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


@pytest.mark.parametrize("nM,nN", [(6, 5), (5, 4), (3, 0)])
def test_two_terms(nM, nN):
    print(f"two terms {nM} {nN}", flush=True)
    batch = 1 << (17 - nM - nN)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), [100]
    pp = tnrcs.PairPlan(m + k, n + k, m + n)
    assert [o["kind"] for o in pp.json()["ops"]] == [2]
    rng = np.random.default_rng(nM)
    a = rng.standard_normal((batch, 1 << nM, 1, 2, 2)).astype(np.float32)
    b = rng.standard_normal((batch, 1, 1 << nN, 2, 2)).astype(np.float32)
    A, B = torch.from_numpy(a.reshape(-1, 2)).cuda(), torch.from_numpy(b.reshape(-1, 2)).cuda()
    C = torch.empty(1 << 17, 2, device="cuda")
    pp.run(A, B, C, batch=batch)
    torch.cuda.synchronize()
    pp.close()
    a, b = np.broadcast_arrays(a, b)
    re = im = np.zeros(a.shape[:3], np.float32)
    for t in range(2):
        re = _fma(-a[..., t, 1], b[..., t, 1], _fma(a[..., t, 0], b[..., t, 0], re))
        im = _fma(a[..., t, 1], b[..., t, 0], _fma(a[..., t, 0], b[..., t, 1], im))
    ref = ((a.astype(np.float64) @ [1, 1j]) * (b.astype(np.float64) @ [1, 1j])).sum(-1).reshape(-1)
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    chain = np.linalg.norm((re.astype(np.float64) + 1j * im).reshape(-1) - ref)
    assert np.linalg.norm(got - ref) <= 1.01 * chain

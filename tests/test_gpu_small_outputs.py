"""Contractions into few outputs on the GPU: the gathered kernel with several
lanes per output (from one term per lane to more than its offset table holds)
and the split-K final sum, against the oracle's contraction of the same rounded
inputs.  FP32 sums of n terms of a random sign stay within u sqrt(n) of the
result normwise; one rounding to 16 bits adds half a unit in the last place."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.tn import pairwise_contract  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402

UNIT = {"c64": 0.0, "f16s": 2.0 ** -11, "bf16s": 2.0 ** -8}


@pytest.mark.parametrize("dtype", ["c64", "f16s", "bf16s"])
@pytest.mark.parametrize("nM,nN,nK", [(0, 0, 0), (1, 0, 1), (0, 0, 9), (2, 1, 6), (3, 2, 11), (4, 3, 11), (5, 5, 6),
                                      (6, 5, 4), (7, 3, 3), (3, 3, 12), (2, 0, 13), (5, 4, 12), (7, 5, 12)])
def test_few_outputs(dtype, nM, nN, nK):
    print(f"few outputs {dtype} {nM} {nN} {nK}", flush=True)
    rng = np.random.default_rng(1000 + 100 * nM + 10 * nN + nK)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    la, lb = [int(x) for x in rng.permutation(m + k)], [int(x) for x in rng.permutation(n + k)]
    lc = [x for x in la if x in m] + [x for x in lb if x in n]
    t = {"c64": torch.float32, "f16s": torch.float16, "bf16s": torch.bfloat16}[dtype]
    A = torch.from_numpy(rng.standard_normal((1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((1 << len(lb), 2))).to(t)
    C = torch.empty(1 << (nM + nN), 2, dtype=t, device="cuda")
    scale = 1.0 if dtype == "c64" else 2.0 ** -(nK // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype)
    pp.run(A.cuda(), B.cuda(), C, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    ref, lr = pairwise_contract(a.reshape((2,) * len(la)), la, b.reshape((2,) * len(lb)), lb)
    ref = np.transpose(ref, [list(lr).index(x) for x in lc]).reshape(-1) * scale if lc else np.asarray(ref).reshape(-1) * scale
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK + 8) + UNIT[dtype]
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)

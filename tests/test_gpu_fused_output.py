"""Pairwise plans whose last kernel writes C in the caller's index order (in
place of a permute): every kernel that can, over its range of columns, terms
and rows, with random orders of all three tensors, against FP64 sums of the
same rounded inputs (bounds as in test_gpu_half_layouts)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402
from tests.test_gpu_half_layouts import UNIT, _offsets, _product  # noqa: E402

# GEMM with A in place (A of 2^20 entries or more); skewed: every column count, K
# from 2, the fewest rows (one pass) and more passes than blocks
GEMM = [(15, 7, 5), (14, 7, 6), (13, 8, 7), (13, 9, 11)]
SKEW = [(7, 0, 2), (8, 1, 1), (9, 2, 3), (10, 3, 4), (9, 4, 5), (8, 5, 6), (9, 6, 6), (11, 6, 4), (17, 3, 4), (18, 5, 3),
        (9, 5, 7), (10, 6, 8)]


@pytest.mark.parametrize("dtype", ["c64", "f16s", "bf16s"])
@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("shape", GEMM + SKEW)
def test_c_in_callers_order(dtype, seed, shape):
    nM, nN, nK = shape
    rng = np.random.default_rng(100 * seed + nM + nN + nK)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    la, lb, lc = ([int(x) for x in rng.permutation(v)] for v in (m + k, n + k, m + n))
    print(f"fused output {dtype} {shape} {la} {lb} {lc}", flush=True)
    t = {"c64": torch.float32, "f16s": torch.float16, "bf16s": torch.bfloat16}[dtype]
    A = torch.from_numpy(rng.standard_normal((2, 1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((2, 1 << len(lb), 2))).to(t)
    C = torch.full((2, 1 << len(lc), 2), float("nan"), dtype=t, device="cuda")
    scale = 1.0 if dtype == "c64" else 2.0 ** -(nK // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype)
    pp.run(A.cuda(), B.cuda(), C, batch=2, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    free = [x for x in la if x < 50] + [x for x in lb if 50 <= x < 100]
    for i in range(2):
        a, b = (x[i].double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
        ref = _product(a, la, b, lb)[_offsets(lc, free)] * scale
        got = C[i].cpu().double().numpy() @ np.array([1.0, 1j])
        bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK + 8) + UNIT.get(dtype, 0.0)
        assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)


def test_most_of_these_orders_are_written_directly():
    fused = total = 0
    for nM, nN, nK in GEMM + SKEW:
        for seed in range(3):
            rng = np.random.default_rng(100 * seed + nM + nN + nK)
            m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
            la, lb, lc = ([int(x) for x in rng.permutation(v)] for v in (m + k, n + k, m + n))
            for dtype in ("c64", "f16s"):
                pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype, dry_run=True)
                fused += pp.json()["fused_out"]
                total += 1
    print(f"{fused} of {total}")
    assert fused > total // 2

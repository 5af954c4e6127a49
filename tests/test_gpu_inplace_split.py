"""GEMMs that read A in place with their sum split in slabs (one to many slabs
of one and more output tiles) or with the smallest A that is read in place:
random orders of all three tensors, against FP64 sums of the same rounded
inputs (bounds as in test_gpu_half_layouts)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2111_01066_amd import tnrcs  # noqa: E402
from tests.test_gpu_half_layouts import UNIT, _offsets, _product  # noqa: E402

# rows, columns, terms (log2) and the slabs that the planner takes
SHAPES = [((11, 7, 9), 2), ((10, 7, 10), 4), ((9, 8, 11), 8), ((7, 7, 13), 32), ((8, 9, 12), 16), ((11, 11, 11), 2)]

# the smallest 16-bit A read in place (2^17 entries), few tiles of short sums
SMALL = [(10, 7, 7), (9, 8, 8), (12, 7, 5)]


def _labels(shape, seed):
    nM, nN, nK = shape
    rng = np.random.default_rng(100 * seed + nM + nN + nK)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    return rng, [[int(x) for x in rng.permutation(v)] for v in (m + k, n + k, m + n)]


@pytest.mark.parametrize("dtype,form", [("c64", "3m"), ("c64", "4m"), ("f16s", "4m"), ("bf16s", "4m")])
@pytest.mark.parametrize("shape,slabs", SHAPES)
def test_planned_slabs(dtype, form, shape, slabs):
    for seed in range(2):
        _, (la, lb, lc) = _labels(shape, seed)
        pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype, gemm_form=form, dry_run=True)
        g = [o for o in pp.json()["ops"] if o["kind"] == 1]
        assert [(o["ga"], o["split_k"], o["split_max"]) for o in g] == [(1, slabs, slabs)]


@pytest.mark.parametrize("dtype", ["c64", "f16s", "bf16s"])
def test_smallest_a_read_in_place(dtype):
    def ga(shape):
        _, (la, lb, lc) = _labels(shape, 0)
        pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype, dry_run=True)
        return [o["ga"] for o in pp.json()["ops"] if o["kind"] == 1]

    assert all(ga(s) == [int(dtype != "c64")] for s in SMALL)
    assert ga((9, 7, 7)) == [0] and ga((13, 7, 7)) == [1]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,form", [("c64", "3m"), ("c64", "4m"), ("f16s", "4m"), ("bf16s", "4m")])
@pytest.mark.parametrize("seed", [0, 1])
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES] + SMALL)
def test_slabs_of_a_read_in_place(dtype, form, seed, shape):
    nM, nN, nK = shape
    rng, (la, lb, lc) = _labels(shape, seed)
    print(f"in-place split {dtype} {form} {shape} {la} {lb} {lc}", flush=True)
    t = {"c64": torch.float32, "f16s": torch.float16, "bf16s": torch.bfloat16}[dtype]
    A = torch.from_numpy(rng.standard_normal((1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((1 << len(lb), 2))).to(t)
    C = torch.full((1 << len(lc), 2), float("nan"), dtype=t, device="cuda")
    scale = 1.0 if dtype == "c64" else 2.0 ** -(nK // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype, gemm_form=form)
    pp.run(A.cuda(), B.cuda(), C, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    free = [x for x in la if x < 50] + [x for x in lb if 50 <= x < 100]
    ref = _product(a, la, b, lb)[_offsets(lc, free)] * scale
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK + 8) + UNIT.get(dtype, 0.0)
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)

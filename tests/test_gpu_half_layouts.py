"""16-bit kernels that read A in place in 16-byte loads: each combination of
row and contracted bits among A's two lowest index bits, for the GEMM and both
skewed kernels (B resident and staged), against FP64 sums of the same rounded
inputs.  An FP32 sum of n products of random sign stays within 2^-24 sqrt(n)
normwise; the result is rounded once to 16 bits (half a unit in the last place)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2111_01066_amd import tnrcs  # noqa: E402
from tests.plan_interp import PlanInterpreter  # noqa: E402

UNIT = {"f16s": 2.0 ** -11, "bf16s": 2.0 ** -8}
SHAPES = [(15, 7, 5), (13, 8, 7), (9, 5, 4), (10, 6, 5), (8, 3, 6), (9, 5, 7), (7, 6, 10)]
LOW = ["kk", "kr", "rk", "rr"]  # A's positions 1, 0: contracted (k) or row (r) bits


def _labels(nM, nN, nK, low, seed):
    rng = np.random.default_rng(seed)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    rng.shuffle(m)
    rng.shuffle(k)
    tail = [(k if x == "k" else m).pop() for x in low]
    la = [int(x) for x in rng.permutation(m + k)] + tail
    lb = [int(x) for x in rng.permutation(n + list(range(100, 100 + nK)))]
    lc = [x for x in la if x < 50] + [x for x in lb if 50 <= x < 100]
    return la, lb, lc


def _offsets(labels, layout):
    off = np.zeros(1, dtype=np.int64)
    for x in labels:
        off = (off[:, None] + np.array([0, 1 << (len(layout) - 1 - layout.index(x))])[None, :]).reshape(-1)
    return off


def _product(A, la, B, lb):
    k = [x for x in la if x in lb]
    m, n = [x for x in la if x not in lb], [x for x in lb if x not in la]
    a = A[_offsets(m, la)[:, None] + _offsets(k, la)[None, :]]
    b = B[_offsets(k, lb)[:, None] + _offsets(n, lb)[None, :]]
    return (a @ b).reshape(-1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16s", "bf16s"])
@pytest.mark.parametrize("low", LOW)
@pytest.mark.parametrize("shape", SHAPES)
def test_low_bits_of_a(dtype, low, shape):
    print(f"half layouts {dtype} {low} {shape}", flush=True)
    la, lb, lc = _labels(*shape, low, seed=sum(shape) + LOW.index(low))
    t = torch.float16 if dtype == "f16s" else torch.bfloat16
    rng = np.random.default_rng(1)
    A = torch.from_numpy(rng.standard_normal((1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((1 << len(lb), 2))).to(t)
    C = torch.empty(1 << len(lc), 2, dtype=t, device="cuda")
    scale = 2.0 ** -(shape[2] // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype)
    pp.run(A.cuda(), B.cuda(), C, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    ref = _product(a, la, b, lb) * scale
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** shape[2]) + UNIT[dtype]
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)


@pytest.mark.parametrize("low", LOW)
@pytest.mark.parametrize("shape", SHAPES)
def test_low_bits_of_a_plan(low, shape):
    la, lb, lc = _labels(*shape, low, seed=sum(shape) + LOW.index(low))
    rng = np.random.default_rng(2)
    A, B = (rng.standard_normal(1 << len(x)) + 1j * rng.standard_normal(1 << len(x)) for x in (la, lb))
    pp = tnrcs.PairPlan(la, lb, lc, dtype="f16s", dry_run=True)
    it = PlanInterpreter.__new__(PlanInterpreter)
    it.js = pp.json()
    it.arena = np.full(it.js["arena_elems"], np.nan, dtype=np.complex128)
    it.leaves = it.bound = np.zeros(0, dtype=np.complex128)
    C = np.full(1 << len(lc), np.nan, dtype=np.complex128)
    it.ext = {3: A, 4: B, 5: C}
    it.run_ops()
    ref = _product(A, la, B, lb)
    assert np.linalg.norm(C - ref) <= 1e-12 * np.linalg.norm(ref)

"""Small networks of many slices: single slices (added to the amplitudes by the
contraction's own kernel) and longer ranges (by a second one) give the same sum
as the whole range, bit for bit, wherever the range is cut."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402
from tests.test_gpu_small_net import _net, _sum  # noqa: E402


@pytest.mark.parametrize("dtype", ["c64", "f16s", "bf16s"])
@pytest.mark.parametrize("shape", [(3, 4, 8, 3, 11), (3, 4, 8, 2, 5), (4, 4, 8, 2, 12)])
def test_cuts(dtype, shape):
    print(f"small network cuts {dtype} {shape}", flush=True)
    c, open_q, bits, pairs, sliced = _net(*shape)
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype=dtype)
    n = plan.info()["n_slices"]
    assert plan.json()["small_net"] and n >= 4
    got = _sum(plan, len(open_q), [0, n])
    rng = np.random.default_rng(n)
    some = sorted({0, 1, 2, n // 2, n // 2 + 1, n - 1, n} | {int(x) for x in rng.integers(0, n, 12)})
    runs = [list(range(n + 1))[:200] + [n], some, [0, n - 1, n], [0, n // 3, n]]
    for cuts in runs:
        assert np.array_equal(got, _sum(plan, len(open_q), sorted(set(cuts))))
    plan.close()

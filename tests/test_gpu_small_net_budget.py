"""A small network's plan keeps to its memory budget: with none to spare for
the results of many slices, slices are launched in smaller groups, with the
same sum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402
from tests.test_gpu_small_net import _net, _sum  # noqa: E402


def test_scratch_within_the_budget():
    print("small network budget", flush=True)
    c, open_q, bits, pairs, sliced = _net(3, 4, 12, 8, 9)
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits)
    info = plan.info()
    need = info["arena_bytes"] + info["leaf_bytes"]
    cuts = [0, 37]
    assert plan.json()["small_net"] and info["n_slices"] == 8192
    ref = _sum(plan, 8, cuts)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for spare in (0, 1 << 14, 1 << 17):  # single slices, a few, and all of them in one launch
        tight = tnrcs.Plan(c, pairs, sliced, open_q, bits, arena_bytes=need + spare)
        assert tight.json()["small_net"]
        # (8 MiB hold 4096 slices' results; device memory comes in blocks of 2 MiB)
        assert free0 - torch.cuda.mem_get_info()[0] < 6 << 20
        assert np.array_equal(ref, _sum(tight, 8, cuts))
        tight.close()
        torch.cuda.synchronize()
    plan.close()

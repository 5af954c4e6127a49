"""Plan statistics count what is launched: a pairwise plan whose last kernel
writes the caller's index order has no permute of the result and no room for
its intermediate, and a small network's slice is one launch."""
import numpy as np
import pytest

from paper_2111_01066_amd import tnrcs
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit
from rqcgen.order import bisection_order

ELEM = {"c64": 8, "f16s": 4}


def _pair(nM, nN, nK, seed):
    rng = np.random.default_rng(seed)
    m, n, k = list(range(nM)), list(range(50, 50 + nN)), list(range(100, 100 + nK))
    return [[int(x) for x in rng.permutation(s)] for s in (m + k, n + k, m + n)]


@pytest.mark.parametrize("dtype", ["c64", "f16s"])
@pytest.mark.parametrize("nM,nN,nK", [(14, 8, 7), (16, 7, 6), (17, 4, 5), (18, 5, 4)])
def test_fused_output(dtype, nM, nN, nK):
    seen = set()
    for seed in range(12):
        pp = tnrcs.PairPlan(*_pair(nM, nN, nK, seed), dtype=dtype, dry_run=True)
        js, info = pp.json(), pp.info()
        pp.close()
        fused = js["fused_out"]
        seen.add(fused)
        run = js["ops"][:-1] if fused else js["ops"]
        assert info["n_kernels"] == len(run)
        assert info["n_permute"] == sum(o["kind"] == 0 for o in run)
        step = (1 << (nM + nK)) + (1 << (nN + nK)) + (1 << (nM + nN))
        assert info["moved_per_slice"] == ELEM[dtype] * sum(2 << o["rank"] if o["kind"] == 0 else step for o in run)
        assert info["arena_bytes"] == ELEM[dtype] * js["arena_elems"] - fused * (ELEM[dtype] << (nM + nN))
        # buffers that the launches use lie within the allocation, apart
        used = {}
        for o in run:
            size = 1 << o["rank"] if o["kind"] == 0 else None
            refs = [(o["a"], size), (o["c"], size)] if o["kind"] == 0 else [(o["a"], 1 << (nM + nK)), (o["b"], 1 << (nN + nK))]
            if o["kind"] != 0 and not fused:
                refs.append((o["c"], 1 << (nM + nN)))
            used.update({r[1]: s for r, s in refs if r[0] == 0})
        end = 0
        for off in sorted(used):
            assert off >= end
            end = off + used[off]
        assert end * ELEM[dtype] <= info["arena_bytes"]
    assert True in seen


def test_small_network():
    c = make_rqc(3, 4, 8, seed=3)
    open_q = [9, 10, 11]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    plan = tnrcs.Plan(c, pairs, slice_to_fit(ns, pairs, 11), open_q, random_bitstrings(12, 1, seed=3)[0], dry_run=True)
    assert plan.json()["small_net"] and plan.info()["n_kernels"] == 1
    plan.close()

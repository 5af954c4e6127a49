"""Rounding of long sums into few outputs in a network that one workgroup
contracts: the one device step (everything else is folded on the host) against
the FP64 sum of the same FP32 leaves.

A chain of N additions of random sign rounds N times, each time by at most
u = 2^-24 of the sum so far: a relative error of u sqrt(N / 6).  Terms are
added four (eight additions) at a time, then in a tree of degree four, then by
the 2^L lanes of an output in a binary one (two thirds of a rounding per level
and half of that); one chain per lane would be 2^(nK + 1 - L) long."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402
from tests.plan_interp import PlanInterpreter  # noqa: E402


# grid, cycles, open qubits: a step of 2^nM x 2^nN outputs over 2^nK terms
@pytest.mark.parametrize("rows,cols,cycles,n_open,extents", [(4, 4, 8, 0, (0, 0, 12)), (2, 5, 12, 4, (4, 0, 10)),
                                                             (2, 6, 12, 4, (2, 2, 11)), (3, 6, 8, 6, (3, 3, 9))])
def test_long_sum_error(rows, cols, cycles, n_open, extents):
    print(f"small-network sum {extents}", flush=True)
    c = make_rqc(rows, cols, cycles, seed=3)
    n = c.n_qubits
    open_q = sorted(list(range(n_open // 2)) + list(range(n - n_open + n_open // 2, n)))
    strings = random_bitstrings(n, 32, seed=7)
    pairs = bisection_order(network_structure(c, open_q), seed=0)
    plan = tnrcs.Plan(c, pairs, [], open_q, strings[0], host_fold_log2=14)
    js = plan.json()
    assert js["small_net"] and [(s["nM"], s["nN"], s["nK"]) for s in js["steps"]] == [extents]
    err = ref2 = 0.0
    for bits in strings:
        plan.set_output_bits(bits)
        it = PlanInterpreter(plan)
        it.leaves = it.leaves.astype(np.complex64).astype(np.complex128)
        ref = np.zeros(1 << n_open, dtype=np.complex128)
        it.run_slice(0, ref)
        amp = torch.zeros(1 << n_open, dtype=torch.complex128, device="cuda")
        plan.contract(0, 1, amp)
        torch.cuda.synchronize()
        err += np.sum(np.abs(amp.cpu().numpy() - ref) ** 2)
        ref2 += np.sum(np.abs(ref) ** 2)
    plan.close()
    lanes = max(0, min(6, extents[2], 8 - extents[0] - extents[1]))
    levels = (extents[2] - lanes - 2 + 1) // 2  # of degree four, above the first four terms
    bound = 2.0 ** -24 * np.sqrt((8 + 4 * levels + 2 * lanes) / 6)
    print(f"error {np.sqrt(err / ref2):.2e}, bound {bound:.2e}", flush=True)
    assert np.sqrt(err / ref2) <= bound

"""tn_plan_profile adds the same slice result as tn_contract_slices, bit for
bit: networks contracted by one workgroup and networks of separate kernels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402


@pytest.mark.parametrize("dtype", ["c64", "f16s"])
@pytest.mark.parametrize("net,small", [((3, 3, 7, 9, 9), True), ((3, 4, 8, 3, 11), True), ((3, 4, 7, 12, 12), True),
                                       ((3, 5, 8, 15, 15), False)])
def test_profile_adds_the_slice(net, small, dtype):
    print(f"profile result {net} {dtype}", flush=True)
    rows, cols, cycles, n_open, cap = net
    c = make_rqc(rows, cols, cycles, seed=3)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    bits = random_bitstrings(c.n_qubits, 1, seed=3)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    plan = tnrcs.Plan(c, pairs, slice_to_fit(ns, pairs, cap), open_q, bits, dtype=dtype)
    assert plan.json()["small_net"] == small
    s = plan.info()["n_slices"] - 1
    a = torch.full((1 << n_open,), 0.5 - 0.25j, dtype=torch.complex128, device="cuda")
    b = a.clone()
    ms = plan.profile(s, a)
    plan.contract(s, s + 1, b)
    torch.cuda.synchronize()
    assert len(ms) == len(plan.json()["ops"]) + 1 and np.all(np.asarray(ms) > 0)
    plan.close()
    assert torch.equal(a, b)

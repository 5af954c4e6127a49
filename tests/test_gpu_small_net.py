"""Networks whose slice is contracted by one workgroup in one launch: against
the oracle's state vector, the same sum for every split of the slice range and
from a batch, and the rule that selects them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402

TOL = {"c64": 1e-5, "f16s": 1e-2, "bf16s": 6e-2}


def _net(rows, cols, cycles, n_open, cap, seed=3):
    c = make_rqc(rows, cols, cycles, seed=seed)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    bits = random_bitstrings(c.n_qubits, 1, seed=seed)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    sliced = slice_to_fit(ns, pairs, cap) if cap else []
    return c, open_q, bits, pairs, sliced


def _sum(plan, n_open, cuts):
    amp = torch.zeros(1 << n_open, dtype=torch.complex128, device="cuda")
    for a, b in zip(cuts[:-1], cuts[1:]):
        plan.contract(a, b, amp)
    torch.cuda.synchronize()
    return amp.cpu().numpy()


@pytest.mark.parametrize("dtype", ["c64", "f16s", "bf16s"])
@pytest.mark.parametrize("shape", [(3, 3, 4, 0, 0), (3, 3, 7, 9, 0), (2, 5, 5, 10, 0), (3, 4, 8, 3, 11), (3, 4, 7, 12, 0),
                                   (3, 4, 8, 2, 5), (4, 4, 8, 2, 12), (3, 6, 8, 6, 13)])
def test_small_network_vs_statevector(dtype, shape):
    print(f"small network {dtype} {shape}", flush=True)
    c, open_q, bits, pairs, sliced = _net(*shape)
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype=dtype)
    assert plan.json()["small_net"]
    n = plan.info()["n_slices"]
    got = _sum(plan, len(open_q), [0, n])
    assert plan.status() == 0
    assert oracle.relative_error_norm(got, oracle.amplitudes_sv(c, open_q, bits)) < TOL[dtype]
    if n > 1:
        assert np.array_equal(got, _sum(plan, len(open_q), [0, 1, n // 2 + 1, n]))
        assert np.array_equal(got, _sum(plan, len(open_q), list(range(n + 1))) if n <= 64 else got)
        amp = torch.zeros(1 << len(open_q), dtype=torch.complex128, device="cuda")
        tnrcs.tn_contract_batch([plan], [(0, n)], [amp])
        assert np.array_equal(got, amp.cpu().numpy())
        if dtype != "c64":
            amp.zero_()
            assert plan.contract_checked(0, n, amp) == 0
            torch.cuda.synchronize()
            assert oracle.relative_error_norm(amp.cpu().numpy(), got) < 1e-12
    plan.close()


def test_more_slices_than_one_launch_takes():
    # 2^13 slices: two launches of 4096
    c = make_rqc(3, 4, 8, seed=5)
    open_q = [11]
    bits = random_bitstrings(12, 1, seed=5)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    sliced = []
    for cap in range(14, 1, -1):
        sliced = slice_to_fit(ns, pairs, cap)
        if len(sliced) >= 13:
            break
    sliced = sliced[:13]
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits, host_fold_log2=8)
    n = plan.info()["n_slices"]
    assert n == 1 << 13 and plan.json()["small_net"]
    got = _sum(plan, 1, [0, n])
    assert oracle.relative_error_norm(got, oracle.amplitudes_sv(c, open_q, bits)) < 1e-5
    assert np.array_equal(got, _sum(plan, 1, [0, 5000, 5001, n]))
    plan.close()


def test_range_flags_and_new_bits():
    c, open_q, bits, pairs, sliced = _net(3, 4, 8, 3, 11)
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype="f16s")
    assert plan.json()["small_net"]
    n = plan.info()["n_slices"]
    other = 1 - bits
    plan.set_output_bits(other)
    got = _sum(plan, 3, [0, n])
    assert oracle.relative_error_norm(got, oracle.amplitudes_sv(c, open_q, other)) < 1e-2
    plan.shift_outputs(-20)  # results 2^20 too large for the format
    _sum(plan, 3, [0, n])
    assert plan.status() & tnrcs.FLAG_OVERFLOW
    plan.close()


def test_wide_steps_stay_on_their_kernels():
    c, open_q, bits, pairs, sliced = _net(3, 5, 8, 15, 0)
    plan = tnrcs.Plan(c, pairs, sliced, open_q, bits, dry_run=True)
    assert not plan.json()["small_net"]
    plan.close()

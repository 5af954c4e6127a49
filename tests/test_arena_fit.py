"""A workspace or budget that holds a plan without the scratch that only gains
speed (slabs of GEMM sums below 1024 terms per slab) is enough: such a plan is
made with fewer slabs instead of being refused."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402
from tests.plan_interp import PlanInterpreter  # noqa: E402

# grid, cycles, open qubits: networks with one or two split GEMMs at the
# arena's largest extent
NETS = [(3, 6, 8, 16), (4, 4, 8, 16), (4, 5, 8, 16)]
CASES = [(NETS[0], "c64"), (NETS[1], "c64"), (NETS[2], "c64"), (NETS[0], "f16s"), (NETS[1], "f16s")]


def _net(rows, cols, cycles, n_open):
    c = make_rqc(rows, cols, cycles, seed=3)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    bits = random_bitstrings(c.n_qubits, 1, seed=3)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    return c, pairs, slice_to_fit(ns, pairs, 20), open_q, bits


def _slab_terms(plan):
    return [o["K"] // o["split_k"] for o in plan.json()["ops"] if o["kind"] == 1 and o["split_k"] > 1]


@pytest.mark.parametrize("net,dtype", CASES)
def test_fewer_slabs_in_a_smaller_budget(net, dtype):
    args = _net(*net)
    full = tnrcs.Plan(*args, dtype=dtype, dry_run=True)
    need = full.info()["arena_bytes"] + full.info()["leaf_bytes"]
    assert min(_slab_terms(full)) < 1024
    same = tnrcs.Plan(*args, dtype=dtype, dry_run=True, arena_bytes=need)
    assert same.json() == full.json()
    small = tnrcs.Plan(*args, dtype=dtype, dry_run=True, arena_bytes=need - 1)
    assert small.info()["arena_bytes"] + small.info()["leaf_bytes"] < need
    assert all(x >= 1024 for x in _slab_terms(small))
    for p in (full, same, small):
        p.close()


def test_smaller_plan_has_the_same_value():
    args = _net(*NETS[0])
    small = tnrcs.Plan(*args, dry_run=True, arena_bytes=1)
    it = PlanInterpreter(small)
    amp = np.zeros(1 << len(args[3]), dtype=np.complex128)
    for s in range(small.info()["n_slices"]):
        it.run_slice(s, amp)
    small.close()
    assert oracle.relative_error_norm(amp, oracle.amplitudes_sv(args[0], args[3], args[4])) < 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("net,dtype", CASES)
def test_runs_in_the_smaller_workspace(net, dtype):
    print(f"smaller workspace {net} {dtype}", flush=True)
    args = _net(*net)
    dry = tnrcs.Plan(*args, dtype=dtype, dry_run=True, arena_bytes=1)
    need = dry.info()["arena_bytes"]
    dry.close()
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    plan = tnrcs.Plan(*args, dtype=dtype, arena=ws)
    assert plan.info()["arena_bytes"] == need
    amp = torch.zeros(1 << len(args[3]), dtype=torch.complex128, device="cuda")
    plan.contract(0, plan.info()["n_slices"], amp)
    torch.cuda.synchronize()
    plan.close()
    ref = oracle.amplitudes_sv(args[0], args[3], args[4])
    assert oracle.relative_error_norm(amp.cpu().numpy(), ref) < {"c64": 1e-5, "f16s": 1e-2}[dtype]
    with pytest.raises(tnrcs.TnError, match="arena"):
        tnrcs.Plan(*args, dtype=dtype, arena=ws[: need - 256])

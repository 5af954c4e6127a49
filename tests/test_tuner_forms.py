"""The class tuner times a step in the form that the tuned plan runs: an FP16
GEMM over a short sum whose A has 2^17 to 2^19 entries is read in place by an
untuned plan, and permuted for a tuned tile by a tuned one."""
import math

import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402

# grid, cycles, open qubits, largest tensor; the step's extents (bits)
NETS = [((4, 4, 8, 10, 20), (12, 8, 6)), ((4, 5, 8, 16, 22), (11, 8, 6))]


def _net(rows, cols, cycles, n_open, cap):
    c = make_rqc(rows, cols, cycles, seed=3)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    bits = random_bitstrings(c.n_qubits, 1, seed=3)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    return c, pairs, slice_to_fit(ns, pairs, cap), open_q, bits


def _gemm(plan, extents):
    g = [o for o in plan.json()["ops"] if o["kind"] == 1 and tuple(int(math.log2(o[x])) for x in "MNK") == extents]
    assert g
    return g[0]


@pytest.mark.parametrize("net,extents", NETS)
def test_forms_differ(net, extents):
    args = _net(*net)
    for tune in (False, True):
        plan = tnrcs.Plan(*args, dtype="f16s", dry_run=True, tune=tune)
        assert _gemm(plan, extents)["ga"] == (0 if tune else 1)
        plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("net,extents", NETS)
def test_class_timed_with_the_tuned_tile(net, extents, tmp_path):
    # timing the permuted form tunes its tile first, so that the tile's line
    # precedes the class's; timing another form leaves the tile for later
    print(f"tuner forms {net}", flush=True)
    args = _net(*net)
    db = tmp_path / "tune.txt"
    plan = tnrcs.Plan(*args, dtype="f16s", tune=True, tune_db=str(db))
    step = next(s for s in plan.json()["steps"] if (s["nM"], s["nN"], s["nK"]) == extents)
    lines = [x.split() for x in db.read_text().splitlines()]
    tile = next(i for i, x in enumerate(lines) if x[0] == "tnrcs-gemm" and x[2:5] == [str(1 << e) for e in extents])
    cls = next(i for i, x in enumerate(lines) if x[0] == "tnrcs-class" and x[2] == step["key"])
    assert tile < cls
    amp = torch.zeros(1 << len(args[3]), dtype=torch.complex128, device="cuda")
    plan.contract(0, plan.info()["n_slices"], amp)
    torch.cuda.synchronize()
    plan.close()
    assert oracle.relative_error_norm(amp.cpu().numpy(), oracle.amplitudes_sv(args[0], args[3], args[4])) < 1e-2

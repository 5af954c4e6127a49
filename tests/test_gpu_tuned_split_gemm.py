"""Tuned complex64 plans whose GEMMs may be split: every tile and split that the
tuner tries runs, 64x64 tiles with slabs among them."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit  # noqa: E402
from rqcgen.order import bisection_order  # noqa: E402


@pytest.mark.parametrize("form", ["3m", "4m"])
@pytest.mark.parametrize("rows,cols,cycles,n_open,mnk", [(3, 6, 8, 16, (256, 256, 512)), (3, 6, 10, 12, (64, 64, 16384))])
def test_plan_and_result(rows, cols, cycles, n_open, mnk, form, tmp_path):
    print(f"tuned split GEMM {mnk} {form}", flush=True)
    c = make_rqc(rows, cols, cycles, seed=3)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    bits = random_bitstrings(c.n_qubits, 1, seed=3)[0]
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    db = tmp_path / "tune.txt"
    plan = tnrcs.Plan(c, pairs, slice_to_fit(ns, pairs, 20), open_q, bits, tune=True, tune_db=str(db), gemm_form=form)
    gemms = [o for o in plan.json()["ops"] if o["kind"] == 1 and (o["M"], o["N"], o["K"]) == mnk]
    assert gemms and all(o["ga"] == 0 and o["split_max"] > 1 for o in gemms)
    amp = torch.zeros(1 << n_open, dtype=torch.complex128, device="cuda")
    plan.contract(0, plan.info()["n_slices"], amp)
    torch.cuda.synchronize()
    plan.close()
    assert oracle.relative_error_norm(amp.cpu().numpy(), oracle.amplitudes_sv(c, open_q, bits)) < 1e-5

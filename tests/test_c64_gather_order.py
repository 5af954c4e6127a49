"""complex64 GEMMs that read A in place: the order of the chunk's k bits (those
among A's positions 1 to 6 of the chunk get the swizzled numbers 3, 0, 1 first),
no permute of a B that is [columns, K] in A's order, and the results for k
bits crowded in A's lowest positions, against FP64 (an FP32 sum of n products of
random sign stays within 2^-24 sqrt(n) normwise)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2111_01066_amd import tnrcs  # noqa: E402

CASES = [(14, 7, [1, 2, 3, 4, 5, 9]), (13, 8, [0, 2, 3, 4, 7, 11, 12]), (14, 7, [0, 1, 2, 3, 8, 9]),
         (14, 7, [7, 8, 9, 10, 11, 12]), (13, 7, [2, 4, 5, 6, 9, 10, 11])]


def _labels(nM, nN, ks, aligned):
    la, m = [], 0
    for p in range(nM + len(ks)):
        if p in ks:
            la.append(100 + ks.index(p))
        else:
            la.append(m)
            m += 1
    la = la[::-1]
    n, k = list(range(50, 50 + nN)), [x for x in la if x >= 100]
    return la, n + (k if aligned else k[::-1]), [x for x in la if x < 50] + n


def _gemm(nM, nN, ks, aligned):
    pp = tnrcs.PairPlan(*_labels(nM, nN, ks, aligned), dry_run=True)
    ops = pp.json()["ops"]
    pp.close()
    assert ops[-1]["ga"] == 1
    return ops, [next(d + j - s for s, d, ln in ops[-1]["aK"] if s <= j < s + ln) for j in range(len(ks))]


@pytest.mark.parametrize("nM,nN,ks", CASES)
def test_k_order(nM, nN, ks):
    ops, pos = _gemm(nM, nN, ks, aligned=True)
    assert len(ops) == 1 and pos == ks
    ops, pos = _gemm(nM, nN, ks, aligned=False)
    assert len(ops) == 2 and pos[4:] == ks[4:]
    chunk = sorted(ks[:4] + [p for p in range(nM + len(ks)) if p not in ks][:7])
    lanes = [p for p in ks[:4] if p in chunk[1:7]]
    others = [p for p in ks[:4] if p not in lanes]
    assert [pos[i] for i in (3, 0, 1, 2)] == lanes + others


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["3m", "4m"])
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("nM,nN,ks", CASES)
def test_result(nM, nN, ks, aligned, form):
    print(f"complex64 A in place {nM} {nN} {ks} {aligned} {form}", flush=True)
    la, lb, lc = _labels(nM, nN, ks, aligned)
    nK = len(ks)
    rng = np.random.default_rng(nM + 10 * nN + nK)
    A, B = (torch.from_numpy(rng.standard_normal((1 << len(x), 2)).astype(np.float32)) for x in (la, lb))
    C = torch.empty(1 << len(lc), 2, device="cuda")
    pp = tnrcs.PairPlan(la, lb, lc, gemm_form=form)
    pp.run(A.cuda(), B.cuda(), C)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    k = [x for x in la if x >= 100]
    a = a.reshape((2,) * len(la)).transpose([la.index(x) for x in la if x < 50] + [la.index(x) for x in k])
    b = b.reshape((2,) * len(lb)).transpose(list(range(nN)) + [lb.index(x) for x in k])
    ref = (a.reshape(1 << nM, 1 << nK) @ b.reshape(1 << nN, 1 << nK).T).reshape(-1)
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    assert np.linalg.norm(got - ref) <= 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK) * np.linalg.norm(ref)

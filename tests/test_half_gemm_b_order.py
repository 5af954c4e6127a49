"""16-bit GEMMs that read A in place, with B stored as [columns, K] in A's K
order: no permute of B, whichever bits A's 16-byte loads cover; results
against FP64 sums of the same rounded inputs (an FP32 sum of n products of random
sign stays within 2^-24 sqrt(n) normwise, the result is rounded once to 16 bits)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2111_01066_amd import tnrcs  # noqa: E402

UNIT = {"f16s": 2.0 ** -11, "bf16s": 2.0 ** -8}
# rows, columns, k positions in A: both, one or none of bits 0 and 1; the
# second and third k bits low or high; one stage of 32 k, several, slabs
CASES = [(13, 7, [0, 1, 4, 9, 12, 15]), (13, 8, [0, 2, 3, 4, 17]), (12, 7, [0, 9, 12, 14, 15, 17]),
         (13, 7, [1, 2, 5, 8, 11, 14, 17]), (12, 9, [1, 10, 11, 13, 15, 16]), (13, 7, [2, 3, 4, 5, 6]),
         (11, 8, [3, 7, 10, 12, 14, 15, 17, 18]), (8, 7, [2, 4, 5, 7, 9, 10, 12, 13, 15, 16]),
         (14, 7, [14, 15, 16, 17, 18])]


def _labels(nM, nN, ks):
    la, m = [], 0
    for p in range(nM + len(ks)):
        if p in ks:
            la.append(100 + ks.index(p))
        else:
            la.append(m)
            m += 1
    la = la[::-1]
    n, k = list(range(50, 50 + nN)), [x for x in la if x >= 100]
    return la, n + k, [x for x in la if x < 50] + n


@pytest.mark.parametrize("nM,nN,ks", CASES)
def test_no_permute_of_b(nM, nN, ks):
    pp = tnrcs.PairPlan(*_labels(nM, nN, ks), dtype="f16s", dry_run=True)
    ops = pp.json()["ops"]
    pp.close()
    assert [o["kind"] for o in ops] == [1] and ops[0]["ga"] == 1


# B as [columns, K] in another order: short sums into few rows permute A
# (False), others B and read A in place
@pytest.mark.parametrize("nM,nN,nK,in_place", [(12, 7, 5, False), (13, 12, 5, False), (13, 9, 6, False), (14, 9, 5, True),
                                               (12, 10, 7, True), (15, 7, 5, True)])
def test_one_permute(nM, nN, nK, in_place):
    ks = [2 + 2 * i for i in range(nK)]
    la, lb, lc = _labels(nM, nN, ks)
    lb = lb[:nN] + lb[nN:][::-1]
    pp = tnrcs.PairPlan(la, lb, lc, dtype="f16s", dry_run=True)
    ops = pp.json()["ops"]
    pp.close()
    assert [o["kind"] for o in ops] == [0, 1] and ops[1]["ga"] == in_place
    assert ops[0]["rank"] == (nN + nK if in_place else nM + nK)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16s", "bf16s"])
@pytest.mark.parametrize("nM,nN,ks", CASES)
def test_result(dtype, nM, nN, ks):
    print(f"16-bit GEMM, B in A's order {dtype} {nM} {nN} {ks}", flush=True)
    la, lb, lc = _labels(nM, nN, ks)
    nK = len(ks)
    t = torch.float16 if dtype == "f16s" else torch.bfloat16
    rng = np.random.default_rng(nM + 10 * nN + nK)
    A = torch.from_numpy(rng.standard_normal((1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((1 << len(lb), 2))).to(t)
    C = torch.empty(1 << len(lc), 2, dtype=t, device="cuda")
    scale = 2.0 ** -(nK // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype)
    pp.run(A.cuda(), B.cuda(), C, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    a = a.reshape((2,) * len(la)).transpose([la.index(x) for x in la if x < 50] + [la.index(x) for x in la if x >= 100])
    ref = (a.reshape(1 << nM, 1 << nK) @ b.reshape(1 << nN, 1 << nK).T).reshape(-1) * scale
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK) + UNIT[dtype]
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)

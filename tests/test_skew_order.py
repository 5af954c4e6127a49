"""16-bit skewed steps: which of the two K orders a step takes (in A's order
with its entries stored one by one, or reordered for stores of four k), and
the results of steps that keep A's order, against FP64 sums of the same rounded
inputs (an FP32 sum of n products of random sign stays within 2^-24 sqrt(n)
normwise, the result is rounded once to 16 bits)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2111_01066_amd import tnrcs  # noqa: E402

UNIT = {"f16s": 2.0 ** -11, "bf16s": 2.0 ** -8}


def _labels(nM, nN, ks, b_in_a_order=False):
    """A with its k bits at positions ks, its rows elsewhere; natural output order."""
    la, m = [], 0
    for p in range(nM + len(ks)):
        if p in ks:
            la.append(100 + ks.index(p))
        else:
            la.append(m)
            m += 1
    la = la[::-1]
    n, k = list(range(50, 50 + nN)), [x for x in la if x >= 100]
    lb = n + k if b_in_a_order else [int(x) for x in np.random.default_rng(nN).permutation(n + k)]
    return la, lb, [x for x in la if x < 50] + [x for x in lb if 50 <= x < 100]


def _plan(nM, nN, ks, aligned):
    pp = tnrcs.PairPlan(*_labels(nM, nN, ks, aligned), dtype="f16s", dry_run=True)
    js = pp.json()
    pp.close()
    op = js["ops"][-1]
    pos = [next(d + j - s for s, d, l in op["aK"] if s <= j < s + l) for j in range(len(ks))]
    return js, op["kind"], pos


# rows, columns, k positions in A, B in A's K order; whether K keeps A's order
PLANS = [(25, 4, [4, 7, 13, 14], False, True), (26, 4, [0, 4, 10, 17, 21], False, True),
         (26, 4, [4, 8, 11, 14], False, True), (23, 6, [1, 7, 9, 23, 24], False, True),
         (24, 5, [1, 10, 13, 25], False, True), (22, 6, [0, 16, 19, 20, 21], False, True),
         (14, 4, [0, 4, 5, 9, 10], False, True), (20, 4, [3, 4, 9, 10], False, True), (24, 4, [5, 18, 23, 24], False, True),
         (22, 5, [16, 19, 20, 22], False, False), (23, 4, [0, 17, 22, 23], False, False),
         (12, 4, [0, 4, 5, 9, 10], False, False), (19, 4, [3, 4, 9, 10], False, False), (23, 4, [5, 18, 23, 24], False, False),
         (24, 3, [4, 7, 13, 14], False, False),
         (22, 5, [0, 4, 5, 21, 22, 23], False, False), (19, 5, [2, 4, 5, 8, 10, 12, 21, 23, 24], False, False),
         (10, 5, [3, 5, 6, 8, 9, 11, 13, 15], True, True), (19, 5, [3, 5, 6, 8, 9, 11, 13, 15], True, False)]


@pytest.mark.parametrize("nM,nN,ks,aligned,plain", PLANS)
def test_order_rule(nM, nN, ks, aligned, plain):
    js, kind, pos = _plan(nM, nN, ks, aligned)
    assert kind == 5
    assert (pos == ks) == plain
    if aligned:
        assert len(js["ops"]) == (1 if plain else 2)  # a permute of B


# every pair of low bits of A (row or k) with K in A's order: one chunk, two,
# and B staged chunk by chunk; few passes of 128 rows
RUNS = [(20, 4, [4, 7, 8, 9], False), (20, 6, [0, 3, 8, 9], False), (20, 5, [1, 4, 9, 12], False),
        (20, 4, [0, 1, 9, 12], False), (13, 4, [0, 4, 8, 9, 12], False), (13, 6, [1, 5, 8, 9, 12], False),
        (13, 3, [0, 1, 5, 9, 17], False), (13, 1, [2, 3, 4, 5, 6], False),
        (10, 5, [2, 3, 5, 6, 8, 9, 11], True), (8, 5, [0, 3, 5, 6, 8, 9, 11, 12], True),
        (7, 5, [1, 3, 5, 6, 8, 9, 11, 12, 14], True), (7, 4, [3, 4, 5, 6, 8, 9, 10, 12, 14, 16], True)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16s", "bf16s"])
@pytest.mark.parametrize("nM,nN,ks,aligned", RUNS)
def test_entry_by_entry(dtype, nM, nN, ks, aligned):
    print(f"skewed step in A's order {dtype} {nM} {nN} {ks}", flush=True)
    js, kind, pos = _plan(nM, nN, ks, aligned)
    assert kind == 5 and pos == ks and len(js["ops"]) == 1
    la, lb, lc = _labels(nM, nN, ks, aligned)
    nK = len(ks)
    t = torch.float16 if dtype == "f16s" else torch.bfloat16
    rng = np.random.default_rng(nM + 10 * nN)
    A = torch.from_numpy(rng.standard_normal((1 << len(la), 2))).to(t)
    B = torch.from_numpy(rng.standard_normal((1 << len(lb), 2))).to(t)
    C = torch.empty(1 << len(lc), 2, dtype=t, device="cuda")
    scale = 2.0 ** -(nK // 2)
    pp = tnrcs.PairPlan(la, lb, lc, dtype=dtype)
    pp.run(A.cuda(), B.cuda(), C, out_scale=scale)
    torch.cuda.synchronize()
    pp.close()
    a, b = (x.double().numpy() @ np.array([1.0, 1j]) for x in (A, B))
    k = [x for x in la if x >= 100]
    a = a.reshape((2,) * len(la)).transpose([la.index(x) for x in lc if x < 50] + [la.index(x) for x in k])
    b = b.reshape((2,) * len(lb)).transpose([lb.index(x) for x in k] + [lb.index(x) for x in lc if x >= 50])
    ref = (a.reshape(-1, 1 << nK) @ b.reshape(1 << nK, -1)).reshape(-1) * scale
    got = C.cpu().double().numpy() @ np.array([1.0, 1j])
    bound = 2.0 ** -24 * 4 * np.sqrt(4.0 * 2 ** nK) + UNIT[dtype]
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref)

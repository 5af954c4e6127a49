"""Performance cases: the work that programs have this library do, through
its public entry points.

Six kinds of case, each with the sizes of the repository's own workloads
(rqcgen/workloads.py, bench.py, tests/):

* net      every slice of one circuit's network (or one slice of the 53-qubit
           network) by Plan.contract: the amplitude bunch of a bit string;
* batch    bunches of several uneven circuits in scaled storage by one Batch;
* pair     one pairwise contraction of labelled tensors by PairPlan.run, in
           the shapes that network steps have: dense (wide on both sides),
           short-sum dense, skewed (few outputs per row), long-sum (few
           outputs), a gate on a state;
* gemm     the complex matrix product on its own, at sizes that are no powers
           of two;
* readout  what is done with the amplitudes of an all-open run: norm,
           cross-entropy sums, the Porter-Thomas histogram and frugal
           sampling.

Plans are made with the default rules (no tuner), so that two runs choose the
same kernels.
"""
from __future__ import annotations

import functools

import numpy as np
import torch

from paper_2111_01066_amd import tnrcs
from rqcgen import make_rqc, network_structure, random_bitstrings, slice_to_fit
from rqcgen.order import bisection_order
from rqcgen.workloads import config3, config5, config5_table

DEV = "cuda"
ELEM = {"c64": 8, "f16s": 4, "bf16s": 4}
HALF = {"f16s": torch.float16, "bf16s": torch.bfloat16}


def listed():
    return [
        # the smallest calls: a 12-qubit circuit, 3 open qubits, 16 slices of a
        # handful of tiny kernels; latency and launches count
        {"name": "net-12q-sliced-c64", "kind": "net", "rows": 3, "cols": 4, "cycles": 8, "open": 3, "cap": 11,
         "dtype": "c64"},
        # all 2^20 amplitudes of a 20-qubit circuit
        {"name": "net-20q-open-c64", "kind": "net", "rows": 4, "cols": 5, "cycles": 8, "open": 20, "cap": 40,
         "dtype": "c64"},
        # one slice of the 53-qubit, 14-cycle network (a bunch of 64), tensors
        # of at most 2^31 entries
        {"name": "net-53q-slice-c64", "kind": "net53", "cap": 31, "dtype": "c64"},
        # eight circuits of the uneven batch (24-40 qubits), one call
        {"name": "batch-uneven-f16s", "kind": "batch", "first": 40, "count": 8, "max_flops": 1e12, "lanes": 4,
         "dtype": "f16s"},
        # compute-bound pairs with scattered indices (rank 27 x rank 25 sharing
        # 12 in scaled FP16, a smaller one in complex64)
        {"name": "pair-dense-f16s", "kind": "pair", "nM": 15, "nN": 13, "nK": 12, "layout": 2, "batch": 1,
         "dtype": "f16s"},
        {"name": "pair-dense-c64", "kind": "pair", "nM": 13, "nN": 11, "nK": 11, "layout": 3, "batch": 2,
         "dtype": "c64"},
        # a wide step over a short sum, as most dense steps of the 53-qubit network
        {"name": "pair-short-bf16s", "kind": "pair", "nM": 21, "nN": 7, "nK": 6, "layout": 4, "batch": 1,
         "dtype": "bf16s"},
        # few outputs per row: the commonest large step of a slice
        {"name": "pair-skew-c64", "kind": "pair", "nM": 22, "nN": 4, "nK": 5, "layout": 5, "batch": 1,
         "dtype": "c64"},
        # the same with a large small operand
        {"name": "pair-skew-long-f16s", "kind": "pair", "nM": 20, "nN": 5, "nK": 9, "layout": 6, "batch": 1,
         "dtype": "f16s"},
        # two large tensors into 64 outputs: the last step of a slice
        {"name": "pair-longsum-c64", "kind": "pair", "nM": 3, "nN": 3, "nK": 24, "layout": 7, "batch": 1,
         "dtype": "c64"},
        # matrix products of ragged sizes
        {"name": "gemm-ragged-c64", "kind": "gemm", "M": 1984, "N": 1088, "K": 1200, "batch": 3, "splits": 1,
         "form": "3m", "dtype": "c64"},
        # the amplitudes of a 24-qubit all-open run
        {"name": "readout-24q", "kind": "readout", "n": 1 << 24, "samples": 100_000, "bins": 64, "bunches": 4096},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(["net", "net", "batch", "pair", "pair", "pair", "pair", "gemm", "gemm", "readout"])
    dtype = rng.choice(["c64", "c64", "f16s", "bf16s"])
    if kind == "net":
        rows, cols = rng.choice([(2, 5), (3, 3), (3, 4), (3, 5), (4, 4), (3, 6), (4, 5), (3, 7)])
        n = rows * cols
        return {"kind": "net", "rows": rows, "cols": cols, "cycles": rng.randint(4, 10), "dtype": dtype,
                "open": rng.choice([rng.randint(0, 6), n if n <= 16 else 6]), "cap": rng.randint(12, 24)}
    if kind == "batch":
        return {"kind": "batch", "first": rng.randint(0, 150), "count": rng.randint(2, 8), "dtype": "f16s",
                "max_flops": 10.0 ** rng.uniform(10.5, 11.9), "lanes": rng.randint(1, 4)}
    if kind == "pair":
        shape = rng.choice(["dense", "short", "skew", "gate", "longsum", "small"])
        if shape == "dense":
            nM, nN, nK = rng.randint(7, 14), rng.randint(6, 12), rng.randint(7, 12)
        elif shape == "short":
            nM, nN, nK = rng.randint(10, 20), rng.randint(7, 9), rng.randint(2, 7)
        elif shape == "skew":
            nM, nN, nK = rng.randint(12, 21), rng.randint(1, 6), rng.randint(3, 9)
        elif shape == "gate":
            nM, nN, nK = rng.randint(10, 24), rng.randint(1, 2), rng.randint(1, 2)
        elif shape == "longsum":
            nM, nN, nK = rng.randint(0, 3), rng.randint(0, 3), rng.randint(12, 23)
        else:
            nM, nN, nK = rng.randint(2, 7), rng.randint(0, 5), rng.randint(1, 8)
        return {"kind": "pair", "nM": nM, "nN": nN, "nK": nK, "layout": rng.randint(0, 10**6),
                "batch": rng.randint(1, 3), "dtype": dtype}
    if kind == "gemm":
        M, N = 64 * log_int(1, 40), 64 * log_int(1, 40)
        splits = rng.choice([1, 1, 2, 4])
        return {"kind": "gemm", "M": M, "N": N, "K": 16 * splits * log_int(1, 160 // splits), "splits": splits,
                "batch": 1 if splits > 1 else rng.randint(1, 3), "form": rng.choice(["3m", "4m"]), "dtype": dtype}
    return {"kind": "readout", "n": log_int(1 << 10, 1 << 24), "samples": log_int(1000, 100_000),
            "bins": rng.randint(8, 200), "bunches": log_int(16, 4096)}


# ------------------------------------------------------------------ inputs --

@functools.lru_cache(maxsize=64)
def _order(rows, cols, cycles, n_open, cap):
    """Open qubits, contraction order and sliced wires of a grid circuit
    (they depend on the circuit's structure, not on its gates)."""
    c = make_rqc(rows, cols, cycles, seed=0)
    open_q = list(range(c.n_qubits - n_open, c.n_qubits))
    ns = network_structure(c, open_q)
    pairs = bisection_order(ns, seed=0)
    return open_q, pairs, slice_to_fit(ns, pairs, max(cap, n_open))


@functools.lru_cache(maxsize=4)
def _order53(cap):
    w = config3()
    return w, slice_to_fit(network_structure(w.circuit, w.open_qubits), w.pairs, cap, initial=w.sliced)


def _bits(n, open_q, seed):
    b = random_bitstrings(n, 1, seed=seed)[0]
    b[list(open_q)] = 0
    return b


def _net(case, seed):
    """Circuit, open qubits, closed bits, order, sliced wires, slice range."""
    if case["kind"] == "net53":
        w, sliced = _order53(case["cap"])
        s = seed % (1 << len(sliced))
        return w.circuit, w.open_qubits, _bits(w.circuit.n_qubits, w.open_qubits, seed), w.pairs, sliced, (s, s + 1)
    open_q, pairs, sliced = _order(case["rows"], case["cols"], case["cycles"], case["open"], case["cap"])
    c = make_rqc(case["rows"], case["cols"], case["cycles"], seed=seed)
    return c, open_q, _bits(c.n_qubits, open_q, seed), pairs, sliced, (0, 1 << len(sliced))


def _batch(case, seed):
    t = config5_table()
    ok = [i for i in range(len(t["S"])) if t["total_flops"][i] <= case["max_flops"]]
    at = min(case["first"], max(0, len(ok) - case["count"]))
    nets = []
    for w in config5(indices=ok[at:at + case["count"]], table=t):
        nets.append((w.circuit, w.open_qubits, _bits(w.circuit.n_qubits, w.open_qubits, seed), w.pairs, w.sliced,
                     (0, 1 << len(w.sliced))))
    return nets


def _labels(case):
    """Index labels of a pair: A, B and C each in an order of its own."""
    rng = np.random.default_rng(case["layout"])
    m = list(range(case["nM"]))
    n = list(range(100, 100 + case["nN"]))
    k = list(range(200, 200 + case["nK"]))
    return [[int(x) for x in rng.permutation(v)] if v else [] for v in (m + k, n + k, m + n)]


def _randn(shape, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if dtype == "c64":
        return torch.randn(*shape, dtype=torch.complex64, device=DEV, generator=g)
    return torch.randn(*shape, 2, device=DEV, generator=g).to(HALF[dtype])


def _scale(case, terms):
    return 1.0 if case["dtype"] == "c64" else 2.0 ** -(int(terms).bit_length() // 2)


def _pair_inputs(case, seed):
    la, lb, _ = _labels(case)
    return (_randn((case["batch"], 1 << len(la)), case["dtype"], 2 * seed),
            _randn((case["batch"], 1 << len(lb)), case["dtype"], 2 * seed + 1))


def _gemm_inputs(case, seed):
    M, N, K, b = case["M"], case["N"], case["K"], case["batch"]
    return _randn((b, M, K), case["dtype"], 2 * seed), _randn((b, N, K), case["dtype"], 2 * seed + 1)


def _readout_inputs(case, seed):
    """Porter-Thomas amplitudes, sampled indices, frugal candidates (bunches
    of 64 consecutive entries) and their uniform numbers."""
    n, g = case["n"], torch.Generator(device=DEV)
    g.manual_seed(seed)
    amp = torch.randn(n, dtype=torch.complex128, device=DEV, generator=g) / n ** 0.5
    idx = torch.randint(0, n, (case["samples"],), device=DEV, generator=g)
    start = torch.randint(0, n // 64, (case["bunches"],), device=DEV, generator=g) * 64
    cand = (start[:, None] + torch.arange(64, device=DEV)[None, :]).reshape(-1)
    return amp, idx, cand, torch.rand(cand.numel(), dtype=torch.float64, device=DEV, generator=g)


def _out(shape, dtype):
    if dtype == "c64":
        return torch.empty(*shape, dtype=torch.complex64, device=DEV)
    return torch.empty(*shape, 2, dtype=HALF[dtype], device=DEV)


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind in ("net", "net53"):
        c, open_q, bits, pairs, sliced, rng = _net(case, seed)
        s["plan"] = tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype=case["dtype"])
        s["amp"] = torch.zeros(1 << len(open_q), dtype=torch.complex128, device=DEV)
        s["range"], s["qubits"] = rng, c.n_qubits
    elif kind == "batch":
        nets, lanes = _batch(case, seed), case["lanes"]
        need = 256
        for c, open_q, bits, pairs, sliced, _ in nets:
            with tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype=case["dtype"], dry_run=True) as dry:
                need = max(need, dry.info()["arena_bytes"])
        s["arenas"] = [torch.empty(need, dtype=torch.uint8, device=DEV) for _ in range(lanes)]
        s["plans"] = [tnrcs.Plan(c, pairs, sliced, open_q, bits, dtype=case["dtype"], arena=s["arenas"][i % lanes])
                      for i, (c, open_q, bits, pairs, sliced, _) in enumerate(nets)]
        s["amps"] = torch.zeros(len(nets), 64, dtype=torch.complex128, device=DEV)
        s["qubits"] = torch.tensor([2.0 ** (net[0].n_qubits / 2) for net in nets], dtype=torch.float64,
                                   device=DEV)[:, None]
        s["batch"] = tnrcs.Batch(s["plans"], [net[5] for net in nets], [s["amps"][i] for i in range(len(nets))])
    elif kind == "pair":
        la, lb, lc = _labels(case)
        s["A"], s["B"] = _pair_inputs(case, seed)
        s["C"] = _out((case["batch"], 1 << len(lc)), case["dtype"])
        s["plan"] = tnrcs.PairPlan(la, lb, lc, dtype=case["dtype"])
        s["scale"] = _scale(case, 1 << case["nK"])
    elif kind == "gemm":
        s["A"], s["B"] = _gemm_inputs(case, seed)
        s["C"] = _out((case["batch"], case["M"], case["N"]), case["dtype"])
        s["work"] = (torch.empty(case["splits"], case["M"], case["N"], dtype=torch.complex64, device=DEV)
                     if case["splits"] > 1 else None)
        s["scale"] = _scale(case, case["K"])
    else:
        s["amp"], s["idx"], s["cand"], s["u"] = _readout_inputs(case, seed)
        s["norm"] = torch.zeros(1, dtype=torch.float64, device=DEV)
        s["xeb"] = torch.zeros(2, dtype=torch.float64, device=DEV)
        s["hist"] = torch.zeros(case["bins"], dtype=torch.int64, device=DEV)
        s["kept"] = torch.empty(s["cand"].numel(), dtype=torch.int64, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind, dtype = case["kind"], case.get("dtype")
    if kind in ("net", "net53"):
        s["amp"].zero_()
        s["plan"].contract(s["range"][0], s["range"][1], s["amp"])
        if dtype == "c64":
            return s["amp"].to(torch.complex64)  # the plan's own precision
        # amplitudes over their Porter-Thomas scale, in the plan's storage type
        return torch.view_as_real(s["amp"] * 2.0 ** (s["qubits"] / 2)).to(HALF[dtype])
    if kind == "batch":
        s["amps"].zero_()
        s["batch"].run()
        return torch.view_as_real(s["amps"] * s["qubits"]).to(HALF[dtype])
    if kind == "pair":
        s["plan"].run(s["A"], s["B"], s["C"], batch=case["batch"], out_scale=s["scale"])
        return s["C"]
    if kind == "gemm":
        if dtype == "c64":
            tnrcs.tn_cgemm_c64(s["A"], s["B"], s["C"], case["M"], case["N"], case["K"], case["batch"],
                               form=case["form"], work=s["work"], splits=case["splits"])
        else:
            tnrcs.tn_cgemm_half(dtype, s["A"], s["B"], s["C"], case["M"], case["N"], case["K"], case["batch"],
                                form=case["form"], out_scale=s["scale"], work=s["work"], splits=case["splits"])
        return s["C"]
    n = case["n"]
    s["hist"].zero_()
    s["kept"].fill_(n)
    tnrcs.tn_amp_norm2(s["amp"], n, s["norm"])
    tnrcs.tn_amp_xeb(s["amp"], n, s["idx"], case["samples"], s["xeb"])
    tnrcs.tn_amp_hist(s["amp"], n, float(n), 10.0, case["bins"], s["hist"])
    tnrcs.tn_amp_frugal(s["amp"], n, s["cand"], s["cand"].numel(), s["u"], float(n), 10.0, s["kept"], s["count"])
    # the kept indices come in any order: sorted, behind them the unused places
    return {"norm": s["norm"], "xeb": s["xeb"], "hist": s["hist"], "kept": s["kept"].sort().values,
            "count": s["count"]}


# -------------------------------------------------------- floor and oracle --

def _network(circuit, open_q, bits):
    """The circuit's tensors as (wires, values): |0> vectors, gates, output
    vectors of the closed qubits; and the open wires in qubit order."""
    n = circuit.n_qubits
    leaves = [([q], np.array([1.0, 0.0], dtype=np.complex128)) for q in range(n)]
    cur, nw = list(range(n)), n
    for g in circuit.gates:
        ins = [cur[q] for q in g.qubits]
        outs = list(range(nw, nw + len(ins)))
        nw += len(ins)
        for q, w in zip(g.qubits, outs):
            cur[q] = w
        leaves.append((outs + ins, np.asarray(g.matrix, dtype=np.complex128).reshape(-1)))
    for q in range(n):
        if q not in set(open_q):
            v = np.zeros(2, dtype=np.complex128)
            v[int(bits[q]) & 1] = 1.0
            leaves.append(([cur[q]], v))
    return leaves, [cur[q] for q in sorted(open_q)]


def _net_work(net, eb):
    """Flops and bytes of the order's steps over the slice range: each step
    reads its two operands and writes its result once."""
    c, open_q, bits, pairs, sliced, (s0, s1) = net
    leaves, _ = _network(c, open_q, bits)
    cut = set(sliced)
    sets = [frozenset(w) - cut for w, _ in leaves]
    flops = entries = 0.0
    for a, b in pairs:
        x, y = sets[a], sets[b]
        sets.append(x ^ y)
        flops += 8.0 * 2.0 ** len(x | y)
        entries += 2.0 ** len(x) + 2.0 ** len(y) + 2.0 ** len(x ^ y)
    return flops * (s1 - s0), entries * eb * (s1 - s0)


def work(case):
    kind = case["kind"]
    if kind in ("net", "net53"):
        f, b = _net_work(_net(case, 0), ELEM[case["dtype"]])
    elif kind == "batch":
        per = [_net_work(net, ELEM[case["dtype"]]) for net in _batch(case, 0)]
        f, b = sum(p[0] for p in per), sum(p[1] for p in per)
    elif kind == "pair":
        m, n, k = case["nM"], case["nN"], case["nK"]
        f = case["batch"] * 8.0 * 2.0 ** (m + n + k)
        b = case["batch"] * ELEM[case["dtype"]] * (2.0 ** (m + k) + 2.0 ** (n + k) + 2.0 ** (m + n))
    elif kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        f = case["batch"] * 8.0 * M * N * K
        b = case["batch"] * ELEM[case["dtype"]] * float(M * K + N * K + M * N)
    else:
        f = 10.0 * case["n"]
        b = 16.0 * case["n"] + 24.0 * case["samples"] + 64 * 32.0 * case["bunches"]
    return {"bytes": b, "flops": f}


def _offsets(labels, layout):
    """Offsets in a tensor stored as `layout` of every value of `labels`
    (both most significant first)."""
    off = torch.zeros(1, dtype=torch.int64, device=DEV)
    for x in labels:
        step = torch.tensor([0, 1 << (len(layout) - 1 - layout.index(x))], dtype=torch.int64, device=DEV)
        off = (off[:, None] + step[None, :]).reshape(-1)
    return off


def _contract(a, la, b, lb):
    """FP64 contraction of two flat tensors over their shared labels; the
    result holds A's free labels, then B's."""
    k = [x for x in la if x in lb]
    m, n = [x for x in la if x not in lb], [x for x in lb if x not in la]
    a2 = a[_offsets(m, la)[:, None] + _offsets(k, la)[None, :]]
    b2 = b[_offsets(k, lb)[:, None] + _offsets(n, lb)[None, :]]
    return (a2 @ b2).reshape(-1), m + n


def _exact_net(net):
    c, open_q, bits, pairs, sliced, (s0, s1) = net
    leaves, ow = _network(c, open_q, bits)
    total = torch.zeros(1 << len(ow), dtype=torch.complex128, device=DEV)
    for s in range(s0, s1):
        fix = {w: (s >> j) & 1 for j, w in enumerate(sliced)}
        ts = []
        for wires, data in leaves:
            t = data.reshape((2,) * len(wires))[tuple(fix.get(w, slice(None)) for w in wires)]
            ts.append((torch.from_numpy(np.ascontiguousarray(t).reshape(-1)).to(DEV),
                       [w for w in wires if w not in fix]))
        for a, b in pairs:
            (x, lx), (y, ly) = ts[a], ts[b]
            ts[a] = ts[b] = None
            ts.append(_contract(x, lx, y, ly))
        root, lr = ts[-1]
        total += root[_offsets(ow, lr)]
    return total


def exact(case, seed):
    kind, dtype = case["kind"], case.get("dtype")
    if kind == "net53":
        return None  # hours in 64 bits
    if kind == "net":
        net = _net(case, seed)
        amp = _exact_net(net)
        return amp if dtype == "c64" else torch.view_as_real(amp * 2.0 ** (net[0].n_qubits / 2))
    if kind == "batch":
        return torch.view_as_real(torch.stack([_exact_net(net) * 2.0 ** (net[0].n_qubits / 2)
                                               for net in _batch(case, seed)]))
    if kind in ("pair", "gemm"):
        A, B = (_pair_inputs if kind == "pair" else _gemm_inputs)(case, seed)
        if dtype != "c64":
            A, B = (torch.view_as_complex(x.double()) for x in (A, B))
        A, B = A.to(torch.complex128), B.to(torch.complex128)
        out = []
        for a, b in zip(A, B):
            if kind == "pair":
                la, lb, lc = _labels(case)
                c, l2 = _contract(a, la, b, lb)
                out.append(c[_offsets(lc, l2)])
            else:
                out.append(a @ b.transpose(0, 1).contiguous())
        C = torch.stack(out)
        return C if dtype == "c64" else torch.view_as_real(C) * _scale(
            case, 1 << case["nK"] if kind == "pair" else case["K"])
    amp, idx, _, _ = _readout_inputs(case, seed)
    p = amp.real ** 2 + amp.imag ** 2
    return {"norm": p.sum().reshape(1), "xeb": torch.stack([p[idx].sum(), (p[idx] ** 2).sum()]), "hist": None,
            "kept": None, "count": None}

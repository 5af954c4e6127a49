"""The amplitude read-out kernels at the edges of their blocks: histogram
(counters in LDS, with fewer copies per bin as the bins grow, and the form for
more bins than LDS holds), norm and frugal sampling, against NumPy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.stats import frugal_accept  # noqa: E402
from paper_2111_01066_amd import tnrcs  # noqa: E402

DEV = "cuda"


def _amps(n, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal(n) + 1j * rng.standard_normal(n)) / np.sqrt(2.0 * n)


@pytest.mark.parametrize("n,bins", [(1, 1), (63, 3), (1025, 64), (4096 * 512 + 77, 200), (100_001, 257),
                                    (50_000, 8192), (50_000, 8193)])
def test_histogram_counts(n, bins):
    print(f"histogram n={n} bins={bins}", flush=True)
    a = _amps(n, n + bins)
    counts = torch.full((bins,), 5, dtype=torch.int64, device=DEV)  # counts are added
    d = torch.from_numpy(a).to(DEV)
    # powers of two: x, x / xmax and the bin are exact functions of |a|^2 up to
    # the rounding of re^2 + im^2, which may be fused
    scale, xmax = float(2 ** int(np.ceil(np.log2(n)))), 8.0
    tnrcs.tn_amp_hist(d, n, scale, xmax, bins, counts)
    torch.cuda.synchronize()
    got = counts.cpu().numpy() - 5
    x = scale * (a.real * a.real + a.imag * a.imag)
    lo = np.bincount(np.minimum((x * (1 - 1e-15) / xmax * bins).astype(np.int64), bins - 1), minlength=bins)
    hi = np.bincount(np.minimum((x * (1 + 1e-15) / xmax * bins).astype(np.int64), bins - 1), minlength=bins)
    assert got.sum() == n
    # an amplitude within rounding of a bin's edge may fall on either side
    assert np.array_equal(got, lo) or np.abs(np.cumsum(got) - np.cumsum(lo)).max() <= np.abs(lo - hi).sum()


@pytest.mark.parametrize("n", [1, 255, 1024 * 256 * 3 + 5, 1024 * 256 * 8])
def test_norm(n):
    a = _amps(n, n)
    out = torch.zeros(1, dtype=torch.float64, device=DEV)
    tnrcs.tn_amp_norm2(torch.from_numpy(a).to(DEV), n, out)
    torch.cuda.synchronize()
    ref = np.sum(np.abs(a) ** 2)
    assert abs(out.item() - ref) < 1e-12 * ref


@pytest.mark.parametrize("n_cand", [1, 255, 1023, 1024, 1025, 8192 * 1024 + 300])
def test_frugal_blocks(n_cand):
    print(f"frugal n_cand={n_cand}", flush=True)
    n = 4099
    a = _amps(n, 7)
    rng = np.random.default_rng(n_cand)
    cand = rng.integers(-3, n + 3, size=n_cand)  # some out of range
    u = rng.random(n_cand)
    kept = torch.full((n_cand,), -1, dtype=torch.int64, device=DEV)
    cnt = torch.full((1,), 99, dtype=torch.int64, device=DEV)
    tnrcs.tn_amp_frugal(torch.from_numpy(a).to(DEV), n, torch.from_numpy(cand).to(DEV), n_cand,
                        torch.from_numpy(u).to(DEV), float(n), 2.0, kept, cnt)
    torch.cuda.synchronize()
    k = int(cnt.item())
    ok = (cand >= 0) & (cand < n)
    want = np.sort(frugal_accept(a, cand[ok], u[ok], float(n), 2.0))
    assert np.array_equal(np.sort(kept[:k].cpu().numpy()), want)
    assert bool((kept[k:] == -1).all())

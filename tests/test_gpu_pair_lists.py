"""Pair build at the edges of its searches: no galaxy, one, none in reach of
another, all in one cell, galaxies on the cells' boundaries (a cell whose
nearest point is exactly the largest separation away), and a catalogue of
rejected positions and weights, whose refusal is read with the pair count.
Pairs and fields are compared exactly with brute force."""
import numpy as np
import pytest

from oracle.pairs import bruteforce_pairs
from synth.configs import Workload, linbins, logbins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
L, SMAX = 96.0, 8.0


def _wl(mode):
    p = dict(p1_edges=linbins(1.0, SMAX, 3), p2_edges=linbins(0.0, 1.0, 2)) if mode == "s_mu" else dict(
        p1_edges=linbins(0.0, 4.8, 3), p2_edges=linbins(0.0, 6.4, 2), pair_dmax=SMAX)
    return Workload(name="edges", L=L, N=64, precision="fp32", pair_mode=mode, out_mode="r_mu",
                    o1_edges=logbins(6.0, 30.0, 2), o2_edges=linbins(0.0, 1.0, 1), catalog_kw={}, **p)


def _positions(kind):
    rng = np.random.default_rng(4)
    if kind == "none":
        return np.zeros((3, 0))
    if kind == "one":
        return np.full((3, 1), 0.25)
    if kind == "apart":
        return np.array([[1.0, 30.0, 60.0], [2.0, 40.0, 70.0], [3.0, 50.0, 80.0]])
    if kind == "one_cell":
        return 40.0 + rng.uniform(0.0, 7.9, (3, 150))
    # on the cells' boundaries (L / 11 apart), a largest separation further, and a
    # step of the last place below each
    x = L / 11 * rng.integers(0, 11, (3, 600))
    x = np.mod(x + np.where(rng.random((3, 600)) < 0.4, SMAX, 0.0), L)
    x = np.where(rng.random((3, 600)) < 0.4, np.maximum(np.nextafter(x, -1.0), 0.0), x)
    return np.where(rng.random((3, 600)) < 0.3, np.mod(x + rng.uniform(0.0, 8.0, (3, 600)), L), x)


@pytest.mark.parametrize("mode", ["s_mu", "rp_pi"])
@pytest.mark.parametrize("kind", ["none", "one", "apart", "one_cell", "boundaries"])
def test_pairs_at_the_edges(kind, mode):
    from paper_1705_03464_amd import Plan, PgxError
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")  # noqa: E731
    wl, x = _wl(mode), _positions(kind)
    assert x.size == 0 or (x.min() >= 0 and x.max() < L)
    plan = Plan.from_workload(wl, precision="fp32")
    n = x.shape[1]
    if n > 1:  # refused first: the plan then builds as if nothing had been
        for bad in (np.nan, np.inf, L, -1.0):
            with pytest.raises(PgxError):
                plan.pairs_build(*(dev(np.full(n, bad)) for _ in range(3)))
        w = np.ones(n)
        w[-1] = -1.0
        with pytest.raises(PgxError):
            plan.pairs_build(*(dev(c) for c in x), w=dev(w, torch.float32))
    P, counts = plan.pairs_build(*(dev(c) for c in x))
    ref = bruteforce_pairs(*x, np.ones(n), L, mode, wl.p1_edges, wl.p2_edges, wl.pair_dmax) if n else None
    ri, rj, rf = (ref["i"], ref["j"], ref["key"]) if n else (np.zeros(0, int),) * 3
    assert P == ri.size
    assert np.array_equal(counts.cpu().numpy(), np.bincount(rf, minlength=wl.n_fields))
    f, i, j = (t.cpu().numpy().astype(np.int64) for t in plan.pairs_export())
    a, b = np.lexsort((j, i, f)), np.lexsort((rj, ri, rf))
    assert np.array_equal(f[a], rf[b]) and np.array_equal(i[a], ri[b]) and np.array_equal(j[a], rj[b])
    out = plan.forward(None)
    assert out["xi_pg"].shape[0] == wl.n_fields

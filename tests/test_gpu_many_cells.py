"""A largest separation so small against the box that the cell list is at its
most cells per side (1290; 1428 would be needed for cells of that width, more
than 32-bit cell indices hold): pairs against brute force."""
import numpy as np
import pytest

from oracle.pairs import bruteforce_pairs
from synth.configs import Workload, linbins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_pairs_with_the_most_cells():
    from paper_1705_03464_amd import Plan
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 32 << 30:
        pytest.skip("needs 32 GiB of free device memory (8.6 GB of cell starts)")
    L, smax = 1000.0, 0.7
    wl = Workload(name="cells", L=L, N=64, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.05, smax, 2),
                  p2_edges=linbins(0.0, 1.0, 2), out_mode="shell", o1_edges=linbins(20.0, 60.0, 2), o2_edges=None,
                  catalog_kw={})
    rng = np.random.default_rng(12)
    c = rng.random((400, 3)) * L
    c[:40] = L - 1e-3 * rng.random((40, 3))  # around the corner of the box, in the last cells
    x = np.mod(np.concatenate([c, np.repeat(c, 6, axis=0) + rng.normal(0.0, 0.3, (2400, 3))]), L).T
    x[x >= L] = 0.0
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    plan = Plan.from_workload(wl, precision="fp32")
    P, counts = plan.pairs_build(*(dev(v) for v in x))
    ref = bruteforce_pairs(*x, np.ones(x.shape[1]), L, "s_mu", wl.p1_edges, wl.p2_edges, wl.pair_dmax)
    assert P == ref["i"].size > 1000
    f, i, j = (t.cpu().numpy().astype(np.int64) for t in plan.pairs_export())
    a, b = np.lexsort((j, i, f)), np.lexsort((ref["j"], ref["i"], ref["key"]))
    assert np.array_equal(f[a], ref["key"][b]) and np.array_equal(i[a], ref["i"][b]) and np.array_equal(j[a], ref["j"][b])
    assert np.isfinite(plan.forward()["xi_gg"].cpu().numpy()).all()
    plan.close()

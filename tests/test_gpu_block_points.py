"""The x-pass scatters take the points of a wavefront's lines, the gathers those
of a block's, as one index range walked by all its threads.  Their edges: more
points on one line than the block keeps in registers, lines and whole blocks
without points, and
a task list that does not fill its last block; at every number of threads per
line below a wavefront (64^3, 128^3, 256^3), CIC and TSC, per-field transforms
and dual form, against the oracle.

Tolerances: the FP32 bar 1e-5 |xi| with the floor of a crowded catalogue (one
FP32 unit of the largest xi_pg), and 1e-3 of the gradient, as for the other
crowded catalogues."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from oracle import grad as OG  # noqa: E402
from synth.catalog import Catalog  # noqa: E402
from synth.configs import Workload, linbins, logbins  # noqa: E402
from test_gpu_grad import grad_close  # noqa: E402
from test_gpu_parity import ALGOS, clustered_catalog  # noqa: E402

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def crowded(L, cell, seed):
    """A clustered catalogue plus 75 galaxies in a tenth of one cell (2775
    pairs on one line, across the box's edge in y and z)."""
    cat = clustered_catalog(L, 60, 600, seed=seed, sat=5, spread=1.5)
    rng = np.random.default_rng(seed)
    spot = np.array([0.3 * L, L - 0.05 * cell, 0.02 * cell]) + 0.1 * cell * rng.random((75, 3))
    pos = np.mod(np.concatenate([cat.positions(), spot]), L)
    n = pos.shape[0]
    return Catalog(L, pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), np.zeros(n), np.zeros(n, np.int8))


@pytest.mark.parametrize("assignment", ["cic", "tsc"])
@pytest.mark.parametrize("N,L", [(64, 110.0), (128, 210.0), (256, 400.0)])
def test_crowded_line_against_oracle(N, L, assignment):
    from paper_1705_03464_amd import Plan
    wl = Workload(name="crowded", L=L, N=N, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.0, 8.0, 3),
                  p2_edges=np.array([0.0, 1.0]), out_mode="shell", o1_edges=logbins(6.0, 30.0, 5), o2_edges=None,
                  catalog_kw={}, assignment=assignment)
    cat = crowded(L, L / N, seed=N)
    rng = np.random.default_rng(N + 1)
    w = rng.uniform(0.5, 1.5, cat.n).astype(np.float32).astype(np.float64)
    g = dict(g_xipg=rng.normal(size=(wl.n_fields, wl.n_out)), g_xigg=rng.normal(size=wl.n_out),
             g_xidp=rng.normal(size=wl.n_fields))
    ref_g, ref = OG.weight_gradient(cat, wl, w, **g)
    for algo, keep in ((0, True), (0, False), (2, False)):
        print(f"{N}^3 {assignment} evaluation {ALGOS[algo]} kept spectra {keep}", flush=True)
        plan = Plan.from_workload(wl, precision="fp32", batch=2)
        plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
        plan.set_schedule(2, 0, 0, *ALGOS[algo])
        plan.keep_spectra(keep)
        for _ in range(2):
            out = {k: v.cpu().numpy() for k, v in plan.forward(dev(w, torch.float32)).items()}
            gw = plan.backward(g_xi_pg=dev(g["g_xipg"]), g_xi_gg=dev(g["g_xigg"]), g_xi_dp=dev(g["g_xidp"]))
        floor = 2.0 ** -23 * np.max(np.abs(ref["xi_pg"]))
        for k in ("xi_gg", "xi_pg"):
            d = np.abs(out[k] - ref[k])
            assert np.all(d <= np.maximum(1e-5 * np.abs(ref[k]), floor)), (k, float(d.max()), floor)
        assert grad_close(gw.cpu().numpy().astype(np.float64), ref_g)
        plan.close()

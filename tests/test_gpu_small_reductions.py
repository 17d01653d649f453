"""Field and bin counts at the edges of the one-wavefront sums (weights, the
finalisation adjoint: one wavefront per field or output bin, 64 lanes; few
fields: many chunks per field) against the oracle's gradient."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from oracle import grad as OG  # noqa: E402
from synth.configs import Workload, linbins, logbins  # noqa: E402
from test_gpu_grad import grad_close, mask_ill_conditioned_q, upstream  # noqa: E402
from test_gpu_parity import clustered_catalog  # noqa: E402

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_s,n_mu,n_r,n_r2", [(1, 1, 1, 1), (5, 13, 2, 1), (2, 1, 13, 5)])
def test_sums_at_wavefront_edges(n_s, n_mu, n_r, n_r2):
    """F x R = 1 x 1, 65 x 2, 2 x 65."""
    from paper_1705_03464_amd import Plan
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")  # noqa: E731
    wl = Workload(name="edges", L=110.0, N=64, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.5, 8.0, n_s),
                  p2_edges=linbins(0.0, 1.0, n_mu), out_mode="r_mu", o1_edges=logbins(6.0, 40.0, n_r),
                  o2_edges=linbins(0.0, 1.0, n_r2), catalog_kw={})
    cat = clustered_catalog(wl.L, 100, 1500, seed=n_s + n_r, sat=6, spread=1.5)
    w = np.random.default_rng(9).uniform(0.5, 1.5, cat.n).astype(np.float32).astype(np.float64)
    g = upstream(wl.n_fields, wl.n_out, 7)
    from oracle.pipeline import forward as ofw
    g = mask_ill_conditioned_q(g, wl, ofw(cat, wl, w=w))
    ref, out = OG.weight_gradient(cat, wl, w, **g)
    plan = Plan.from_workload(wl, precision="fp32", batch=3)
    plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
    got = plan.forward(dev(w, torch.float32))
    assert np.allclose(got["wsum"].cpu().numpy(), out["wsum"], rtol=1e-12)
    gw = plan.backward(g_b_pg=dev(g["g_b"]), g_q_eff=dev(g["g_q"]), g_xi_pg=dev(g["g_xipg"]),
                       g_xi_gg=dev(g["g_xigg"]), g_xi_dp=dev(g["g_xidp"]))
    assert grad_close(gw.cpu().numpy().astype(np.float64), ref)

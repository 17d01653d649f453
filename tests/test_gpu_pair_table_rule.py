"""The pair gradient just above the rule that sums it per galaxy in LDS first
(24 pairs per galaxy, 2^20 pairs) against the oracle; 1e-3 of the gradient, as for
the other crowded catalogues."""
import numpy as np
import pytest

from synth.configs import linbins, logbins

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_pair_gradient_at_the_table_rule():
    """About 30 pairs per galaxy, more than 2^20 pairs: against the oracle."""
    from oracle import grad as OG
    from paper_1705_03464_amd import Plan
    from synth.catalog import Catalog
    from synth.configs import Workload
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L, n = 90.0, 38000
    rng = np.random.default_rng(2)
    c = rng.random((n // 64, 3)) * L
    pos = np.mod(np.repeat(c, 64, axis=0) + rng.normal(0.0, 1.0, (n // 64 * 64, 3)), L)
    pos[pos >= L] = 0.0
    cat = Catalog(L, *(pos[:, k].copy() for k in range(3)), np.zeros(len(pos)), np.zeros(len(pos), np.int8))
    wl = Workload(name="table", L=L, N=64, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.0, 3.4, 2),
                  p2_edges=np.array([0.0, 1.0]), out_mode="shell", o1_edges=logbins(6.0, 25.0, 3), o2_edges=None,
                  catalog_kw={})
    w = rng.uniform(0.5, 1.5, cat.n).astype(np.float32).astype(np.float64)
    g = dict(g_xipg=rng.normal(size=(2, 3)), g_xigg=rng.normal(size=3), g_xidp=1e-3 * rng.normal(size=2))
    ref, _ = OG.weight_gradient(cat, wl, w, **g)
    dev = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")  # noqa: E731
    plan = Plan.from_workload(wl, precision="fp32")
    P, _ = plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
    print(f"{P} pairs, {P / cat.n:.1f} per galaxy", flush=True)
    assert P >= 1 << 20 and 24 <= P // cat.n < 64
    plan.forward(dev(w, torch.float32))
    gw = plan.backward(g_xi_pg=dev(g["g_xipg"]), g_xi_gg=dev(g["g_xigg"]), g_xi_dp=dev(g["g_xidp"])).cpu().numpy()
    assert np.linalg.norm(gw - ref) <= 1e-3 * np.linalg.norm(ref) and np.max(np.abs(gw - ref)) <= 1e-3 * np.max(np.abs(ref))
    plan.close()

"""Branches that only crowded catalogues or wide batches reach, against the
oracle (or, at 1024^3, against narrower batches of the same plan):

* the pair gradient with sums per galaxy in LDS first (from 2^20 pairs and 64
  pairs per galaxy on): two clumps whose 1030 galaxies each exceed the table's
  1024 slots, so that a block's additions also take the way past it, and a pair
  count that leaves the last block part empty;
* the Pi scatter of the multipoles' adjoint where a block's wavefronts take the
  points of a crowded line together;
* the cross-power pass of 1024^3 grids with more slots than it stages plane
  masks for at a time (16).

Tolerances: 1e-3 of the gradient, as for the other crowded catalogues; at
1024^3 the FP32 bar 1e-5 max(|xi|, 1e-2) (the arithmetic of a field does not
depend on its slot)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from oracle import grad as OG  # noqa: E402
from oracle import multipoles as OM  # noqa: E402
from oracle.pipeline import forward as oracle_forward  # noqa: E402
from synth.catalog import Catalog  # noqa: E402
from synth.configs import Workload, linbins, logbins  # noqa: E402
from test_gpu_block_points import crowded  # noqa: E402
from test_gpu_grad import grad_close  # noqa: E402
from test_gpu_parity import ALGOS, xi_err_ok  # noqa: E402

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def _catalog(L, pos):
    pos = np.mod(pos, L)
    n = pos.shape[0]
    return Catalog(L, pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), np.zeros(n), np.zeros(n, np.int8))


@pytest.mark.parametrize("assignment,algo", [("cic", 0), ("cic", 2), ("tsc", 0)])
def test_pair_gradient_with_sums_per_galaxy(assignment, algo):
    from paper_1705_03464_amd import Plan
    L, N = 110.0, 64
    wl = Workload(name="clumps", L=L, N=N, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.0, 8.0, 2),
                  p2_edges=np.array([0.0, 1.0]), out_mode="shell", o1_edges=logbins(6.0, 30.0, 4), o2_edges=None,
                  catalog_kw={}, assignment=assignment)
    rng = np.random.default_rng(3)
    clump = lambda c: np.array(c) + rng.uniform(-1.2, 1.2, (1030, 3))  # noqa: E731
    cat = _catalog(L, np.concatenate([clump([30.0, 109.5, 40.2]), clump([81.3, 60.0, 75.0]), rng.random((400, 3)) * L]))
    w = rng.uniform(0.5, 1.5, cat.n).astype(np.float32).astype(np.float64)
    g = dict(g_xipg=rng.normal(size=(wl.n_fields, wl.n_out)), g_xigg=rng.normal(size=wl.n_out),
             g_xidp=1e-3 * rng.normal(size=wl.n_fields))
    ref_g, _ = OG.weight_gradient(cat, wl, w, **g)
    plan = Plan.from_workload(wl, precision="fp32", batch=1)
    P, _ = plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
    print(f"{assignment} evaluation {ALGOS[algo]}: {P} pairs of {cat.n} galaxies", flush=True)
    assert P >= 1 << 20 and P // 64 >= cat.n and P % 2048 != 0
    plan.set_schedule(1, 0, 0, *ALGOS[algo])
    for _ in range(3):  # eager, recorded, replayed
        plan.forward(dev(w, torch.float32))
        gw = plan.backward(g_xi_pg=dev(g["g_xipg"]), g_xi_gg=dev(g["g_xigg"]), g_xi_dp=dev(g["g_xidp"]))
        assert grad_close(gw.cpu().numpy().astype(np.float64), ref_g)
    plan.close()


@pytest.mark.parametrize("N,L", [(64, 110.0), (128, 210.0)])
def test_multipole_adjoint_of_a_crowded_line(N, L):
    from paper_1705_03464_amd import Plan
    wl = Workload(name="crowded", L=L, N=N, precision="fp32", pair_mode="s_mu", p1_edges=np.array([1e-3, 2.0, 8.0]),
                  p2_edges=linbins(0.0, 1.0, 2), out_mode="shell", o1_edges=logbins(6.0, 30.0, 3), o2_edges=None,
                  catalog_kw={})
    cat = crowded(L, L / N, seed=N)
    rng = np.random.default_rng(N + 2)
    w = rng.uniform(0.5, 1.5, cat.n).astype(np.float32).astype(np.float64)
    ref = oracle_forward(cat, wl, w=w)
    plan = Plan.from_workload(wl, precision="fp32", batch=4)
    P, _ = plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
    plan.forward(dev(w, torch.float32))
    xi = plan.multipoles(2).cpu().numpy()
    g = rng.normal(size=xi.shape)
    g[~np.isfinite(xi)] = 0.0
    gw = plan.multipoles_backward(dev(g)).cpu().numpy().astype(np.float64)
    # galaxies of the crowded line (the last 75) and others
    idx = np.concatenate([cat.n - 1 - np.arange(0, 75, 13), np.argsort(-np.abs(gw))[:3], rng.choice(cat.n, 4, replace=False)])
    fd = OM.fd_weight_gradient(cat, wl, w, idx, g, ref["pairs"], ells=(0, 2), h=1e-3)
    err = np.abs(gw[idx] - fd)
    print(f"{N}^3: {P} pairs, fd max abs err {err.max():.3e}, largest entry {np.abs(gw).max():.3e}", flush=True)
    assert np.all(err <= 1e-3 * np.abs(gw).max())
    plan.close()


def test_more_slots_than_staged_plane_masks_1024():
    from paper_1705_03464_amd import Plan
    if torch.cuda.mem_get_info()[0] < 220 << 30:
        pytest.skip("needs 220 GiB of free device memory")
    L, N = 2000.0, 1024
    wl = Workload(name="slots", L=L, N=N, precision="fp32", pair_mode="s_mu", p1_edges=linbins(0.0, 20.0, 37),
                  p2_edges=np.array([0.0, 1.0]), out_mode="shell", o1_edges=linbins(8.0, 24.0, 2), o2_edges=None,
                  catalog_kw={})
    rng = np.random.default_rng(8)
    c = rng.random((150, 3)) * L
    cat = _catalog(L, np.concatenate([c, np.repeat(c, 5, axis=0) + rng.normal(0.0, 5.0, (750, 3))]))
    plan = Plan.from_workload(wl, precision="fp32", batch=8)
    P, counts = plan.pairs_build(dev(cat.x), dev(cat.y), dev(cat.z))
    out = {}
    for batch in (19, 8):  # one batch of 19 field pairs, then three
        print(f"1024^3, {P} pairs in {wl.n_fields} fields, {batch} slots", flush=True)
        plan.set_schedule(batch)
        out[batch] = {k: v.cpu().numpy() for k, v in plan.forward().items()}
    plan.close()
    full = counts.cpu().numpy() > 0
    assert np.isfinite(out[8]["xi_pg"][full]).all() and np.all(full[32:].sum() >= 3)
    for k in ("xi_gg", "xi_pg"):
        assert xi_err_ok(out[19][k], out[8][k]) <= 1.0, k

"""A wrong catalogue is refused as such (PGX_EINVAL) whatever the workspace: in
regions from below the plan's tables up to the whole build, a bad position or
weight is never reported as a lack of room once the tables fit, and the flags
of a refused or failed build do not reach the next one."""
import numpy as np
import pytest

from synth import get_config

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def _code(plan, x, y, z, w=None):
    """Status of one build (0: built)."""
    from paper_1705_03464_amd import PgxError
    try:
        plan.pairs_build(x, y, z, w=w)
    except PgxError as e:
        return e.code
    return 0


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_wrong_catalogues_are_refused_before_room_is_short(precision):
    from paper_1705_03464_amd import Plan
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = get_config("cfg4tiny")
    cat = wl.catalog()
    x, y, z = _dev(cat.x), _dev(cat.y), _dev(cat.z)
    far, nan, neg = x.clone(), x.clone(), torch.ones(cat.n, dtype=torch.float32, device="cuda")
    far[cat.n // 2], nan[-1], neg[0] = wl.L, float("nan"), -1.0
    seen = {0: 0, 2: 0}
    size = 32 << 10
    while size < 64 << 20:
        plan = Plan.from_workload(wl, precision=precision)
        plan.set_workspace(size)
        codes = [_code(plan, far, y, z), _code(plan, nan, y, z), _code(plan, x, y, z, w=neg)]
        good = _code(plan, x, y, z)
        tables = plan.workspace_used()[0] > 0
        print(f"{precision} workspace {size >> 10} KiB: tables {'fit' if tables else 'do not fit'}, "
              f"refusals {codes}, good catalogue {good}", flush=True)
        assert good in (0, 2)
        assert codes == ([1, 1, 1] if tables else [2, 2, 2])
        seen[good] += tables
        plan.close()
        size = size * 5 // 4
    assert seen[0] >= 2 and seen[2] >= 4  # both sides of the build's needs were tried


@pytest.mark.parametrize("workspace", [False, True])
def test_page_locked_host_memory_can_be_missing(workspace, monkeypatch):
    """The plan's block of page-locked host memory is the first allocation of its
    first device work; when it fails (injected) the call returns PGX_EHIP and the
    plan works afterwards, with its own device memory and with a workspace, where
    it is the only allocation."""
    from paper_1705_03464_amd import PgxError, Plan
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = get_config("cfg4tiny")
    cat = wl.catalog()
    x, y, z = _dev(cat.x), _dev(cat.y), _dev(cat.z)
    plan = Plan.from_workload(wl, precision="fp32")
    if workspace:
        plan.set_workspace(512 << 20)
    monkeypatch.setenv("PGX_DEBUG_FAIL_ALLOC", "1")
    with pytest.raises(PgxError) as e:
        plan.pairs_build(x, y, z)
    assert e.value.code == 3 and "hipHostMalloc" in str(e.value) and "injected" in str(e.value)
    monkeypatch.delenv("PGX_DEBUG_FAIL_ALLOC")
    P, _ = plan.pairs_build(x, y, z)
    assert P > 0
    plan.close()


def test_refusal_does_not_wait_for_the_search():
    """1.5e5 galaxies in one cell (too many pairs, found by a search of 1.1e10
    candidates): with one bad weight the catalogue is refused as wrong, and in less
    than a quarter of the time of the search."""
    import time

    from paper_1705_03464_amd import Plan
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = get_config("cfg4tiny")
    n = 150000
    x = [_dev(40.0 + np.random.default_rng(k).random(n)) for k in range(3)]
    w = torch.ones(n, dtype=torch.float32, device="cuda")
    plan = Plan.from_workload(wl, precision="fp32")
    took = {}
    for _ in range(3):  # the first of each also allocates
        for bad in (False, True):
            w[n // 3] = -1.0 if bad else 1.0
            torch.cuda.synchronize()
            t = time.perf_counter()
            assert _code(plan, *x, w=w) == (1 if bad else 4)
            took[bad] = time.perf_counter() - t
    print(f"search {took[False] * 1e3:.2f} ms, refusal {took[True] * 1e3:.2f} ms", flush=True)
    assert took[True] < 0.25 * took[False]
    plan.close()

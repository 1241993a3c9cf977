"""The stages of a prescribed flow, which start from the bases of the stage before, against
stencils solved cold for the same cloud in a context of their own: the same update.  Where
the check of the bases settles almost all LPs, none (an exact lattice: fewer fractions than
moments) and a part; what it leaves in a queue for eight lanes per LP (up to 32768) and in a
longer one, for one thread per LP."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def vrm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_06379_amd as v
    v.lib()
    return v


def _rate(vrm, src, n, mask, P):
    """sum_j fhat_ji Gamma_j of the cloud's cold stencils, in FP64."""
    x, y, g, ids = [t[:n].cpu().numpy() for t in (src.x, src.y, src.gamma, src.id)]
    cloud = vrm.Cloud(x, y, g, ids=ids, capacity=n)
    ctx = vrm.Context(n)
    ctx.vrm_set_diffused(cloud, mask)
    st = vrm.Stencils.alloc(n)
    ctx.vrm_solve_fractions(cloud, P, st)
    torch.cuda.synchronize()
    S = {k: getattr(st, k).cpu().numpy() for k in
         ("small_idx", "small_f", "fii", "status", "full_k", "full_idx", "full_f")}
    g = g.astype(np.float64)
    rate = S["fii"].astype(np.float64) * g
    small = S["status"] == vrm.ST_SMALL
    idx = np.where(S["small_idx"] >= 0, S["small_idx"], 0)
    np.add.at(rate, idx[small], np.where(S["small_idx"] >= 0, S["small_f"], 0.0)[small] * g[small][:, None])
    full = S["status"] == vrm.ST_FULL
    used = (np.arange(vrm.KMAX) < S["full_k"][:, None]) & full[:, None]
    who, col = np.nonzero(used)
    np.add.at(rate, S["full_idx"][who, col], S["full_f"][who, col].astype(np.float64) * g[who])
    return rate, g


@pytest.mark.parametrize("q,side,jitter,scale,warm", [
    (2, 181, 0.0, 1.0, 0),      # all left: 32761
    (2, 200, 0.0, 1.0, 0),      # all left: 40000
    (2, 200, 0.25, 1.0, 0),     # few left
    (2, 200, 0.25, 40.0, 0),    # a part
    (2, 200, 0.0, 1.0, 2),
    (3, 100, 0.4, 40.0, 0),
    (3, 100, 0.4, 40.0, 2)])
def test_stages_against_cold_stencils(vrm, q, side, jitter, scale, warm):
    h = 0.015625   # the lattice is exact
    half = 0.5 * h * (side - 1)
    wl = workloads._vortex_cloud("flow", -half, half, h, 3, 3, 31, 32, 0.0, q)
    x, y = workloads.lattice(-half, half, h)
    rng = np.random.default_rng(7)
    wl.x = (x + rng.uniform(-jitter, jitter, x.size) * h).astype(np.float32)
    wl.y = (y + rng.uniform(-jitter, jitter, x.size) * h).astype(np.float32)
    wl.vortices["gamma"] = wl.vortices["gamma"] * scale
    P = vrm.params_of(wl)
    vt = vrm.vortex_table(wl.vortices)
    n = wl.n
    cloud = vrm.Cloud(wl.x, wl.y, wl.gamma, capacity=n)
    ctx = vrm.Context(n)
    ctx.vrm_set_warm_start(warm)
    mask = torch.ones(n, dtype=torch.uint8, device="cuda")
    ctx.vrm_set_diffused(cloud, mask)
    u = torch.zeros(n, device="cuda")
    v = torch.zeros(n, device="cuda")
    g0 = wl.gamma.astype(np.float64)
    lam = wl.nu / wl.h ** 2
    print("case cold stages", q, side, jitter, scale, warm, n, flush=True)
    for s, (a, b, c) in enumerate(((0.0, 1.0, 0.0), (0.75, 0.25, 1.0), (1.0 / 3.0, 2.0 / 3.0, 0.5))):
        ctx.vrm_vortex_velocity(cloud, vt, wl.nu, wl.t0 + c * wl.dt, u, v)
        rate, g = _rate(vrm, cloud, n, mask, P)
        ctx.vrm_rk_stage(cloud, P, s, u, v)
        torch.cuda.synchronize()
        got = cloud.gamma[:n].double().cpu().numpy()
        want = a * g0 + b * (g + wl.dt * lam * rate)
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print("  stage", s, "rel L2", err, "pivots", ctx.vrm_read_counters()["pivots"], flush=True)
        assert err <= 1e-6   # FP32 fractions and sums

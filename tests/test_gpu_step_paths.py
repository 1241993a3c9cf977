"""The stages of vrm_step that take another route than three vrm_rk_stage calls: the
same step, to the order of the atomic sums (relative L2 1e-6 as for the launch
shapes; the fixed-point sums differ only where a fraction rounds to the other of
two neighbouring FP32 values)."""
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


def _by_id(cloud):
    x, y, g, ids = cloud.numpy()
    o = np.argsort(ids)
    return ids[o], x[o].astype(np.float64), y[o].astype(np.float64), g[o].astype(np.float64)


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


@pytest.mark.parametrize("q,objective,warm,tuning", [
    (2, 0, 0, None), (2, 0, 0, {"lp_small_coop": 1}), (2, 0, 2, None), (2, 1, 0, None), (2, 2, 0, None),
    (3, 0, 0, None), (3, 0, 2, None), (3, 1, 0, None), (3, 2, 0, None)])
@pytest.mark.parametrize("det", [0, 1])
def test_fixed_positions_apply_the_kept_stencils(vrm, q, objective, warm, tuning, det):
    """Without a velocity vrm_step solves the LPs once and applies the stencils in
    three stages; vrm_rk_stage solves them in every stage.  Two steps, the second
    from another state (kept stencils are replaced), on a cloud with particles that
    have no stencil (a lone one far away) and ragged counts."""
    wl = workloads.config_jittered(h=0.05, q=q, seed=11, jitter=0.4)
    x = np.append(wl.x, np.float32(3.0))
    y = np.append(wl.y, np.float32(3.0))
    g = np.append(wl.gamma, wl.gamma.max())
    P = vrm.params_of(wl, deterministic=det)
    print("case fixed", q, objective, warm, tuning, det, flush=True)
    res = []
    for whole in (True, False):
        cloud = vrm.Cloud(x, y, g, capacity=4 * x.size)
        ctx = vrm.Context(cloud.capacity)
        ctx.vrm_set_lp_objective(objective)
        ctx.vrm_set_warm_start(warm)
        ctx.vrm_set_tuning(tuning)
        for _ in range(2):
            if whole:
                ctx.vrm_step(cloud, P, None, wl.t0)
            else:
                ctx.step(cloud, P)
        torch.cuda.synchronize()
        res.append((_by_id(cloud), ctx.vrm_read_counters()))
    (a, ca), (b, cb) = res
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])
    np.testing.assert_array_equal(a[2], b[2])
    assert _rel(a[3], b[3]) <= 1e-6
    # the same stencils applied, in a third of the LP solves
    assert ca["redistributions"] == cb["redistributions"] > 0
    assert 3 * (ca["n_small"] + ca["n_full"]) == cb["n_small"] + cb["n_full"]


def _stencils(vrm, x, y, g, P, mask, n):
    cloud = vrm.Cloud(x, y, g, capacity=x.size + 64)
    ctx = vrm.Context(cloud.capacity)
    m = torch.zeros(cloud.capacity, dtype=torch.uint8, device="cuda")
    m[:n] = torch.as_tensor(mask, device="cuda")
    ctx.vrm_set_diffused(cloud, m)
    st = vrm.Stencils.alloc(cloud.capacity)
    ctx.vrm_solve_fractions(cloud, P, st)
    torch.cuda.synchronize()
    out = [t[:n].cpu().numpy() for t in (st.small_idx, st.small_f, st.fii, st.status, st.full_k, st.full_idx, st.full_f)]
    c = ctx.vrm_read_counters()
    return out, {k: c[k] for k in ("n_small", "n_full", "n_infeasible", "n_uncertified", "n_truncated", "pivots",
                                   "full_cols")}


@pytest.mark.parametrize("jitter,r_full,keep", [
    (0.0, 3.0, 1.0),     # a lattice: degenerate LPs, exact certifications
    (0.45, 3.0, 1.0),    # up to 48 columns
    (0.45, 3.0, 0.35),   # holes: few columns, infeasible LPs, none at all
    (0.3, 3.9, 1.0),     # 48 to 64 members: the 48 nearest
    (0.3, 4.5, 1.0)])    # more than 64: the 48th nearest by bisection
def test_sixteen_lane_complete_lps_match_one_thread_ones(vrm, jitter, r_full, keep):
    """Small clouds solve the nine-row LPs with sixteen lanes each, large ones with one
    thread: the same particles in a cloud padded past the limit with far, undiffused
    ones get bit-identical stencils, in the same order, with the same pivots."""
    print("case sixteen", jitter, r_full, keep, flush=True)
    wl = workloads.config_jittered(h=0.04, q=3, seed=3, jitter=jitter)
    sel = np.random.default_rng(7).random(wl.n) < keep
    x, y, g = wl.x[sel], wl.y[sel], wl.gamma[sel]
    n = x.size
    P = vrm.make_params(wl.h, nu=wl.nu, q=3, dt=wl.dt, R_full=r_full)
    mask = (np.arange(n) % 7 != 3).astype(np.uint8)
    small = _stencils(vrm, x, y, g, P, mask, n)
    side = 400
    px, py = np.meshgrid(5.0 + 0.3 * np.arange(side), 5.0 + 0.3 * np.arange(side))
    pad = np.zeros(side * side, np.float32)
    large = _stencils(vrm, np.append(x, px.ravel().astype(np.float32)), np.append(y, py.ravel().astype(np.float32)),
                      np.append(g, pad), P, mask, n)
    assert n < (1 << 17) < n + pad.size
    for a, b in zip(small[0], large[0]):
        np.testing.assert_array_equal(a, b)
    assert small[1] == large[1]
    assert small[1]["n_full"] > 0

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


def _flow_run(vrm, wl, P, vt, warm, hints, steps, u, v):
    """`steps` steps by single stages; hints: the stages of a step one after the other;
    else a selection between them, after which a stage starts from no basis."""
    cloud = vrm.Cloud(wl.x, wl.y, wl.gamma, capacity=4 * wl.n)
    ctx = vrm.Context(cloud.capacity)
    ctx.vrm_set_warm_start(warm)
    t = wl.t0
    for _ in range(steps):
        ctx.vrm_insert_particles(cloud, P)
        for s, c in enumerate((0.0, 1.0, 0.5)):
            ctx.vrm_vortex_velocity(cloud, vt, wl.nu, t + c * wl.dt, u, v)
            ctx.vrm_rk_stage(cloud, P, s, u, v)
        t += wl.dt
    torch.cuda.synchronize()
    return _by_id(cloud), ctx.vrm_read_counters()


@pytest.mark.parametrize("scale", [1.0, 40.0])
@pytest.mark.parametrize("warm", [0, 2])
@pytest.mark.parametrize("q", [2, 3])
def test_stages_from_the_bases_of_the_stage_before(vrm, orc, q, warm, scale):
    """A prescribed flow: stages 1 and 2 check the bases of the stage before
    (warm start 2: also the step's first stage, the previous step's) and solve only what
    the check does not settle.  The same Gamma as the FP64 oracle's step, also with a
    velocity forty times larger, where many bases change within a step."""
    wl = workloads._vortex_cloud("flow", -0.5, 0.5, 0.02, 3, 3, 31, 32, 0.1, q)
    wl.vortices["gamma"] = wl.vortices["gamma"] * scale
    P = vrm.params_of(wl)
    vt = vrm.vortex_table(wl.vortices)
    u = torch.zeros(4 * wl.n, device="cuda")
    v = torch.zeros(4 * wl.n, device="cuda")
    (ids, x, y, g), c = _flow_run(vrm, wl, P, vt, warm, True, 2, u, v)
    ref = orc.run(wl, steps=2)
    print("case bases", q, warm, scale, "N", ids.size, ref.x.size, c, flush=True)
    np.testing.assert_array_equal(ids, ref.ids)
    # Gamma within the stated 1e-5 of the oracle
    assert _rel(g, ref.gamma) <= 1e-5
    assert c["redistributions"] == c["n_small"] + c["n_full"] > 0
    if scale == 1.0:
        # one LP in three (first step of warm start 2: the same) takes pivots, eight or twelve each
        assert c["pivots"] < 0.5 * (8 * c["n_small"] + 12 * c["n_full"])
    if warm == 2:
        assert c["warm_hit"] > 0


def test_changed_bases_are_solved_again(vrm):
    """Kept bases are hints: a stage whose particles were moved far from those of stage 0
    (other neighbourhoods altogether) gives the stencils of its own positions."""
    wl = workloads.config_jittered(h=0.05, q=3, seed=4)
    P = vrm.params_of(wl)
    rng = np.random.default_rng(5)
    n = wl.n
    perm = rng.permutation(n)
    out = []
    for hints in (True, False):
        cloud = vrm.Cloud(wl.x, wl.y, wl.gamma, capacity=n + 64)
        ctx = vrm.Context(cloud.capacity)
        ctx.vrm_set_diffused(cloud, torch.ones(cloud.capacity, dtype=torch.uint8, device="cuda"))
        zero = torch.zeros(cloud.capacity, device="cuda")
        ctx.vrm_rk_stage(cloud, P, 0, zero, zero)
        g1 = cloud.gamma.clone()
        # other positions for every particle, from outside (the velocity of stage 0 leaves
        # the cell list to be rebuilt)
        cloud.x[:n] = torch.as_tensor(wl.x[perm], device="cuda")
        cloud.y[:n] = torch.as_tensor(wl.y[perm], device="cuda")
        ctx.vrm_rk_stage(cloud, P, 1, zero, zero) if hints else None
        if hints:
            # stage 1: g = 3/4 g0 + 1/4 (g1 + dt rate); the rate from the stencils
            torch.cuda.synchronize()
            got = cloud.gamma[:n].double().cpu().numpy()
        else:
            st = vrm.Stencils.alloc(cloud.capacity)
            ctx.vrm_solve_fractions(cloud, P, st)
            torch.cuda.synchronize()
            rate = np.zeros(n)
            gg = g1[:n].double().cpu().numpy()
            k, idx, f = (t.cpu().numpy() for t in (st.full_k, st.full_idx, st.full_f))
            for i in range(n):
                np.add.at(rate, idx[i, :k[i]], f[i, :k[i]].astype(np.float64) * gg[i])
            rate += st.fii[:n].double().cpu().numpy() * gg
            lam = wl.nu / wl.h ** 2
            out.append(0.75 * wl.gamma.astype(np.float64) + 0.25 * (gg + wl.dt * lam * rate))
    print("case changed bases", flush=True)
    assert _rel(got, out[0]) <= 1e-6

"""Clouds whose ids are not distinct, on lattices (many members at one distance): every
member keeps a column of its own, the stencils meet the moment conditions, and there are
as many as with distinct ids (but for the few nine-row LPs beside holes whose phase I the
order of the columns decides: with distinct ids, too, one or two of 2724 come out
infeasible or not by their order)."""
import numpy as np
import pytest

import moments

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def vrm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_06379_amd as v
    v.lib()
    return v


def _lattice(side, keep, seed):
    gx, gy = np.meshgrid(np.arange(side), np.arange(side))
    sel = np.random.default_rng(seed).random(side * side) < keep
    return gx.ravel()[sel] * 0.125, gy.ravel()[sel] * 0.125


def _stencils(vrm, x, y, ids, P):
    n = x.size
    cloud = vrm.Cloud(x, y, np.ones(n), ids=ids, capacity=n + 64)
    ctx = vrm.Context(cloud.capacity)
    ctx.vrm_set_diffused(cloud, torch.ones(cloud.capacity, dtype=torch.uint8, device="cuda"))
    st = vrm.Stencils.alloc(cloud.capacity)
    ctx.vrm_solve_fractions(cloud, P, st)
    torch.cuda.synchronize()
    return {k: getattr(st, k)[:n].cpu().numpy() for k in
            ("small_idx", "small_f", "fii", "status", "full_k", "full_idx", "full_f")}


# (2, .): what the small neighbourhoods leave; (3, 60): sixteen lanes per LP; (3, 400):
# column lists, one thread per LP
@pytest.mark.parametrize("q,side,keep", [(2, 60, 0.6), (3, 60, 1.0), (3, 60, 0.75), (3, 400, 0.9)])
def test_stencils_with_equal_ids(vrm, q, side, keep):
    x, y = _lattice(side, keep, 5)
    n = x.size
    P = vrm.make_params(0.125, nu=1e-3, q=q, dt=1e-3, R_full=3.0)
    print("case equal ids", q, side, keep, n, flush=True)
    S = _stencils(vrm, x, y, np.zeros(n, np.int32), P)
    ref = _stencils(vrm, x, y, None, P)
    differ = int((S["status"] != ref["status"]).sum())
    assert differ == 0 if q == 2 or keep == 1.0 else differ <= 0.005 * n
    assert (S["status"] == vrm.ST_FULL).any()
    full = S["status"] == vrm.ST_FULL
    k = S["full_k"]
    used = (np.arange(vrm.KMAX) < k[:, None]) & full[:, None]
    assert (S["full_idx"][used] >= 0).all() and (S["full_idx"][used] < n).all() and (S["full_f"][used] > 0).all()
    for i in np.nonzero(full)[0][:2000]:
        assert np.unique(S["full_idx"][i, :k[i]]).size == k[i]
    rows, cols, f = moments.stencil_columns(S)
    res = moments.residuals(x, y, 0.125, q, rows, cols, f)
    print("  with a stencil", rows.size, "complete", int(full.sum()), "residual", res.max(), flush=True)
    assert res.max() <= 1e-6


def test_removal_with_equal_ids(vrm):
    """The candidates' ids are distinct (they decide who goes), all others equal."""
    x, y = _lattice(60, 1.0, 5)
    rng = np.random.default_rng(6)
    pick = (rng.random(x.size) < 0.03) & (np.abs(x - x.mean()) < 3.5) & (np.abs(y - y.mean()) < 3.5)   # not on the hull
    n0 = x.size
    x = np.append(x, x[pick] + 0.03).astype(np.float32)
    y = np.append(y, y[pick] + 0.015).astype(np.float32)
    n = x.size
    g = rng.normal(0, 1, n).astype(np.float32)
    near = np.append(pick, np.ones(n - n0, bool))
    P = vrm.make_params(0.125, nu=1e-3, q=2, dt=1e-3)
    print("case removal with equal ids", n, int(near.sum()), flush=True)
    out = []
    for ids in (np.arange(n, dtype=np.int32), np.where(near, np.arange(n), n).astype(np.int32)):
        cloud = vrm.Cloud(x, y, g, ids=ids, capacity=n)
        ctx = vrm.Context(n)
        nr, nc = ctx.vrm_remove_particles(cloud, P)
        torch.cuda.synchronize()
        xs, ys, gs, _ = cloud.numpy()
        out.append((nr, nc, xs, ys))
        # I0 and I1: FP32 weights and sums
        G, s = g.astype(np.float64), np.abs(g.astype(np.float64)).sum()
        assert abs(gs.astype(np.float64).sum() - G.sum()) <= 1e-6 * s
        assert abs((gs.astype(np.float64) * xs).sum() - (G * x).sum()) <= 1e-6 * s * x.max()
        assert abs((gs.astype(np.float64) * ys).sum() - (G * y).sum()) <= 1e-6 * s * y.max()
    assert out[0][0] == out[1][0] > 0 and out[0][1] == out[1][1]
    np.testing.assert_array_equal(out[0][2], out[1][2])
    np.testing.assert_array_equal(out[0][3], out[1][3])

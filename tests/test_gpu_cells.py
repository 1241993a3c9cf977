"""Cell lists: counts by runs of lanes, the scan over chunks in one launch, and the grid
found by the last workgroup, at the sizes where chunks and waves end, through the
neighbourhoods (whose members the brute-force search of the oracle's distances names)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def vrm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_06379_amd as v
    v.lib()
    return v


def _counts_by_sort(x, y, h, lo, hi):
    """Particles within lo h .. hi h of each one, from all pairs (FP64, small clouds)."""
    d = np.hypot(x[:, None] - x[None, :], y[:, None] - y[None, :])
    m = (d >= lo * h) & (d <= hi * h)
    return m.sum(1)


# kind: cells in slot order or not, all in one cell, far apart (the grid is clamped)
@pytest.mark.parametrize("kind", ["sorted", "shuffled", "one_cell", "far", "line"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 255, 257, 2049])
def test_neighbourhood_sizes(vrm, n, kind):
    rng = np.random.default_rng(n + len(kind))
    h = 0.05
    if kind == "one_cell":
        x, y = rng.uniform(0, 0.1, n), rng.uniform(0, 0.1, n)
        h = 0.05 * min(1.0, 6.0 / np.sqrt(n))   # at most about 40 members each
    elif kind == "line":
        x, y = np.linspace(0, 0.6 * h * n, n), np.zeros(n)
    else:
        side = 0.06 * np.sqrt(n)
        x, y = rng.uniform(0, side, n), rng.uniform(0, side, n)
        if kind == "far":
            x[: n // 2] += 1.0e4
        if kind == "sorted":
            o = np.lexsort((np.floor(x / (2 * h)), np.floor(y / (2 * h))))
            x, y = x[o], y[o]
    x, y = x.astype(np.float32), y.astype(np.float32)
    cloud = vrm.Cloud(x, y, np.ones(n, np.float32), capacity=n + 8)
    ctx = vrm.Context(cloud.capacity)
    P = vrm.make_params(h=h, q=2, r=0.5, R=2.0)
    kfull = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda")
    small = torch.full((n + 8, 8), -7, dtype=torch.int32, device="cuda")
    want = _counts_by_sort(x.astype(np.float64), y.astype(np.float64), h, 0.5, 2.0)
    edge = np.abs(np.hypot(x[:, None].astype(float) - x[None], y[:, None].astype(float) - y[None]) / h)
    # pairs on a limit to the FP32 rounding of the squared distance are not decided here
    clear = (np.abs(edge - 2.0).min(1) > 1e-5) & (np.abs(edge - 0.5).min(1) > 1e-5)
    print("case cells", n, kind, "undecided", int((~clear).sum()), flush=True)
    for _ in range(2):   # the second build finds the counts cleared
        ctx.vrm_set_diffused(cloud, torch.ones(n + 8, dtype=torch.uint8, device="cuda"))
        ctx.vrm_build_neighbourhoods(cloud, P, small, kfull)
        torch.cuda.synchronize()
        got = kfull[:n].cpu().numpy()
        np.testing.assert_array_equal(got[clear], np.minimum(want, 1 << 30)[clear])
        assert (kfull[n:] == -7).all()

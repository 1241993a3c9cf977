"""The induced velocity by boxes (large clouds) against the FP64 sum over all sources at
sampled targets: clouds that fill their boxes evenly and not, with empty boxes, on a line,
stretched by an outlier, of a few boxes (large eps), and counts at the edges of tiles; and
the cases that fall back to the direct sum.  FP32: 1e-5 relative L2 as for the direct sum
(an expansion leaves at most 2e-8 of a box's part)."""
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


def _cloud(kind, n, rng):
    h = 1.0 / np.sqrt(n)
    if kind == "lattice":
        k = int(np.ceil(np.sqrt(n)))
        gx, gy = np.meshgrid(np.arange(k), np.arange(k))
        x = (gx.ravel()[:n] + rng.uniform(-0.25, 0.25, n)) * h
        y = (gy.ravel()[:n] + rng.uniform(-0.25, 0.25, n)) * h
    elif kind == "gauss":
        x, y = rng.normal(0, 0.3, n), rng.normal(0, 0.3, n)
    elif kind == "rings":       # empty boxes inside
        a, r = rng.uniform(0, 2 * np.pi, n), rng.choice([1.0, 3.0], n) + rng.normal(0, 0.02, n)
        x, y = 50.0 + r * np.cos(a), -20.0 + r * np.sin(a)
    elif kind == "line":
        x, y = np.linspace(0, 1, n), np.zeros(n)
    elif kind == "outlier":
        x, y = rng.uniform(0, 1, n), rng.uniform(0, 1, n)
        x[3] = 1.0e4
    else:                       # one place
        x, y = np.full(n, 0.25), np.full(n, 0.5)
    return x.astype(np.float32), y.astype(np.float32), rng.normal(0, 1, n).astype(np.float32) / n, 3.0 * h


def _run(vrm, x, y, g, eps, count=None):
    n = x.size
    cloud = vrm.Cloud(x, y, g, capacity=n + 33)
    ctx = vrm.Context(cloud.capacity)
    u = torch.full((n + 33,), 7.0, device="cuda")
    v = torch.full((n + 33,), 7.0, device="cuda")
    ctx.vrm_biot_savart(cloud, eps, u, v)
    if count is not None:   # fewer on the device than the context knows of
        u.fill_(7.0)
        v.fill_(7.0)
        cloud.n_dev.fill_(count)
        ctx.vrm_biot_savart(cloud, eps, u, v)
    torch.cuda.synchronize()
    m = n if count is None else count
    assert (u[m:] == 7.0).all() and (v[m:] == 7.0).all()
    return u[:m], v[:m]


def _check(u, v, x, y, g, eps, rng):
    n = u.numel()
    at = torch.as_tensor(rng.permutation(n)[:1500], device="cuda")
    X, Y, G = [torch.as_tensor(a[:n].astype(np.float64), device="cuda") for a in (x, y, g)]
    dx, dy = X[at][:, None] - X[None], Y[at][:, None] - Y[None]
    r2 = dx * dx + dy * dy
    K = torch.where(r2 > 0, -torch.expm1(-r2 / eps ** 2) / (2 * np.pi * torch.where(r2 > 0, r2, 1.0)), 0.0)
    U, V = -(K * dy) @ G, (K * dx) @ G
    err = torch.sqrt(((u[at].double() - U) ** 2 + (v[at].double() - V) ** 2).sum())
    ref = torch.sqrt((U ** 2 + V ** 2).sum())
    print("  rel L2", float(err / ref) if float(ref) else float(err), flush=True)
    assert float(err) <= 1e-5 * float(ref)


@pytest.mark.parametrize("kind", ["lattice", "gauss", "rings", "line", "outlier"])
@pytest.mark.parametrize("n,scale", [(14000, 1.0), (30011, 1.0), (30011, 8.0)])
def test_boxes_against_all_pairs(vrm, n, scale, kind):
    rng = np.random.default_rng(n)
    x, y, g, eps = _cloud(kind, n, rng)
    print("case velocity", kind, n, scale, flush=True)
    u, v = _run(vrm, x, y, g, eps * scale)
    _check(u, v, x, y, g, eps * scale, rng)


@pytest.mark.parametrize("count", [0, 1, 127, 129, 20000])
def test_a_smaller_count_on_the_device(vrm, count):
    rng = np.random.default_rng(count)
    x, y, g, eps = _cloud("gauss", 20011, rng)
    u, v = _run(vrm, x, y, g, eps, count)
    if count > 1:
        _check(u, v, x, y, g, eps, rng)
    elif count == 1:
        assert float(u[0]) == 0.0 and float(v[0]) == 0.0


def test_one_place_and_values_that_are_not_finite(vrm):
    rng = np.random.default_rng(1)
    x, y, g, eps = _cloud("place", 15000, rng)
    u, v = _run(vrm, x, y, g, eps)
    assert (u == 0).all() and (v == 0).all()
    x, y, g, eps = _cloud("lattice", 15000, rng)
    for a in (x, g):
        bad = a.copy()
        bad[77] = np.nan
        u, v = _run(vrm, *((bad, y, g) if a is x else (x, y, bad)), eps)
        assert torch.isnan(u).all() and torch.isnan(v).all()   # as the sum over all pairs

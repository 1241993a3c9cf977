"""The induced velocity of clouds of 2 10^5 to 10^6 particles against the FP64 sum over all
sources at sampled targets: boxes of several tiles of targets, grids of larger boxes, and
clouds with boxes too full for an expansion, among them exactly 256 of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOX_MOST = 4096          # particles of a box that has an expansion


@pytest.fixture(scope="module")
def vrm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_06379_amd as v
    v.lib()
    return v


def _boxes(x, y, eps):
    """Counts of the boxes the library bins the cloud into (FP64)."""
    n = x.size
    lx, ly = float(x.max()) - float(x.min()), float(y.max()) - float(y.min())
    fill = 109 * max(1.0, np.floor(np.sqrt(n / 8.0) / 109 + 0.5))
    s = max(np.sqrt(lx * ly * fill / n), max(lx, ly) * fill / n, 2.1 * float(np.float32(eps)))
    nx, ny = int(lx / s) + 1, int(ly / s) + 1
    bx = np.minimum(((x.astype(np.float64) - x.min()) / s).astype(int), nx - 1)
    by = np.minimum(((y.astype(np.float64) - y.min()) / s).astype(int), ny - 1)
    return np.bincount(by * nx + bx, minlength=nx * ny)


def _cloud(kind, n, rng):
    h = 1.0 / np.sqrt(n)
    if kind == "lattice":
        k = int(round(np.sqrt(n)))
        gx, gy = np.meshgrid(np.arange(k), np.arange(k))
        x, y = gx.ravel() * h, gy.ravel() * h
    elif kind == "jittered":
        k = int(np.ceil(np.sqrt(n)))
        gx, gy = np.meshgrid(np.arange(k), np.arange(k))
        x = (gx.ravel()[:n] + rng.uniform(-0.25, 0.25, n)) * h
        y = (gy.ravel()[:n] + rng.uniform(-0.25, 0.25, n)) * h
    else:
        x, y = rng.normal(0, 0.3, n), rng.normal(0, 0.3, n)
    return x.astype(np.float32), y.astype(np.float32), (rng.normal(0, 1, n) / n).astype(np.float32), h


@pytest.mark.parametrize("kind,n,eps,over", [
    ("jittered", 250000, 3.0, 0),              # boxes of twice the fill
    ("gauss", 250000, 3.0, 0),                 # boxes of one to about twenty tiles
    ("gauss", 700000, 3.0, None),              # some boxes too full
    ("lattice", 1056 * 1056, 31.43, 256),      # 16 x 16 boxes, all too full
    ("lattice", 1056 * 1056, 31.0, 256),       # 17 x 17 boxes, all but the last row and column too full
])
def test_large_clouds_against_all_pairs(vrm, kind, n, eps, over):
    rng = np.random.default_rng(n)
    x, y, g, h = _cloud(kind, n, rng)
    n, eps = x.size, eps * h
    counts = _boxes(x, y, eps)
    full = int((counts > BOX_MOST).sum())
    assert full == over if over is not None else 0 < full < counts.size
    print("case many boxes", kind, n, "boxes", counts.size, "fullest", counts.max(), "too full", full, flush=True)
    cloud = vrm.Cloud(x, y, g, capacity=n + 64)
    ctx = vrm.Context(cloud.capacity)
    u = torch.full((n + 64,), 7.0, device="cuda")
    v = torch.full((n + 64,), 7.0, device="cuda")
    ctx.vrm_biot_savart(cloud, eps, u, v)
    torch.cuda.synchronize()
    assert (u[n:] == 7.0).all() and (v[n:] == 7.0).all()
    at = torch.as_tensor(rng.permutation(n)[:400], device="cuda")
    X, Y, G = [torch.as_tensor(a.astype(np.float64), device="cuda") for a in (x, y, g)]
    err = ref = 0.0
    for part in at.split(50):
        dx, dy = X[part][:, None] - X[None], Y[part][:, None] - Y[None]
        r2 = dx * dx + dy * dy
        K = torch.where(r2 > 0, -torch.expm1(-r2 / eps ** 2) / (2 * np.pi * torch.where(r2 > 0, r2, 1.0)), 0.0)
        U, V = -(K * dy) @ G, (K * dx) @ G
        err += float(((u[part].double() - U) ** 2 + (v[part].double() - V) ** 2).sum())
        ref += float((U ** 2 + V ** 2).sum())
    # FP32 sums in a row: half an ulp of the running sum each, a random walk.  Directly up to
    # all N terms; by boxes an eighth of the 25 boxes around, and 2e-8 from the expansions
    terms = n if full else 25 * counts.max() / 8
    tol = np.sqrt(terms) * 2.0 ** -24 + 2e-8
    print("  rel L2", np.sqrt(err / ref), "tolerance", tol, flush=True)
    assert np.sqrt(err / ref) <= tol

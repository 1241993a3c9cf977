"""Insertion with more candidates than one workgroup resolves, bit for bit against the
oracle: the order by marks of ids below the capacity, by sorting where ids are larger or
not unique, a chain that takes more rounds than one batch holds, and a full cloud."""
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


def _oracle(orc, P, x, y, g, ids, q=2):
    mask, _, _ = orc.diffused(g, ids, P.h, q)
    X, Y, G, I, nc = orc.insert(x.astype(np.float64), y.astype(np.float64), g.astype(np.float64), ids, mask, P)
    return X.astype(np.float32), Y.astype(np.float32), G.astype(np.float32), I, nc


def _holes(n, seed):
    """A jittered lattice with every third particle gone."""
    rng = np.random.default_rng(seed)
    k = int(np.ceil(np.sqrt(1.5 * n)))
    gx, gy = np.meshgrid(np.arange(k), np.arange(k))
    keep = np.sort(rng.permutation(k * k)[:n])
    x = (gx.ravel()[keep] + rng.uniform(-0.2, 0.2, n)) * 0.05
    y = (gy.ravel()[keep] + rng.uniform(-0.2, 0.2, n)) * 0.05
    return x.astype(np.float32), y.astype(np.float32), rng.uniform(0.5, 1.0, n).astype(np.float32)


# ids: 0..n-1, in another order, just below the capacity, from it up, and spread far
@pytest.mark.parametrize("ids", ["dense", "permuted", "below", "at", "far"])
@pytest.mark.parametrize("n", [1200, 4111])
def test_order_of_the_inserted(vrm, orc, n, ids):
    wl = workloads.config_jittered(h=0.05, q=2, seed=3, jitter=0.4)
    x, y, g = _holes(n, n)
    cap = 5 * n + 3
    rng = np.random.default_rng(5)
    i = {"dense": np.arange(n), "permuted": rng.permutation(n), "below": cap - n + rng.permutation(n),
         "at": cap - n + 1 + rng.permutation(n), "far": 1000003 * rng.permutation(n) % (1 << 30)}[ids].astype(np.int32)
    assert np.unique(i).size == n
    P = vrm.params_of(wl)
    X, Y, G, I, nc = _oracle(orc, orc.params_of(wl), x, y, g, i)
    cloud = vrm.Cloud(x, y, g, ids=i, capacity=cap)
    ctx = vrm.Context(cap + 17)
    print("case insert", n, ids, "candidates", nc, "to", X.size, flush=True)
    assert nc > 1024
    ctx.vrm_insert_particles(cloud, P)
    cnt = ctx.vrm_read_counters()
    assert (cnt["n_candidates"], cnt["n_inserted"], cnt["n"]) == (nc, X.size - n, X.size)
    a = cloud.numpy()
    o, r = np.argsort(a[3]), np.argsort(I)
    for got, want in zip(a, (X, Y, G, I)):
        np.testing.assert_array_equal(got[o], want[r])
    # the same context once more (by id: the order of the particles of a cell is open)
    mid = vrm.Cloud(x, y, g, ids=i, capacity=cap)
    ctx.vrm_insert_particles(mid, P)
    b = mid.numpy()
    p = np.argsort(b[3])
    for got, want in zip(b, a):
        np.testing.assert_array_equal(got[p], want[o])


def test_ids_that_are_not_unique(vrm):
    """The same particles appended (their order among equal keys is open)."""
    n = 1500
    wl = workloads.config_jittered(h=0.05, q=2, seed=3, jitter=0.4)
    x, y, g = _holes(n, 9)
    i = (np.arange(n) // 2).astype(np.int32)
    res = []
    for shift in (0, 1 << 24):
        cloud = vrm.Cloud(x, y, g, ids=i + shift, capacity=6 * n)
        ctx = vrm.Context(cloud.capacity)
        ctx.vrm_insert_particles(cloud, vrm.params_of(wl))
        a = cloud.numpy()
        assert ctx.vrm_read_counters()["n"] == a[0].size > n
        new = a[3] > i.max() + shift
        assert np.array_equal(np.sort(a[3][new]), np.arange(new.sum()) + i.max() + 1 + shift)
        o = np.lexsort((a[1], a[0]))
        res.append((a[0][o], a[1][o], a[2][o]))
    for p, q in zip(*res):
        np.testing.assert_array_equal(p, q)


def test_a_chain_longer_than_a_batch_of_rounds(vrm, orc):
    """A line of lone particles with ids along it: each one's candidates wait for those of
    the one before."""
    wl = workloads.config_jittered(h=0.05, q=2, seed=3, jitter=0.4)
    n = 600
    x = (np.arange(n) * 0.9 * 0.05).astype(np.float32)
    y = np.zeros(n, np.float32)
    g = np.ones(n, np.float32)
    ids = np.arange(n, dtype=np.int32)
    X, Y, G, I, nc = _oracle(orc, orc.params_of(wl), x, y, g, ids)
    cloud = vrm.Cloud(x, y, g, capacity=9 * n)
    ctx = vrm.Context(cloud.capacity)
    ctx.vrm_insert_particles(cloud, vrm.params_of(wl))
    cnt = ctx.vrm_read_counters()
    print("candidates", nc, "rounds", cnt["mis_rounds"], flush=True)
    assert nc > 1024 and cnt["mis_rounds"] % 4 == 0 and cnt["n_inserted"] == X.size - n
    a = cloud.numpy()
    o, r = np.argsort(a[3]), np.argsort(I)
    for got, want in zip(a, (X, Y, G, I)):
        np.testing.assert_array_equal(got[o], want[r])


def test_a_cloud_without_room(vrm):
    wl = workloads.config_jittered(h=0.05, q=2, seed=3, jitter=0.4)
    n = 2000
    x, y, g = _holes(n, 21)
    P = vrm.params_of(wl)
    cloud = vrm.Cloud(x, y, g, capacity=n + 100)
    ctx = vrm.Context(3 * n)
    before = cloud.numpy()
    with pytest.raises(vrm.VrmError) as e:
        ctx.vrm_insert_particles(cloud, P)
    assert e.value.code == vrm.E_CAPACITY
    for a, b in zip(before, cloud.numpy()):
        np.testing.assert_array_equal(a, b)
    need = ctx.vrm_read_counters()["capacity_needed"]
    roomy = vrm.Cloud(x, y, g, capacity=3 * n)
    ctx.vrm_insert_particles(roomy, P)
    assert roomy.n == need

"""Selection (Sec. 3.5) by three passes over 11, 11 and 10 bits of the key, whose last
workgroup picks the bin: against a sort in FP64 on the host, and against the entry
point without a context (four passes of 8 bits); and the count the first pass reads."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TIE_BAND = np.float32(1.0 - 2.0 ** -16)


@pytest.fixture(scope="module")
def vrm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_06379_amd as v
    v.lib()
    return v


def _host_mask(g, bound):
    """|Gamma| >= fl32(T (1 - 2^-16)), T the first value whose cumulative sum passes the bound."""
    a = np.abs(g)
    s = np.sort(a)
    cum = np.cumsum(s.astype(np.float64))
    # the inputs stay clear of a tie between the sum and the bound: the order of the
    # FP64 additions moves the sums by less than n 2^-53 of the total
    assert np.abs(cum - bound).min() > g.size * 2.0 ** -53 * cum[-1]
    above = np.nonzero(cum > bound)[0]
    if above.size == 0:
        return np.zeros(g.size, np.uint8)
    return (a >= s[above[0]] * TIE_BAND).astype(np.uint8)


def _gamma(kind, n, rng):
    if kind == "decades":       # bins far apart, zeros and subnormals among them
        g = 10.0 ** rng.uniform(-42, 3, n)
    elif kind == "one_bin":     # one bin of the first two passes
        g = 1.0 + rng.integers(0, 1024, n) * 2.0 ** -23
    else:                       # one value
        g = np.full(n, 0.3)
    g = (g * rng.choice([-1.0, 1.0], n)).astype(np.float32)
    if kind == "decades":
        g[rng.random(n) < 0.1] = 0.0
        g[0] = 100.0
    return g


# one particle, the edges of a wave, a workgroup and the whole grid of 256 x 1024
@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1025, 262143, 262145, 600001])
@pytest.mark.parametrize("kind", ["decades", "one_bin", "one_value"])
def test_selection_against_a_sort(vrm, n, kind):
    rng = np.random.default_rng(n)
    g = _gamma(kind, n, rng)
    x, y = rng.uniform(0, 1, n), rng.uniform(0, 1, n)
    cloud = vrm.Cloud(x, y, g, capacity=n + 8)
    ctx = vrm.Context(cloud.capacity)
    mask = torch.full((n + 8,), 7, dtype=torch.uint8, device="cuda")
    flat = torch.full((n + 8,), 7, dtype=torch.uint8, device="cuda")
    for h, c_diff in ((0.07, 1.0), (0.61, 2.0), (0.9, 5.0)):   # the last: above the norm, none
        print("case select", n, kind, h, flush=True)
        bound = c_diff * h ** 3 * np.abs(g.astype(np.float64)).sum()
        want = _host_mask(g, bound)
        P = vrm.make_params(h=h, q=2, c_diff=c_diff)
        ctx.vrm_select_diffused(cloud, P, mask)
        vrm.vrm_select_diffused_static(cloud.gamma, n, h, 2, c_diff, flat)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(mask[:n].cpu().numpy(), want)
        np.testing.assert_array_equal(flat[:n].cpu().numpy(), want)
        assert (mask[n:] == 7).all() and (flat[n:] == 7).all()
        assert ctx.vrm_read_counters()["n_diffused"] == int(want.sum())


def test_the_count_is_the_devices(vrm):
    """A count changed behind the context is the one selected and inserted for; one out
    of range is refused, and the next call is as if it had not been."""
    wl = workloads.config_jittered(h=0.05, q=2, seed=3, jitter=0.4)
    P = vrm.params_of(wl)
    n = wl.x.size
    cloud = vrm.Cloud(wl.x, wl.y, wl.gamma, capacity=4 * n)
    ctx = vrm.Context(cloud.capacity)
    start = [t.clone() for t in (cloud.x, cloud.y, cloud.gamma, cloud.id)]
    for count in (n, n // 2, 0, n):
        for t, s in zip((cloud.x, cloud.y, cloud.gamma, cloud.id), start):
            t.copy_(s)
        for bad in (-1, cloud.capacity + 1):
            cloud.n_dev.fill_(bad)
            with pytest.raises(vrm.VrmError) as e:
                ctx.vrm_insert_particles(cloud, P)
            assert e.value.code == vrm.E_ARG
        cloud.n_dev.fill_(count)
        ctx.vrm_insert_particles(cloud, P)
        got = [a[np.argsort(cloud.numpy()[3])] for a in cloud.numpy()]
        fresh = vrm.Cloud(wl.x[:count], wl.y[:count], wl.gamma[:count], capacity=4 * n)
        other = vrm.Context(cloud.capacity)
        other.vrm_insert_particles(fresh, P)
        want = [a[np.argsort(fresh.numpy()[3])] for a in fresh.numpy()]
        print("count", count, "after", got[0].size, flush=True)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
        assert got[0].size >= count

"""Cell lists whose grid would have more than 2^24 cells on a side: a few particles far
apart in a context of 2^23 particles or more."""
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


@pytest.mark.parametrize("along", ["x", "y"])
@pytest.mark.parametrize("capacity", [1 << 23, (1 << 23) + 12345])
def test_the_last_cell_of_a_long_side(vrm, capacity, along):
    """Two neighbours at each end of a strip of 10^9 cells: each has the other, and a
    lone particle between them none."""
    h = 0.05
    near = np.array([0.0, h, 5.0e7, 1.0e8, 1.0e8])
    other = np.array([0.0, 0.0, 0.0, 0.0, h])
    x, y = (near, other) if along == "x" else (other, near)
    n = x.size
    cloud = vrm.Cloud(x, y, np.ones(n), capacity=n)
    ctx = vrm.Context(capacity)
    P = vrm.make_params(h=h, q=2, r=0.5, R=2.0)
    kfull = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    small = torch.full((n, 8), -7, dtype=torch.int32, device="cuda")
    print("case long grid", capacity, along, flush=True)
    for _ in range(2):   # the second build finds the counts cleared
        ctx.vrm_set_diffused(cloud, torch.ones(n, dtype=torch.uint8, device="cuda"))
        ctx.vrm_build_neighbourhoods(cloud, P, small, kfull)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(kfull.cpu().numpy(), [1, 1, 0, 1, 1])
        got = [sorted(set(row.tolist()) - {-1}) for row in small.cpu().numpy()]
        assert got == [[1], [0], [], [4], [3]]
    assert ctx.vrm_read_counters()["n_grid_clamped"] == 2

"""Deterministic sums: the stages of a step give the same bits whatever the context did
before.  A particle whose stencil of one stage comes from its complete neighbourhood has
no basis of five to leave for the next one, also where an earlier step left one."""
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


@pytest.mark.parametrize("q", [2, 3])
def test_the_same_bits_after_another_step(vrm, q):
    """Stage 0 on holes (complete neighbourhoods for q = 2), then every particle at another
    place, then stage 1; once in a new context and once in one that did stage 0 there, with
    small neighbourhoods, before."""
    wl = workloads.config_jittered(h=0.02, q=q, seed=5, jitter=0.1)
    rng = np.random.default_rng(6)
    n = wl.n
    P = vrm.params_of(wl, deterministic=1)
    # a tenth of the particles pushed together: their neighbours have empty segments
    x0, y0 = wl.x.copy(), wl.y.copy()
    move = rng.random(n) < 0.1
    x0[move] += np.float32(0.8 * wl.h)
    y0[move] += np.float32(0.3 * wl.h)
    zero = torch.zeros(n, device="cuda")
    ones = torch.ones(n, dtype=torch.uint8, device="cuda")
    out, full = [], []
    for used in (False, True):
        cloud = vrm.Cloud(x0, y0, wl.gamma, capacity=n)
        ctx = vrm.Context(n)

        def put(x, y):
            cloud.x[:n] = torch.as_tensor(x, device="cuda")
            cloud.y[:n] = torch.as_tensor(y, device="cuda")

        ctx.vrm_set_diffused(cloud, ones)
        if used:
            put(wl.x, wl.y)
            ctx.vrm_rk_stage(cloud, P, 0, zero, zero)   # (the velocity leaves the cell list to be rebuilt)
            cloud.gamma[:n] = torch.as_tensor(wl.gamma, device="cuda")
            put(x0, y0)
        before = ctx.vrm_read_counters()["n_full"]
        ctx.vrm_rk_stage(cloud, P, 0, zero, zero)
        full.append(ctx.vrm_read_counters()["n_full"] - before)
        put(wl.x, wl.y)
        ctx.vrm_rk_stage(cloud, P, 1, zero, zero)
        torch.cuda.synchronize()
        out.append(cloud.gamma[:n].cpu().numpy())
    print("case reproducible", q, "complete", full, "differ", int((out[0] != out[1]).sum()), flush=True)
    assert full[0] == full[1] > 0
    np.testing.assert_array_equal(out[0].view(np.uint32), out[1].view(np.uint32))

"""The two kernels of a training step at the sizes where their tiles end: 16-row tiles in
blocks of 32 rows, one tile per workgroup up to 4096 rows, more of them above."""
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


def _bf(t):
    return t.to(torch.bfloat16).double()


def _reference(theta, X, T, wf):
    """Loss and gradient in FP64 with BF16 roundings where the operands of the products
    are BF16: inputs, weights, activations and the derivatives that enter a product."""
    import paper_1508_06379_amd.learned as L
    parts, o = [], 0
    for shape in L.SHAPES:
        n = int(np.prod(shape))
        parts.append(theta[o:o + n].double().reshape(shape))
        o += n
    W1, b1, W2, b2, W3, b3 = parts
    W1, W2, W3 = _bf(W1), _bf(W2), _bf(W3)
    k, c = np.sqrt(2.0 / np.pi), 0.044715

    def gelu(z):
        return 0.5 * z * (1.0 + torch.tanh(k * (z + c * z ** 3)))

    def grad(z):
        t = torch.tanh(k * (z + c * z ** 3))
        return 0.5 * (1.0 + t) + 0.5 * z * (1.0 - t * t) * k * (1.0 + 3.0 * c * z * z)

    X, T = X.double(), T.double()
    rows = X.shape[0]
    z1 = X @ W1 + b1
    h1 = _bf(gelu(z1))
    z2 = h1 @ W2 + b2
    h2 = _bf(gelu(z2))
    y = h2 @ W3 + b3
    m = X[:, 64:96]
    z, p = y[:, :32], y[:, 32:]
    loss = (m * (torch.nn.functional.softplus(z) - T[:, :32] * z + wf * (p - T[:, 32:]) ** 2)).sum() / rows
    dy = torch.cat([m * (torch.sigmoid(z) - T[:, :32]), m * wf * 2.0 * (p - T[:, 32:])], 1) / rows
    dz2 = (_bf(dy) @ W3.t()) * grad(z2)
    dz1 = (_bf(dz2) @ W2.t()) * grad(z1)
    return loss, [X.t() @ _bf(dz1), dz1.sum(0), h1.t() @ _bf(dz2), dz2.sum(0), h2.t() @ _bf(dy), dy.sum(0)]


@pytest.mark.parametrize("rows", [1, 15, 17, 31, 33, 4095, 4113, 8209])
def test_step_at_the_edges_of_the_tiles(vrm, rows):
    import paper_1508_06379_amd.learned as L
    gen = torch.Generator().manual_seed(rows)
    theta = torch.as_tensor(L.init_params(3)) + 0.02 * torch.randn(vrm.MLP_PARAMS, generator=gen)
    pad = 40
    X = torch.randn(rows + pad, 128, generator=gen)
    X[:, 64:96] = (torch.rand(rows + pad, 32, generator=gen) < 0.7).float()
    T = torch.rand(rows + pad, 64, generator=gen)
    X[rows:] = float("nan")   # past the rows: not read
    T[rows:] = float("nan")
    Xb = X.to(torch.bfloat16)
    Xd = Xb.view(torch.int16).cuda()
    Td = T.cuda()
    ctx = vrm.Context(64)
    ctx.vrm_mlp_load(theta.cuda())
    grad = torch.full((vrm.MLP_PARAMS + 8,), 7.0, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    print("case train", rows, flush=True)
    ctx.vrm_mlp_train_step(Xd, Td, rows, 0.0, 0.0, 0.3, loss, grad)
    torch.cuda.synchronize()
    g = grad.cpu()
    assert (g[vrm.MLP_PARAMS:] == 7.0).all()
    ref_loss, ref = _reference(theta, Xb[:rows].float(), T[:rows], 0.3)
    # the loss's terms are FP32 of FP32 sums over 128 products; BF16 activations that
    # round to the other neighbour (2^-8 relative, at most one in 16) move an L2 norm by
    # 2^-8 / 4
    assert abs(float(loss.item()) - float(ref_loss)) <= 1e-3 * abs(float(ref_loss))
    o = 0
    for r in ref:
        n = r.numel()
        a = g[o:o + n].double().reshape(r.shape)
        rel = float((a - r).norm() / r.norm())
        print("  block", tuple(r.shape), "rel", rel, flush=True)
        assert rel <= 1e-3
        o += n
    # an input that is not 16-byte aligned, and a second run: the same bits
    buf = torch.zeros(Xd.numel() + 1, dtype=torch.int16, device="cuda")
    buf[1:] = Xd.flatten()
    again = torch.zeros(vrm.MLP_PARAMS, device="cuda")
    ctx.vrm_mlp_train_step(buf[1:], Td, rows, 0.0, 0.0, 0.3, None, again)
    torch.cuda.synchronize()
    assert torch.equal(again.cpu(), g[:vrm.MLP_PARAMS])
    # a step: the network that infers afterwards is the one that is read out
    ctx.vrm_mlp_train_step(Xd, Td, rows, 1e-2, 1e-2, 0.3)
    w = torch.zeros(vrm.MLP_PARAMS, device="cuda")
    ctx.vrm_mlp_read(w)
    assert float((w.cpu() - theta).abs().max()) > 1e-3
    fresh = vrm.Context(64)
    fresh.vrm_mlp_load(w)
    n = min(rows, 256)
    ya, yb = torch.zeros(n, 64, device="cuda"), torch.zeros(n, 64, device="cuda")
    ctx.vrm_mlp_infer(Xd, n, ya)
    fresh.vrm_mlp_infer(Xd, n, yb)
    torch.cuda.synchronize()
    assert torch.equal(ya, yb)

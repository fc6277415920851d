"""The training kernels at the edges of their 64-record workgroups and of the
partial sums' slices: loss and gradient, and the gradient of sum dc c, against
the network in FP64 (torch autograd), and one training step against the two calls."""
import numpy as np
import pytest

from tests._gpu_common import need_gpu

pytestmark = pytest.mark.gpu


def _data(n, seed):
    rng = np.random.default_rng(seed)
    feat = np.stack([rng.uniform(-9, 5, n), rng.uniform(-1, 1, n), rng.uniform(-27, 0, n), rng.normal(0.97, 0.02, n)], 1)
    l1 = 10.0 ** rng.uniform(-3, 2, n)
    l2 = l1 * rng.uniform(-0.99, 0.99, n)
    p = rng.standard_normal(n)
    rec = np.stack([p + 0.1 * rng.standard_normal(n), p, l1, l2, l1 * l1 - l2 * l2, np.full(n, 1.0 / n)], 1)
    par = np.concatenate([rng.uniform(-0.4, 0.4, 1248), [0.5]])
    return feat.astype(np.float32), rec.astype(np.float32), par.astype(np.float32)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 511, 513, 4096 + 3])
def test_loss_grad_and_step(n):
    torch = need_gpu()
    from paper_2502_04217_amd import csipm
    feat, rec, par = _data(n, n)
    dev = lambda a: torch.tensor(a, device="cuda")
    f, r, p = dev(feat), dev(rec), dev(par)
    loss, grad = csipm.mlp_loss_grad(p, f, r)
    t = torch.tensor(par, dtype=torch.float64, requires_grad=True)
    x, q = torch.tensor(feat, dtype=torch.float64), torch.tensor(rec, dtype=torch.float64)
    h = torch.tanh(x @ t[:128].view(32, 4).T + t[128:160])
    o = torch.tanh(h @ t[160:1184].view(32, 32).T + t[1184:1216]) @ t[1216:1248] + t[1248]
    c = torch.nn.functional.softplus(o) + 1e-6
    ref = (q[:, 5] * (q[:, 2] ** 2 + q[:, 3] ** 2) / (q[:, 2] + q[:, 4]) ** 2 * (q[:, 0] - c * q[:, 1]) ** 2).sum()
    g, = torch.autograd.grad(ref, t, retain_graph=True)
    # FP32 network (about 60 roundings of 6e-8 along a path), FP64 sums
    assert abs(loss.item() - ref.item()) <= 1e-5 * ref.item()
    assert (grad.cpu().double() - g).norm() <= 1e-5 * g.norm()
    dc = np.random.default_rng(1).standard_normal(n).astype(np.float32)
    gb, = torch.autograd.grad((c * torch.tensor(dc, dtype=torch.float64)).sum(), t)
    start = torch.full((1249,), 0.25, device="cuda")
    back = csipm.mlp_backward(p, f, dev(dc), start.clone())
    assert (back.cpu().double() - 0.25 - gb).norm() <= 1e-5 * gb.norm() + 1249 ** 0.5 * 0.25 * 6e-8
    m, v, p2 = torch.zeros_like(p), torch.zeros_like(p), p.clone()
    l2, g2 = csipm.mlp_train_step(p2, m, v, 1, 1e-3, f, r)
    m3, v3, p3 = torch.zeros_like(p), torch.zeros_like(p), p.clone()
    csipm.mlp_adam(p3, grad, m3, v3, 1, 1e-3)
    assert torch.equal(l2, loss) and torch.equal(g2, grad)
    assert torch.equal(p2, p3) and torch.equal(m, m3) and torch.equal(v, v3)

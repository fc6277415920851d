"""The network's inference on the matrix cores (the 32x32 layer as products of
bf16 parts): record counts around a chunk of 64, a workgroup and the grid,
against 64 bits, and infinite and NaN features and weights."""
import pytest

from paper_2502_04217_amd import csipm

pytestmark = pytest.mark.gpu


def _layers(p):
    return p[:128].view(32, 4), p[128:160], p[160:1184].view(32, 32), p[1184:1216], p[1216:1248], p[1248]


def _exact(p, x):
    import torch
    w1, b1, w2, b2, w3, b3 = _layers(p.double())
    h1 = torch.tanh(x.double() @ w1.t() + b1)
    h2 = torch.tanh(h1 @ w2.t() + b2)
    o = h2 @ w3 + b3
    return h1, h2, torch.clamp(o, min=0) + torch.log1p(torch.exp(-o.abs())) + 1e-6


@pytest.mark.parametrize("scale", [0.1, 1.0, 3.0])
@pytest.mark.parametrize("n", [1, 15, 17, 63, 64, 65, 257, 655361])
def test_forward_against_64_bits(n, scale):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    p = torch.randn(1249, device="cuda", generator=g) * scale
    x = torch.randn(n, 4, device="cuda", generator=g) * 3.0
    c = csipm.mlp_forward(p, x).double()
    w1, b1, w2, b2, w3, b3 = _layers(p.double().abs())
    h1, h2, want = _exact(p, x)
    # sums of k terms: k half-ulps of the sum of magnitudes; tanh to 2^-21
    # absolute, plus its argument's error (slope at most 1)
    u = 2.0 ** -24
    e1 = 6 * u * (x.double().abs() @ w1.t() + b1) + 2.0 ** -21
    e2 = e1 @ w2.t() + 34 * u * (h1.abs() @ w2.t() + b2) + 2.0 ** -21
    eo = e2 @ w3 + 34 * u * (h2.abs() @ w3 + b3)
    assert bool(((c - want).abs() <= eo + 8 * u * want).all())


def test_infinities_and_nan():
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    p = torch.randn(1249, device="cuda", generator=g)
    x = torch.randn(96, 4, device="cuda", generator=g)
    x[3, 1] = float("inf")
    x[70, 2] = -float("inf")
    x[64, 0] = float("nan")
    c = csipm.mlp_forward(p, x).double()
    want = _exact(p, x)[2]
    assert bool(torch.isnan(c[64])) and int(torch.isnan(c).sum()) == 1
    ok = ~torch.isnan(want)
    assert float((c - want)[ok].abs().max()) <= 1e-3
    q = p.clone()
    q[160 + 32 * 5 + 7] = float("inf")      # one infinite weight saturates its neuron
    q[160 + 32 * 20 + 9] = -3.4028234e38    # (the largest finite one: no overflow to NaN)
    c = csipm.mlp_forward(q, x).double()
    want = _exact(q, x)[2]
    assert float((c - want)[~torch.isnan(want)].abs().max()) <= 1e-3 and int(torch.isnan(c).sum()) == 1
    q[160 + 32 * 5 + 7] = float("nan")
    assert bool(torch.isnan(csipm.mlp_forward(q, x)).all())

"""The operators of a small grid in one launch, at the edges of that route:
the smallest grids, the largest it takes (6144 points) and the next larger
ones, one long extent, extents of 1, non-power-of-two plans, and arrays that
start at an odd element of the beta side."""
import numpy as np
import pytest

from oracle import dft3
from paper_2502_04217_amd import csipm
from paper_2502_04217_amd import workload as wl

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 4), (1, 2, 4), (2, 1, 6), (3, 5, 4), (4, 4, 4), (7, 9, 10), (8, 8, 16), (8, 16, 8), (16, 16, 16),
          (20, 14, 18), (16, 16, 24), (6, 32, 32), (16, 18, 24), (1, 6, 1024), (1024, 1, 6), (1, 1024, 6),
          (1, 1, 1024), (2, 1024, 4), (25, 27, 8)]


@pytest.mark.parametrize("shape", SHAPES)
def test_operators_of_small_grids(shape):
    import torch
    rng = np.random.default_rng(11)
    obs = (rng.random(shape) > 0.2).astype(np.uint8)
    obs.ravel()[0] = 1
    n = obs.size
    pr = csipm.Problem(np.where(obs, rng.standard_normal(shape), 0.0), obs)
    s1, s2 = wl.random_barrier(shape, 3, spread=1.0)
    pr.set_barrier(torch.tensor(s1, device="cuda"), torch.tensor(s2, device="cuda"))
    pb, pz, x = (rng.standard_normal(shape) for _ in range(3))
    h = dft3.apply_At(obs * dft3.apply_A(pb))
    d, a = s1 + s2, s1 - s2
    for dt, eps in ((torch.float64, 2.0 ** -53), (torch.float32, 2.0 ** -24)):
        tol = 8 * eps * (2 * np.log2(n) + 1)   # a few eps per radix-2 level of two transforms

        def dev(v):
            buf = torch.zeros(n + 1, dtype=dt, device="cuda")
            buf[1:] = torch.tensor(v.ravel(), device="cuda").to(dt)
            return buf[1:].view(shape)
        qb, qz = pr.apply_K(dev(pb), dev(pz))
        for got, want in ((qb, h + d * pb + a * pz), (qz, a * pb + d * pz), (pr.apply_A(dev(pb)), dft3.apply_A(pb)),
                          (pr.apply_H(dev(pb)), h),
                          (pr.apply_At(torch.tensor(x, device="cuda").to(dt)), dft3.apply_At(x))):
            assert np.max(np.abs(got.double().cpu().numpy() - want)) <= tol * np.max(np.abs(want))


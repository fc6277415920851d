"""The operator applies' axis-1 passes on the caller's arrays in the external
layout, and the row pairs of an odd N3, at the edges of their tiles: every
operator against the oracle with one extent at a time around the tile widths
(16 pencils of FP32, 8 of FP64 and their multiples), N3/2 smaller than a
tile, odd pencil counts (the last row pair has one row), both parities, long
pencils in numbers that take narrower tiles (down to 4 pencils, and to 1 pair of
rows), and arrays that start at an odd element (the beta side takes any element
alignment)."""
import numpy as np
import pytest

from oracle import dft3
from paper_2502_04217_amd import csipm
from paper_2502_04217_amd import workload as wl

pytestmark = pytest.mark.gpu

SHAPES = [(4, 3, 6), (5, 7, 4), (8, 1, 32), (16, 2, 32), (6, 6, 14), (9, 16, 30), (18, 5, 10), (64, 3, 16),
          (10, 10, 36), (256, 2, 4), (3, 5, 7), (5, 5, 3), (1, 1, 15), (2, 7, 45), (15, 1, 49), (10, 3, 27),
          (7, 9, 125), (64, 4, 9), (1, 15, 21), (3, 1, 945), (1, 1, 945), (9, 27, 315), (1, 63, 75), (980, 3, 6),
          (600, 16, 16), (2, 735, 10), (75, 2, 60), (315, 5, 15)]


def _err(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("shape", SHAPES)
def test_operators_on_the_callers_arrays(shape):
    import torch
    rng = np.random.default_rng(7)
    obs = (rng.random(shape) > 0.2).astype(np.uint8)
    obs.ravel()[0] = 1
    n = obs.size
    pr = csipm.Problem(np.where(obs, rng.standard_normal(shape), 0.0), obs)
    s1, s2 = wl.random_barrier(shape, 3, spread=1.0)
    pr.set_barrier(torch.tensor(s1, device="cuda"), torch.tensor(s2, device="cuda"))
    pb, pz, x = (rng.standard_normal(shape) for _ in range(3))
    h = dft3.apply_At(obs * dft3.apply_A(pb))
    for dt, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
        def dev(a):   # element 1 of a larger buffer: no 16- (or 8-) byte alignment
            buf = torch.zeros(n + 1, dtype=dt, device="cuda")
            buf[1:] = torch.tensor(a.ravel(), device="cuda").to(dt)
            return buf[1:].view(shape)
        d, a, b = s1 + s2, s1 - s2, dev(pb)
        assert _err(pr.apply_A(b).double().cpu().numpy(), dft3.apply_A(pb)) <= tol
        assert _err(pr.apply_H(b).double().cpu().numpy(), h) <= tol
        qb, qz = (q.double().cpu().numpy() for q in pr.apply_K(b, dev(pz)))
        assert _err(qb, h + d * pb + a * pz) <= tol and _err(qz, a * pb + d * pz) <= tol
        y = pr.apply_At(torch.tensor(x, device="cuda").to(dt)).double().cpu().numpy()
        assert _err(y, dft3.apply_At(x)) <= tol

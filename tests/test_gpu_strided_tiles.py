"""The power-of-two strided passes at the edges of their tiles (rows of 128
bytes: 8 pencils of FP64, 16 of FP32; 256 bytes on the forward pass of axis 1;
more where a workgroup would not be a whole wave): pencil counts one row (or two) short
of a tile, one tile, one row more, and the longest pencils, whose tiles are
bound by LDS and the threads of a workgroup."""
import numpy as np
import pytest

from oracle import dft3
from paper_2502_04217_amd import csipm
from paper_2502_04217_amd import workload as wl

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1, 14), (64, 1, 16), (64, 3, 6), (32, 15, 4), (32, 16, 4), (32, 18, 4), (16, 30, 4), (16, 35, 4),
          (8, 9, 14), (128, 1, 30), (256, 4, 4), (256, 3, 6), (512, 1, 36), (512, 3, 4), (1024, 1, 18), (1024, 3, 4),
          (3, 64, 6), (1, 128, 36), (5, 512, 4), (3, 1024, 6), (1, 1024, 16)]


@pytest.mark.parametrize("shape", SHAPES)
def test_tile_edges(shape):
    import torch
    rng = np.random.default_rng(5)
    obs = (rng.random(shape) > 0.2).astype(np.uint8)
    obs.ravel()[0] = 1
    pr = csipm.Problem(np.where(obs, rng.standard_normal(shape), 0.0), obs)
    s1, s2 = wl.random_barrier(shape, 3, spread=1.0)
    pr.set_barrier(torch.tensor(s1, device="cuda"), torch.tensor(s2, device="cuda"))
    pb, pz = rng.standard_normal(shape), rng.standard_normal(shape)
    h = dft3.apply_At(obs * dft3.apply_A(pb))
    d, a = s1 + s2, s1 - s2
    for dt, eps in ((torch.float64, 2.0 ** -53), (torch.float32, 2.0 ** -24)):
        # a radix stage adds a few eps to each value; two transforms of log2 n
        # radix-2 levels each, and the rounded input
        tol = 8 * eps * (2 * np.log2(obs.size) + 1)
        qb, qz = (q.double().cpu().numpy()
                  for q in pr.apply_K(*(torch.tensor(v, device="cuda").to(dt) for v in (pb, pz))))
        for got, want in ((qb, h + d * pb + a * pz), (qz, a * pb + d * pz)):
            assert np.max(np.abs(got - want)) <= tol * np.max(np.abs(want))

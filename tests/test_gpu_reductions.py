"""The finalize kernels of the solves at partial counts around their wave
and unroll widths (1, 2, 64, 70 and 2048 partials per quantity): the residual
measures and the certificate sums of an iterate against the same sums formed
by numpy, and a breakdown-free solve whose steps come from alpha formed in the
update pass."""
import numpy as np
import pytest

from oracle import dft3, ipm
from paper_2502_04217_amd import csipm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (16, 16, 8), (64, 32, 32), (32, 40, 56), (128, 128, 128)])
def test_residual_measures(shape):
    rng = np.random.default_rng(9)
    obs = (rng.random(shape) > 0.2).astype(np.uint8)
    obs.ravel()[0] = 1
    pr = csipm.Problem(np.where(obs, rng.standard_normal(shape), 0.0), obs)
    lam = pr.lambda_rule(0.05)
    info = pr.solve(tol=1e-12, precision=csipm.FP64, max_iter=4)
    assert info["ipm_iters"] == 4 and info["status_name"] == "NOT_CONVERGED"
    res = pr.residuals()
    beta, z, nu1, nu2 = (pr.get(k).cpu().numpy() for k in (csipm.BETA, csipm.Z, csipm.NU1, csipm.NU2))
    g = dft3.apply_At(obs * (dft3.apply_A(beta) - pr.signal.cpu().numpy()))
    c1, c2 = (z + beta) * nu1, (z - beta) * nu2
    # n additions in any order: n eps of the sum of magnitudes (all positive);
    # the transform pair a few eps per radix-2 level of max |g|
    eps, n = 2.0 ** -53, obs.size
    scale = np.max(np.abs(g)) + lam
    assert abs(res["mu"] - (c1.sum() + c2.sum()) / (2 * n)) <= n * eps * res["mu"] + 4 * eps * scale
    assert abs(res["compl_max"] - max(c1.max(), c2.max())) <= 4 * eps * res["compl_max"]
    tol = 32 * eps * (np.log2(n) + 1) * scale
    assert abs(res["res_beta_inf"] - np.max(np.abs(g - nu1 + nu2))) <= tol
    assert abs(res["res_z_inf"] - np.max(np.abs(lam - nu1 - nu2))) <= tol
    assert abs(res["g_inf"] - np.max(np.abs(g))) <= tol
    cert = ipm.lasso_certificate(beta, pr.signal.cpu().numpy(), obs, lam)
    assert abs(res["objective"] - cert.primal) <= (n * eps + 1e-13) * abs(cert.primal)

"""Noise-parameter draw where the score's slope overflows at the search's first point:
an n_corr 1e152 times as strong as the white noise, f_knee at the spectrum's
logarithmic middle, so that at alpha = 0 the score of some 1e307 is finite and its
derivative is not.  The counts c_b are then 1e-300 of the score's other term, and
alpha is the root of sum J_b x_b e^(-alpha x_b), here by bisection in 64 bits;
1e-12, as for the draw elsewhere."""
import numpy as np
import pytest
import torch
from scipy import optimize

from oracle import noise as on
from test_gpu_row_launches import layout

pytestmark = pytest.mark.gpu


def test_slope_overflow():
    from paper_2201_03509_amd import ops
    n, fs = 4096, 32.5
    rng = np.random.default_rng(21)
    nc = np.where(np.arange(n) % 2, rng.normal(size=n), 0.0)
    w = np.where(np.arange(n) % 2, 0.0, 4.5e-153 * rng.normal(size=n))
    fk = 5.0
    J, c, f = on.periodogram_bins(nc, fs)
    sigma0 = np.sqrt((w @ w) / on.wilson_hilferty_chi2(n, 0.0))
    x, a = np.log(f / fk), J / sigma0 ** 2
    with np.errstate(over="ignore"):
        assert np.isfinite(a).all() and np.isfinite(np.sum(np.abs(a * x))) and np.isinf(np.sum(a * x * x))
    ref = optimize.brentq(lambda al: np.sum(J * x * np.exp(-al * x)), -1.0, 1.0, xtol=1e-15, rtol=1e-15)
    assert 0.01 < abs(ref) < 0.9
    c_ = ops.Context(0)
    try:
        tod = layout([n])
        dev = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float64)).cuda()
        s0, fkn, al = (torch.empty(1, dtype=torch.float64, device="cuda") for _ in range(3))
        c_.sample_noise(tod, "fp64", dev(nc + w), dev(np.zeros(n)), dev(nc), 1, 2, s0, fkn, al, mean_only=True,
                        fknee=dev([fk]))
        c_.sync()
        s0, al = float(s0[0]), float(al[0])
    finally:
        c_.close()
    assert abs(s0 - sigma0) <= 1e-12 * sigma0
    assert abs(al - ref) <= 1e-12 * abs(ref), (al, ref)

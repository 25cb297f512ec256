"""FP64 mode arithmetic of the compiled rows at the ends of its range, over short
rows (4096 samples) and long ones (100000).

A segment whose alpha is NaN gets NaN everywhere, as its filter has no value
(the other segments are not touched).  With alpha = -90 the filter
1/(sigma0^2 + P_k) meets q = (f/f_knee)^90 from 0 to 1.7e308, a fifth of the
modes beyond 1e300, where it is 1/sigma0^2: the gain and its width against the
oracle within 1e-12 (ln(f/f_knee) is off by some units of 2e-16 times its
largest term, 90 times that is 3e-13 of q, and q counts where it is near 1).

chi^2 of a faint n_corr (1e-9 sigma0) that is the whole TOD, under a flat spectrum
of 1: its value is the sum of |n_k|^2 / P_k, 1e-18 each, with nothing larger beside
them; 1e-12 of it, as of any sum of magnitudes."""
import numpy as np
import pytest
import torch

import synth
from oracle import gain as og
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu


def make(n):
    return synth.make(1, nscan=3, length=("list", n), bands=(Band(64, 32.5, 1),), keep_truth=True)


@pytest.mark.parametrize("mean_only", [True, False])
@pytest.mark.parametrize("n", [4096, 100000])
def test_nan_parameter_stays_nan(n, mean_only):
    from paper_2201_03509_amd import ops
    ts = make(n)
    s = ot.project_all(ts, ts.maps, ts.pix, ts.psi)
    ts.alpha[1] = np.nan
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        out = torch.zeros(ts.nsamp, dtype=torch.float64, device="cuda")
        c.sample_ncorr(tod, "fp64", tod.d, torch.from_numpy(s).cuda(), 5, 1, out, mean_only=mean_only)
        with pytest.raises(ops.CorruptStream):
            c.sync()
        assert c.device_error_bits() == 64
        got = out.cpu().numpy().reshape(3, n)
    finally:
        c.close()
    assert np.isnan(got[1]).all() and np.isfinite(got[0]).all() and np.isfinite(got[2]).all()


@pytest.mark.parametrize("n", [4096, 100000])
def test_steep_filter(n):
    from paper_2201_03509_amd import ops
    ts = make(n)
    t = ot.project(ts.maps, ot.global_pix(ts, ts.pix), ts.psi, 1.0)
    ts.alpha[:] = -90.0
    ts.fknee[:] = 0.5 * 32.5 / 2660.0
    ts.sigma0[:] = (0.25, 1.0, 3.0)
    q = 2660.0 ** 90
    assert 1.7e308 < q < np.inf
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        g, sg = (torch.empty(3, dtype=torch.float64, device="cuda") for _ in range(2))
        c.sample_gain(tod, "fp64", tod.d, torch.from_numpy(t).cuda(), 5, 1, g, sg)
        c.sync()
        g, sg = g.cpu().numpy(), sg.cpu().numpy()
    finally:
        c.close()
    ref, ref_s = og.sample_gain_all(ts, ts.d, t, 5, 1)
    assert np.all(np.abs(sg - ref_s) <= 1e-12 * ref_s)
    assert np.all(np.abs(g - ref) <= 1e-12 * np.abs(ref))


@pytest.mark.parametrize("n", [4096, 100000])
def test_faint_whittle_sum(n):
    from paper_2201_03509_amd import ops
    ts = make(n)
    ts.alpha[:] = -1e-280
    ts.sigma0[:] = 1.0
    ts.maps[:] = 0.0
    nc = 1e-9 * np.random.default_rng(8).normal(size=ts.nsamp)
    ref = ot.chisq_all(ts, ts.maps, ts.pix, ts.psi, nc, nc)
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
        J = torch.empty(ts.nseg, dtype=torch.float64, device="cuda")
        c.tod_chisq(tod, "fp64", dev(ts.pix.astype(np.int32)), dev(ts.psi.astype(np.uint16)), dev(nc), dev(nc),
                    dev(ts.maps), J)
        c.sync()
        got = J.cpu().numpy()
    finally:
        c.close()
    assert np.all(np.abs(got - ref) <= 1e-12 * ref), (got, ref)

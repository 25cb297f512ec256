"""Maps read as records where samples do not return to their pixel: 700 segments shorter
than the revisit period, 1.3e6 samples over 2e5 pixels (under 16 a pixel, so that the
pixel changes alone choose the records).  Projection and the chi^2's map adjoint
against 64-bit references (1e-5 of FP32 values, 1e-12 of FP64 and of the adjoint's
sums of magnitudes); the sweep, eager on its first call (the period is probed
there) and replayed from its graph after, against the steps called one by one."""
import numpy as np
import pytest
import torch

import synth
from synth.configs import Band
from test_gpu_tile_parts import template

pytestmark = pytest.mark.gpu

NSIDE, SEGS = 128, 700


@pytest.fixture(scope="module")
def ts():
    t = synth.make(1, nscan=SEGS, length=("uniform", 1700, 1940), bands=(Band(NSIDE, 32.5, 1),), keep_truth=True)
    # the most frequent lag of the first three segments repeats few pixels: at least
    # 1e6 changes, and half the map's pixels (0.7 in FP64)
    segs = [t.pix[t.seg_off[q]:t.seg_off[q + 1]] for q in range(3)]
    equal = {lag: sum(int(np.sum(p[lag:] == p[:-lag])) for p in segs if len(p) > lag) for lag in range(64, 1940)}
    lag = max(equal, key=equal.get)
    q = equal[lag] / sum(max(0, len(p) - lag) for p in segs)
    assert (1 - q) * t.nsamp >= 1e6 and t.npix_total <= 1e6 and t.nsamp < 16 * t.npix_total
    return t


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_records_without_revisits(ts, prec):
    from paper_2201_03509_amd import ops
    ft, tol = (torch.float32, 1e-5) if prec == "mixed" else (torch.float64, 1e-12)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        pix, psi = dev(ts.pix.astype(np.int32)), dev(ts.psi.astype(np.uint16))
        maps = dev(ts.maps).to(ft)
        seg = torch.repeat_interleave(torch.arange(ts.nseg, device="cuda"), dev(np.diff(ts.seg_off)))
        Pm = template(maps, pix, dev(ts.psi.astype(np.int32)))
        g = tod.gain[seg]
        s = torch.empty(ts.nsamp, dtype=ft, device="cuda")
        c.project_sky(tod, prec, pix, psi, maps, s)
        assert torch.linalg.norm(s.double() - g * Pm) <= tol * torch.linalg.norm(g * Pm)
        # the sweep: eager, then twice from its graph, against the steps
        steps = torch.empty_like(s)
        for it in range(3):
            o = ops.new_outputs(tod, prec)
            c.tod_sweep(tod, prec, maps, 7, it, o["ncorr"], o["acc"], o["pix"], o["psi"], use_graph=True)
            c.sample_ncorr(tod, prec, tod.d, s, 7, it, steps)
            c.sync()
            assert torch.linalg.norm((o["ncorr"] - steps).double()) <= 2 * tol * torch.linalg.norm(steps.double())
            assert torch.equal(o["acc"][9].long(), torch.bincount(pix, minlength=ts.npix_total))
        # the map adjoint: -2 g r / sigma0^2 (1, c, s) summed per pixel
        gm = torch.empty((3, ts.npix_total), dtype=torch.float64, device="cuda")
        c.tod_chisq_backward(tod, prec, pix, psi, tod.d, steps, maps, 1.0, gm)
        c.sync()
        a = torch.pi * (2.0 * dev(ts.psi.astype(np.float64)) + 1.0) / 2048.0
        w = -2.0 * g / tod.sigma0[seg] ** 2 * (tod.d.double() - g * Pm - steps.double())
        for j, f in enumerate((torch.ones_like(a), torch.cos(a), torch.sin(a))):
            z = torch.zeros(ts.npix_total, dtype=torch.float64, device="cuda")
            ref, mag = z.index_add(0, pix.long(), w * f), z.index_add(0, pix.long(), (w * f).abs())
            assert torch.all((gm[j] - ref).abs() <= 1e-12 * mag), j
    finally:
        c.close()

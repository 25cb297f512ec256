"""Strided tiles cut along time, at the edges of their parts: few segments, so
that every launch is split, with revisit counts just below, at and above a
multiple of the eight in flight, one lane per tile (stride 1), a stride as
long as the segment, an odd group (three detectors), coarse maps where whole
waves of neighbouring lanes hold one pixel (their records are summed before
they are added), and both forms of the maps (planes; records where samples
outnumber pixels 16 to 1).  Bars as in the parity suites."""
import numpy as np
import pytest
import torch

import synth
from chisq_bounds import magnitudes
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu

TOL = {"mixed": 1e-5, "fp64": 1e-12}
# nside, detectors, segment length, stride
SETS = [(2, 2, 4097, 1), (2, 2, 2100, 700), (8, 3, 4160, 65), (8, 3, 4161, 64), (8, 2, 4095, 64),
        (64, 3, 4097, 513), (64, 2, 2048, 2048), (64, 1, 3001, 257)]


@pytest.mark.parametrize("nside,ndet,n,stride", SETS)
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_split_tiles(prec, nside, ndet, n, stride):
    from paper_2201_03509_amd import ops
    ts = synth.make(1, nscan=2, length=("list", n, n - 1), bands=(Band(nside, 32.5, ndet),), keep_truth=True)
    nf, tf = (np.float32, torch.float32) if prec == "mixed" else (np.float64, torch.float64)
    rng = np.random.default_rng(n)
    maps, nc = ts.maps.astype(nf), (0.3 * rng.normal(size=ts.nsamp)).astype(nf)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    pix, psi = dev(ts.pix.astype(np.int32)), dev(ts.psi.astype(np.uint16))
    c = ops.Context(0)
    try:
        c.set_bin_stride(0, stride)
        tod = ops.DeviceTod(ts, "cuda:0")
        s = torch.empty(ts.nsamp, dtype=tf, device="cuda")
        c.project_sky(tod, prec, pix, psi, dev(maps), s)
        acc = ops.new_acc(ts.npix_total, "cuda")
        c.bin_tod(tod, prec, pix, psi, tod.d, dev(nc), acc)
        J = torch.empty(ts.nseg, dtype=torch.float64, device="cuda")
        c.tod_chisq(tod, prec, pix, psi, tod.d, dev(nc), dev(maps), J)
        gm = torch.empty((3, ts.npix_total), dtype=torch.float64, device="cuda")
        gg = torch.empty(ts.nseg, dtype=torch.float64, device="cuda")
        c.tod_chisq_backward(tod, prec, pix, psi, tod.d, dev(nc), dev(maps), 1.0, gm, gg)
        c.sync()
        s, acc, J, gm, gg = (x.cpu().numpy() for x in (s, acc, J, gm, gg))
    finally:
        c.close()
    m_r, nc_r = maps.astype(np.float64), nc.astype(np.float64)
    tol = TOL[prec]
    ref = ot.project_all(ts, m_r, ts.pix, ts.psi)
    assert np.linalg.norm(s - ref) <= tol * np.linalg.norm(ref)
    b, A, hits = ot.bin_tod(ts, ts.pix, ts.psi, ts.d, nc_r)
    assert np.array_equal(acc[9], hits)
    assert np.linalg.norm(acc[:3] - b) <= 1e-12 * np.linalg.norm(b)
    assert np.linalg.norm(acc[3:9] - A) <= 1e-12 * np.linalg.norm(A)
    eps = float(np.finfo(nf).eps)
    mag, fft, gmag = magnitudes(ts, m_r, nc_r, eps)
    Jr = ot.chisq_all(ts, m_r, ts.pix, ts.psi, ts.d, nc_r)
    assert np.all(np.abs(J - Jr) <= tol * mag[0] + fft[0])
    gr = ot.chisq_grad_all(ts, m_r, ts.pix, ts.psi, ts.d, nc_r)
    hit = gmag > 0
    assert np.all(gm[~hit] == 0.0)
    assert np.all(np.abs(gm[hit] - gr[0][hit]) <= 1e-12 * gmag[hit])
    assert np.all(np.abs(gg - gr[1]) <= tol * mag[1])

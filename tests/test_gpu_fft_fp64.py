"""FP64 transforms on the compiled kernels: every row length (160..512 and
1200..2400), each with one of the register column lengths in turn (even ones,
whose rows k1 = 0 and M1/2 share a task, and odd ones, whose row k1 = 0 is
paired with another segment's or, of the last segment, with itself), in every
mode, against the oracle.

Bounds: n_corr and the gain 1e-12 of their norm, the chi^2 1e-12 of its terms'
magnitudes plus the transforms' rounding (chisq_bounds), as for the generic
FP64 kernels.  The noise draw: periodogram bins carry 4 eps log2 N = 1.5e-14 of
their size and the fitted parameters at most some hundred times that: 1e-11."""
import json

import numpy as np
import pytest
import torch

import synth
from chisq_bounds import magnitudes
from oracle import gain as og
from oracle import noise as on
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu

TOL = 1e-12
COLS = [16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81]


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


SHORT = [160, 180, 192, 200, 216, 225, 240, 250, 256, 270, 288, 300, 320, 324, 360, 384, 400, 405, 432, 450, 480,
         486, 500, 512]
LONG = [L for L in range(1200, 2401) if _smooth(L)]
CASES = [(COLS[i % len(COLS)], L) for i, L in enumerate(SHORT + LONG)]


def _rows(L):
    r = []
    while L > 1:
        r.append(max(c for c in (2, 3, 4, 5, 6, 8, 9, 10) if L % c == 0))
        L //= r[-1]
    return r


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d" % c)
def test_compiled_fp64(tmp_path, case):
    from paper_2201_03509_amd import ops
    M1, L = case
    M = M1 * L
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"fft": [{"mixed": 0, "M": M, "M1": M1, "M2": L, "B": 64, "colreg": 1, "r1": [],
                                         "r2": _rows(L)}], "bin_stride": {}}))
    # three segments: n = M, and M the next 5-smooth number above n where there
    # is room (odd and even n, an odd sample offset)
    lens = [M] + [n if not any(_smooth(m) for m in range(n, M)) else M for n in (M - 1, M - 2)]
    ts = synth.make(1, nscan=3, length=("list", *lens), bands=(Band(64, 32.5, 1),), keep_truth=True)
    t = ot.project(ts.maps, ot.global_pix(ts, ts.pix), ts.psi, 1.0)
    s = t * np.repeat(ts.gain, np.diff(ts.seg_off))
    seed, it = 53, 4
    refs = [ot.sample_ncorr_all(ts, ts.d, s, seed, it, mean_only=mo) for mo in (False, True)]
    nc = refs[0]
    c = ops.Context(0)
    try:
        c.load_tuning(str(path))
        tod = ops.DeviceTod(ts, "cuda:0")
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
        f64 = dict(dtype=torch.float64, device="cuda")
        outs = []
        for mo, d in ((False, tod.d), (False, tod.d.double()), (True, tod.d.double())):
            out = torch.empty(ts.nsamp, **f64)
            c.sample_ncorr(tod, "fp64", d, dev(s), seed, it, out, mean_only=mo)
            outs.append((mo, out))
        sw = ops.new_outputs(tod, "fp64")
        c.tod_sweep(tod, "fp64", dev(ts.maps), seed, it, sw["ncorr"], sw["acc"], sw["pix"], sw["psi"])
        outs.append((False, sw["ncorr"]))
        g = torch.empty(ts.nseg, **f64)
        c.sample_gain(tod, "fp64", tod.d, dev(t), seed, it, g)
        J = torch.empty(ts.nseg, **f64)
        c.tod_chisq(tod, "fp64", dev(ts.pix.astype(np.int32)), dev(ts.psi.astype(np.uint16)), tod.d, dev(nc),
                    dev(ts.maps), J)
        nz = [torch.empty(ts.nseg, **f64) for _ in range(3)]
        c.sample_noise(tod, "fp64", tod.d, dev(t), dev(nc), seed, it, *nz, fknee=dev(np.asarray(ts.fknee, float)))
        c.sync()
    finally:
        c.close()
    for j, (mo, out) in enumerate(outs):
        got = out.cpu().numpy()
        for q in range(ts.nseg):
            a, b = ts.seg_off[q], ts.seg_off[q + 1]
            ref = refs[1 if mo else 0][a:b]
            assert np.linalg.norm(got[a:b] - ref) <= TOL * np.linalg.norm(ref), (j, q)
    g_ref, _ = og.sample_gain_all(ts, ts.d, t, seed, it)
    assert np.all(np.abs(g.cpu().numpy() - g_ref) <= TOL * np.abs(g_ref))
    mag, fft, _ = magnitudes(ts, ts.maps, nc, float(np.finfo(np.float64).eps))
    J_ref = ot.chisq_all(ts, ts.maps, ts.pix, ts.psi, ts.d, nc)
    assert np.all(np.abs(J.cpu().numpy() - J_ref) <= TOL * mag[0] + fft[0])
    nz_ref = on.sample_noise_all(ts, ts.d, t, ts.gain, nc, ts.fknee, seed, it)
    got = np.stack([x.cpu().numpy() for x in nz])
    assert (np.abs(got - nz_ref) / np.abs(nz_ref)).max() < 1e-11

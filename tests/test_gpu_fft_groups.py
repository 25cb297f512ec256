"""FFT launches that serve several lengths at once: segments whose column and
row lengths fall into every class of the compiled kernels (columns up to 36, 64
and 100; rows of both register classes; rows k1 = 0 and M1/2 paired across
segments; a short transform on the generic kernels) in one call, against the
oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu

# complex lengths 16 x 2000, 16 x 2500, 64 x 2000, 64 x 4860, 75 x 4860, generic; padded ones
LENGTHS = (32000, 40000, 128000, 311040, 364500, 4096, 31993, 363999)


def draw(lengths, r, prec):
    from paper_2201_03509_amd import ops
    ts = synth.make(1, nscan=len(lengths), length=("list",) + lengths, bands=(Band(16, 32.5, 1),))
    tf = torch.float32 if prec == "mixed" else torch.float64
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        d = torch.from_numpy(np.concatenate(r)).cuda()
        out = torch.empty(ts.nsamp, dtype=tf, device="cuda")
        c.sample_ncorr(tod, prec, d, torch.zeros(ts.nsamp, dtype=tf, device="cuda"), 3, 0, out, mean_only=True)
        c.sync()
        return ts, np.split(out.cpu().numpy(), ts.seg_off[1:-1])
    finally:
        c.close()


def test_lengths_share_launches():
    rng = np.random.default_rng(4)
    r = [(np.cumsum(rng.normal(size=n)) * 0.01 + rng.normal(size=n)).astype(np.float32) for n in LENGTHS]
    ts, got = draw(LENGTHS, r, "mixed")
    for q, n in enumerate(LENGTHS):
        ref = ot.sample_ncorr_segment(r[q].astype(np.float64), 32.5, ts.sigma0[q], ts.fknee[q], ts.alpha[q], 3, q, 0,
                                      mean_only=True)
        assert np.linalg.norm(got[q] - ref) <= 1e-5 * np.linalg.norm(ref), n

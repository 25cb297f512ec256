"""FP32 columns of 64 points at both occupancies they are compiled for: 40 blocks a
segment (rows of 2500 points), 3 segments (two waves per SIMD) and 64 (2560 blocks:
three), in every form of input.  n_corr of FP32 and of FP64 data and of the masked
draw with nothing masked (a whole extended vector in), and the gain, of the first
and the last segment against the oracle: 1e-5."""
import numpy as np
import pytest
import torch

from oracle import gain as og
from oracle import tod as ot
from test_gpu_row_launches import layout

pytestmark = pytest.mark.gpu

N = 64 * 2500


@pytest.mark.parametrize("nseg", [3, 64])
def test_both_occupancies(nseg):
    from paper_2201_03509_amd import ops
    c = ops.Context(0)
    try:
        tod = layout([N] * nseg)
        g = torch.Generator("cuda").manual_seed(nseg)
        rand = lambda: torch.randn(tod.nsamp, device="cuda", generator=g)
        d, s = rand(), 0.3 * rand()
        t = 1.0 + s
        outs = [torch.empty_like(d) for _ in range(3)]
        c.sample_ncorr(tod, "mixed", d, s, 3, 1, outs[0])
        c.sample_ncorr(tod, "mixed", d.double(), s, 3, 1, outs[1])
        c.sample_ncorr_masked(tod, "mixed", d, s, torch.ones(tod.nsamp, dtype=torch.uint8, device="cuda"), 3, 1, outs[2])
        gain = torch.empty(nseg, dtype=torch.float64, device="cuda")
        c.sample_gain(tod, "mixed", d + t, t, 3, 1, gain)
        c.sync()
        gain = gain.cpu().numpy()
        for q in (0, nseg - 1):
            f64 = lambda x: x[q * N:(q + 1) * N].cpu().numpy().astype(np.float64)
            ref = ot.sample_ncorr_segment(f64(d) - f64(s), 32.5, 1.0, 0.1, -1.2, 3, q, 1)
            for i, o in enumerate(outs):
                assert np.linalg.norm(f64(o) - ref) <= 1e-5 * np.linalg.norm(ref), (i, q)
            g_ref = og.sample_gain_segment(f64(d + t), f64(t), 32.5, 1.0, 0.1, -1.2, 3, q, 1)[0]
            assert abs(gain[q] - g_ref) <= 1e-5 * abs(g_ref), q
    finally:
        c.close()

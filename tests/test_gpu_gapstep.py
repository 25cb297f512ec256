"""Masked draw, the vector part of a CG iteration: gap lists of less than a tile,
of exactly some tiles, of one entry pair more, and of more tiles than a wave has
lanes (1024 extended entries a tile), with a segment without masked samples and
one with a few beside it, against the oracle's iterates.  Bar: the FP64
one of the masked draw, 1e-12 of each segment's norm."""
import numpy as np
import pytest
import torch

import synth
from oracle import gapfill as og
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked", [12, 512, 4097, 32768, 40000])
def test_gap_list_sizes(masked):
    from paper_2201_03509_amd import ops
    n = max(2 * masked, 300)
    ts = synth.make(1, nscan=3, length=("list", n, 777, 500), bands=(Band(64, 32.5, 1),), keep_truth=True)
    mask = np.ones(ts.nsamp, dtype=np.uint8)
    rng = np.random.default_rng(masked)
    start = rng.integers(0, n - masked + 1)
    mask[start:start + masked] = 0  # one gap
    mask[n + 777 + 13:n + 777 + 32] = 0  # 19 samples of the third, none of the second
    s = ot.project_all(ts, ts.maps, ts.pix, ts.psi)
    seed, it = 9, 2
    ref, _ = og.cg_ncorr_all_gap(ts, ts.d, s, mask, seed, it, tol=0.0, maxiter=4)
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        out = torch.empty(ts.nsamp, dtype=torch.float64, device="cuda")
        iters = torch.empty(ts.nseg, dtype=torch.int32, device="cuda")
        for _ in range(2):  # the second call finds the counters as the first left them
            c.sample_ncorr_masked(tod, "fp64", tod.d, torch.from_numpy(s).cuda(), torch.from_numpy(mask).cuda(), seed,
                                  it, out, tol=0.0, max_iter=4, iters=iters)
            c.sync()
            got = out.cpu().numpy()
            for q in range(ts.nseg):
                a, b = ts.seg_off[q], ts.seg_off[q + 1]
                assert np.linalg.norm(got[a:b] - ref[a:b]) <= 1e-12 * np.linalg.norm(ref[a:b]), q
            k = iters.cpu().numpy()
            assert k[1] == 0 and k[0] != 0
    finally:
        c.close()

"""Masked draw with gap lists of so many tiles (1024 extended entries each) that their
sums are added up in groups of 64 first: 400 tiles, the last size without groups,
401 (six groups and 17 tiles), and 448 (seven whole groups), with a segment
without masked samples and one with a few beside it, against the oracle's
iterates.  Bar: the FP64 one of the masked draw, 1e-12 of each segment's norm.
The launches an iteration, three or five, tell which way the sums went."""
import numpy as np
import pytest
import torch

import synth
from oracle import gapfill as og
from oracle import tod as ot
from synth.configs import Band

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked,launches", [(204800, 3), (204801, 5), (229376, 5)])
def test_many_gap_tiles(masked, launches):
    from paper_2201_03509_amd import ops
    n = 240000
    ts = synth.make(1, nscan=3, length=("list", n, 777, 500), bands=(Band(64, 32.5, 1),), keep_truth=True)
    mask = np.ones(ts.nsamp, dtype=np.uint8)
    mask[5000:5000 + masked] = 0
    mask[n + 777 + 13:n + 777 + 32] = 0  # 19 samples of the third, none of the second
    s = ot.project_all(ts, ts.maps, ts.pix, ts.psi)
    seed, it = 9, 2
    ref, _ = og.cg_ncorr_all_gap(ts, ts.d, s, mask, seed, it, tol=0.0, maxiter=4)
    c = ops.Context(0)
    try:
        tod = ops.DeviceTod(ts, "cuda:0")
        out = torch.empty(ts.nsamp, dtype=torch.float64, device="cuda")
        iters = torch.empty(ts.nseg, dtype=torch.int32, device="cuda")
        dev = (tod.d, torch.from_numpy(s).cuda(), torch.from_numpy(mask).cuda())
        c.enable_timing(True)
        count = []
        for k in (2, 4):
            c.sample_ncorr_masked(tod, "fp64", *dev, seed, it, out, tol=0.0, max_iter=k, iters=iters)
            count.append(c.kernel_times()["cg_vector"][1])
        c.sync()
        got, k = out.cpu().numpy(), iters.cpu().numpy()
    finally:
        c.close()
    assert count[1] - count[0] == 2 * launches
    for q in range(ts.nseg):
        a, b = ts.seg_off[q], ts.seg_off[q + 1]
        assert np.linalg.norm(got[a:b] - ref[a:b]) <= 1e-12 * np.linalg.norm(ref[a:b]), q
    assert k[0] == -4 and k[1] == 0

"""FP32 rows: which lengths share a launch.  Lengths of one register class (2000, 2250 and
2304 points; 25 tasks of two rows a segment) have launches of their own from
kOwnPoints points each, or all of them from (k - 1) times that together on, and
share one below.  The launches are counted by the library's kernel timing, and
n_corr of a segment of each length is held against the oracle (1e-5) either way."""
import os
import re
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from oracle import tod as ot

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_03509_amd", "csrc")
POINTS = int(re.search(r"kOwnPoints = (\d+);", open(os.path.join(CSRC, "tune.h")).read()).group(1))
M1, TASKS = 50, 25   # rows k1 and M1 - k1 a task, 1..24; rows 0 and 25 in one


def layout(lens):
    """A layout without streams: `lens` are the segments' lengths."""
    from paper_2201_03509_amd import ops
    m, off = len(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    z = lambda n, t: np.zeros(n, t)
    h = SimpleNamespace(words=z(1, np.uint32), seg_word_off=z(m + 1, np.int64), seg_table=z(m, np.int32),
                        tables=z(40, np.uint32), table_off=np.array([0, 40]), chunk_bit=z(1, np.uint32),
                        chunk_prev=z(1, np.int32), seg_chunk_off=z(m + 1, np.int64), chunk_len=32)
    return ops.DeviceTod(SimpleNamespace(
        nseg=m, nband=1, ndet=1, nsamp=int(off[-1]), npix_total=12, seg_off=off, seg_band=z(m, np.int32),
        seg_det=z(m, np.int32), seg_accept=np.ones(m, np.uint8), band_nside=[1], band_npix=[12], band_pix_off=[0],
        band_fsamp=[32.5], d=z(1, np.float32), gain=np.ones(m), sigma0=np.ones(m), fknee=np.full(m, 0.1),
        alpha=np.full(m, -1.2), pix_huff=h, psi_huff=h), "cuda:0")


def least(points, *lengths):
    """segments of each length that together have at least so many points"""
    return -(-points // (TASKS * sum(lengths)))


A, B, C = 2000, 2250, 2304
TWO, THREE, ONE = least(POINTS, A, B), least(2 * POINTS, A, B, C), least(POINTS, A)


@pytest.mark.parametrize("counts,launches", [
    ({A: 2}, 1), ({A: TWO - 1, B: TWO - 1}, 1), ({A: TWO, B: TWO}, 2), ({A: ONE - 5, B: 2}, 1), ({A: ONE, B: 2}, 2),
    ({A: 2, B: 2, C: 2}, 1), ({A: ONE, B: 2, C: 2}, 2), ({A: THREE - 1, B: THREE - 1, C: THREE - 1}, 1),
    ({A: THREE, B: THREE, C: THREE}, 3)], ids=str)
def test_launches(counts, launches):
    from paper_2201_03509_amd import ops
    lens = [M1 * L for L, m in counts.items() for _ in range(m)]
    c = ops.Context(0)
    try:
        tod = layout(lens)
        g = torch.Generator("cuda").manual_seed(1)
        d = torch.randn(tod.nsamp, device="cuda", generator=g)
        out = torch.empty_like(d)
        c.enable_timing(True)
        c.kernel_times()
        c.sample_ncorr(tod, "mixed", d, torch.zeros_like(d), 3, 1, out)
        n = c.kernel_times()["fft_row"][1]
        c.sync()
        assert n == launches
        first = np.concatenate([[0], np.cumsum(list(counts.values()))])
        for q in list(first[:-1]) + [len(lens) - 1]:
            a, b = int(tod.h_seg_off[q]), int(tod.h_seg_off[q + 1])
            r = d[a:b].cpu().numpy().astype(np.float64)
            ref = ot.sample_ncorr_segment(r, 32.5, 1.0, 0.1, -1.2, 3, int(q), 1)
            assert np.linalg.norm(out[a:b].cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref), q
    finally:
        c.close()

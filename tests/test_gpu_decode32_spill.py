"""The decoders of 32-symbol chunks beyond what a block holds on chip, with the conditions
asserted on the host: in "dense" a segment of 70016 samples, nearly all of
different differences, has blocks of 512 chunks whose words do not fit the
block's LDS (and a last, short one whose words do) while the stream's average
keeps the decoder; in "symbols" one table holds more symbols than the block.
Bit-exact against the arrays that were encoded; the error word stays clear."""
import os
import re

import numpy as np
import pytest
import torch

import synth
from synth.configs import Band
from test_gpu_decode32 import encode

pytestmark = pytest.mark.gpu

SRC = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_03509_amd", "csrc",
                        "decode.hip")).read()
KSP, KSQ = (int(x) for x in re.search(r"KSP = (\d+), KSQ = (\d+);", SRC).groups())
CHUNKS, PER = 512, 36     # chunks of a block, words a chunk may touch
up16 = lambda n: (n + 15) // 16 * 16
lds = lambda ks: up16(up16(34 * 8 + 34 * 4 + 24 + 4096) + 2 * (ks + 2))       # a stream's table and symbols
PAIR = (163840 // 2 - 256 - (lds(KSP) + lds(KSQ))) // 4                       # words two streams may stage
ONE = (163840 // 3 // 1280 * 1280 - 256 - lds(KSQ)) // 4
LENGTHS = (33, 2049, 16384 + 7, 0, 40001, 70016)


def spans(*streams):
    """Words that each block of 512 chunks touches, over the streams together."""
    out = []
    h0 = streams[0]
    for s in range(len(h0.seg_chunk_off) - 1):
        a, b = int(h0.seg_chunk_off[s]), int(h0.seg_chunk_off[s + 1])
        for c in range(a, b, CHUNKS):
            last = min(c + CHUNKS, b) - 1
            out.append(sum((int(h.chunk_bit[last]) >> 5) - (int(h.chunk_bit[c]) >> 5) + PER for h in streams))
    return np.array(out)


def on_chip(room, *streams):
    """The rule that picks the decoder: 512 chunks of the average size, a twentieth to spare."""
    words = sum(len(h.words) for h in streams)
    return words / len(streams[0].chunk_bit) * CHUNKS * 1.05 + 2 * PER <= room


def test_rooms():
    assert (PAIR, ONE) == (12000, 8144)


@pytest.mark.parametrize("kind", ["dense", "symbols"])
def test_beyond_the_block(kind):
    from paper_2201_03509_amd import ops
    rng = np.random.default_rng(12)
    ts = synth.make(1, nscan=len(LENGTHS), length=("list",) + LENGTHS, bands=(Band(1024, 32.5, 1),))
    npix = ts.npix_total
    pix, psi, tod = [], [], []
    for i, n in enumerate(LENGTHS):
        if kind == "symbols":
            jump = rng.random(n) < 0.3
            pix.append(np.cumsum(np.where(jump, rng.integers(-npix, npix, n), 1)) % npix)
            psi.append(np.cumsum(rng.integers(-3, 4, n)) % 4096)
            tod.append(np.cumsum(np.where(jump, rng.integers(-200000, 200000, n), rng.integers(-9, 10, n))))
        elif n == max(LENGTHS):
            pix.append(rng.integers(0, npix, n)), psi.append(rng.integers(0, 4096, n))
            tod.append(rng.integers(-2**28, 2**28, n))
        else:
            pix.append(np.full(n, 5 + i)), psi.append(np.full(n, 4095)), tod.append(np.full(n, -7))
    one = [0] * len(LENGTHS) if kind == "symbols" else None
    hp, hs, ht = encode(pix, one), encode(psi), encode(tod, one)
    assert on_chip(PAIR, hp, hs) and on_chip(ONE, ht)
    both, single = spans(hp, hs), spans(ht)
    if kind == "dense":
        assert both.max() > PAIR and single.max() > ONE and both[-1] <= PAIR and single[-1] <= ONE
    else:
        assert hp.tables[0] > KSP and ht.tables[0] > KSQ
    ts.pix_huff, ts.psi_huff, ts.tod_huff, ts.flag_huff = hp, hs, ht, ht
    ts.tod_quantum = 0.25
    c = ops.Context(0)
    try:
        dt = ops.DeviceTod(ts, "cuda:0")
        e = lambda t: torch.empty(ts.nsamp, dtype=t, device="cuda")
        p, s, p2, s2 = e(torch.int32), e(torch.uint16), e(torch.int32), e(torch.uint16)
        f32, f64, fl, mk = e(torch.float32), e(torch.float64), e(torch.int32), e(torch.uint8)
        c.decode_pointing(dt, p, s)
        c.decode_pointing_noalloc(dt, p2, s2)
        c.decode_tod(dt, "mixed", f32)
        c.decode_tod(dt, "fp64", f64)
        c.decode_flags(dt, 5, fl, mk)
        c.sync()
        p, s, p2, s2, f32, f64, fl, mk = (x.cpu().numpy() for x in (p, s, p2, s2, f32, f64, fl, mk))
    finally:
        c.close()
    pix, psi, tod = (np.concatenate(x) for x in (pix, psi, tod))
    for a, b in ((p, s), (p2, s2)):
        assert np.array_equal(a, pix) and np.array_equal(b.astype(np.int64), psi)
    assert np.array_equal(f64, 0.25 * tod) and np.array_equal(f32, (0.25 * tod).astype(np.float32))
    assert np.array_equal(fl, tod.astype(np.int32)) and np.array_equal(mk, ((tod & 5) == 0).astype(np.uint8))

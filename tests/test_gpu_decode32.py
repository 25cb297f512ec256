"""The decoders of 32-symbol chunks at the edges of what they hold on chip: a
table with more symbols than the block keeps (the rest are read from memory),
symbols wider than 16 bits, a segment whose stream words do not fit the block
although the average does, segments that end inside a wave, a chunk or a block
of 512 chunks, and odd sample offsets (unaligned wide stores).  Bit-exact
against the arrays that were encoded; the error word stays clear."""
import numpy as np
import pytest
import torch

import synth
from synth import huffman_enc as H
from synth.configs import Band
from synth.make import HuffStream

pytestmark = pytest.mark.gpu

LENGTHS = (1, 31, 33, 2047, 2048, 2049, 16383, 16384 + 7, 0, 40000)


def encode(segs, table_of=None):
    """HuffStream of a list of integer arrays (chunks of 32), one table each or
    one for all (table_of: list of table ids)."""
    table_of = list(range(len(segs))) if table_of is None else table_of
    h = HuffStream(32)
    diffs = [H.difference(v) for v in segs]
    tabs = [H.build_table(np.concatenate([d for d, t in zip(diffs, table_of) if t == k] or [np.zeros(0)]))
            for k in range(max(table_of) + 1)]
    words, cb, cp = [], [], []
    for v, d, t in zip(segs, diffs, table_of):
        if len(v):
            w, pos = H.encode_values(d, tabs[t][1])
            b, p = H.chunk_index(v, pos, 32)
        else:
            w, b, p = np.zeros(0), np.zeros(0), np.zeros(0)
        words.append(w)
        cb.append(b)
        cp.append(p)
    off = lambda x: np.concatenate([[0], np.cumsum([len(a) for a in x])]).astype(np.int64)
    h.words, h.seg_word_off = np.concatenate(words).astype(np.uint32), off(words)
    h.tables, h.table_off = np.concatenate([b for b, _ in tabs]).astype(np.uint32), off([b for b, _ in tabs])
    h.chunk_bit, h.chunk_prev = np.concatenate(cb).astype(np.uint32), np.concatenate(cp).astype(np.int32)
    h.seg_chunk_off = off(cb)
    h.seg_table = np.array(table_of, dtype=np.int32)
    return h


def streams(kind, rng, npix):
    """(pix, psi, tod) arrays per segment."""
    pix, psi, tod = [], [], []
    for i, n in enumerate(LENGTHS):
        jump = rng.random(n) < (0.02 if kind == "jumps" else 0.3)
        p = np.cumsum(np.where(jump, rng.integers(-npix, npix, n), 1)) % npix
        s = np.cumsum(rng.integers(-3, 4, n)) % 4096
        t = np.cumsum(np.where(jump, rng.integers(-200000, 200000, n), rng.integers(-9, 10, n)))
        if kind == "one_dense" and i == len(LENGTHS) - 1:  # its words overflow the block's
            p, s, t = rng.integers(0, npix, n), rng.integers(0, 4096, n), rng.integers(-2**28, 2**28, n)
        elif kind == "one_dense":
            p, s, t = np.full(n, 5 + i), np.full(n, 4095), np.full(n, -7)
        pix.append(p), psi.append(s), tod.append(t)
    return pix, psi, tod


@pytest.mark.parametrize("kind", ["jumps", "many_jumps", "one_dense"])
def test_decode32(kind):
    from paper_2201_03509_amd import ops
    rng = np.random.default_rng(3)
    ts = synth.make(1, nscan=len(LENGTHS), length=("list",) + LENGTHS, bands=(Band(1024, 32.5, 1),))
    pix, psi, tod = streams(kind, rng, ts.npix_total)
    one = [0] * len(LENGTHS) if kind != "one_dense" else None  # one table: thousands of symbols
    ts.pix_huff, ts.psi_huff, ts.tod_huff, ts.flag_huff = encode(pix, one), encode(psi), encode(tod, one), encode(tod, one)
    ts.tod_quantum = 0.25
    if kind == "jumps":
        assert ts.pix_huff.tables[0] > 512
    c = ops.Context(0)
    try:
        dt = ops.DeviceTod(ts, "cuda:0")
        e = lambda t: torch.empty(ts.nsamp, dtype=t, device="cuda")
        p, s, f32, f64, fl, mk = e(torch.int32), e(torch.uint16), e(torch.float32), e(torch.float64), e(torch.int32), e(torch.uint8)
        p2, s2 = e(torch.int32), e(torch.uint16)
        c.decode_pointing(dt, p, s)
        c.decode_pointing_noalloc(dt, p2, s2)
        c.decode_tod(dt, "mixed", f32)
        c.decode_tod(dt, "fp64", f64)
        c.decode_flags(dt, 5, fl, mk)
        c.sync()
        p, s, f32, f64, fl, mk, p2, s2 = (x.cpu().numpy() for x in (p, s, f32, f64, fl, mk, p2, s2))
    finally:
        c.close()
    pix, psi, tod = (np.concatenate(x) for x in (pix, psi, tod))
    for a, b in ((p, s), (p2, s2)):
        assert np.array_equal(a, pix) and np.array_equal(b.astype(np.int64), psi)
    assert np.array_equal(f64, 0.25 * tod) and np.array_equal(f32, (0.25 * tod).astype(np.float32))
    assert np.array_equal(fl, tod.astype(np.int32)) and np.array_equal(mk, ((tod & 5) == 0).astype(np.uint8))

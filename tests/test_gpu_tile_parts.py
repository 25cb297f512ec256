"""Strided tiles whole, and cut into even and odd numbers of parts side by side: sets of
20, 600 and 1200 pairs of segments (one tile a pair with stride 1, lengths 1 to 40, so
8 to 40 revisits and last parts of every length; 1200 tiles are not cut, 600 only
where more than a short part is left).  Every sample is projected and binned once:
projection against a gather in 64 bits, 1e-5 and 1e-12; hits exact."""
import numpy as np
import pytest
import torch

from test_gpu_row_launches import layout

pytestmark = pytest.mark.gpu


def template(maps, pix, psi):
    """P m in 64 bits (torch, on the GPU)."""
    a = torch.pi * (2.0 * psi.double() + 1.0) / 2048.0
    m = maps.double()[:, pix.long()]
    return m[0] + m[1] * torch.cos(a) + m[2] * torch.sin(a)


@pytest.mark.parametrize("top", [10, 16, 40])
@pytest.mark.parametrize("pairs", [20, 600, 1200])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_parts_cover_every_sample(prec, pairs, top):
    from paper_2201_03509_amd import ops
    ft, tol = (torch.float32, 1e-5) if prec == "mixed" else (torch.float64, 1e-12)
    lens = np.repeat(np.random.default_rng(pairs + top).integers(1, top + 1, pairs), 2)
    c = ops.Context(0)
    try:
        tod = layout(lens)
        g = torch.Generator("cuda").manual_seed(top)
        pix = torch.randint(0, 12, (tod.nsamp,), device="cuda", generator=g, dtype=torch.int32)
        psi = torch.randint(0, 4096, (tod.nsamp,), device="cuda", generator=g, dtype=torch.int32)
        maps = torch.randn((3, 12), device="cuda", generator=g).to(ft)
        d = torch.randn(tod.nsamp, device="cuda", generator=g).to(ft)
        ref = template(maps, pix, psi)
        for stride in (1, 3):
            c.set_bin_stride(0, stride)
            s = torch.full((tod.nsamp,), float("nan"), dtype=ft, device="cuda")
            c.project_sky(tod, prec, pix, psi.to(torch.uint16), maps, s)
            acc = ops.new_acc(12, "cuda")
            c.bin_tod(tod, prec, pix, psi.to(torch.uint16), d, None, acc)
            c.sync()
            assert torch.linalg.norm(s.double() - ref) <= tol * torch.linalg.norm(ref)
            assert torch.equal(acc[9].long(), torch.bincount(pix, minlength=12))
    finally:
        c.close()

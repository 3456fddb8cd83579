"""The blur of the atlas over bitmap sizes: narrow bitmaps (a wave takes several rows), bands cut evenly
and to the bitmap's height, the band that asks for the most LDS; and small bitmaps cost about as
much per texel as large ones. Against the float64 oracle, with the tolerance of test_gpu_sa_init.py."""
import numpy as np
import pytest
import torch

from oracle import aids as oaids
from paper_2602_22625_amd import aids

pytestmark = pytest.mark.gpu


# (bitmaps, height, width, sigma): widths around the powers of two a wave's rows change at; heights that
# a band does not divide, below, at and above 64 rows; radius 16, 64 columns and 64 rows (60 KB)
@pytest.mark.parametrize("B,Hb,Wb,sigma", [(7, 5, 1, 1.0), (7, 33, 2, 1.0), (5, 65, 7, 1.0), (5, 129, 8, 2.0),
                                           (5, 64, 9, 1.0), (5, 30, 16, 5.3), (5, 31, 17, 1.0),
                                           (3, 100, 32, 1.0), (3, 100, 33, 2.0), (2000, 31, 20, 1.0),
                                           (400, 90, 12, 3.0), (520, 64, 64, 5.4), (300, 127, 64, 5.4)])
def test_sizes(B, Hb, Wb, sigma):
    g = np.random.default_rng(B + Hb + Wb)
    a = g.uniform(0, 1, (B, Hb, Wb)).astype(np.float32)
    out = aids.blur_atlas(torch.tensor(a, device="cuda"), sigma)
    torch.cuda.synchronize()
    assert np.max(np.abs(out.double().cpu().numpy() - oaids.gaussian_blur(a, sigma))) <= 1e-6


def _us(B, S):
    a = torch.rand(B, S, S, device="cuda")
    out = torch.empty_like(a)
    t = []
    for _ in range(15):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(10):
            aids.dbmp_blur_atlas(0, a, B, S, S, 0, 1.0, 3.0, out)
        e[1].record()
        e[1].synchronize()
        t.append(e[0].elapsed_time(e[1]) * 100)
    return min(t)


def test_small_bitmaps_are_fast():
    """3.84 million texels as bitmaps of 8 x 8 and of 64 x 64: 32 and 16 us (221 for 8 x 8 with a row per
    wave, 124 with threads dealt by division). The line is at 4 times."""
    small, large = _us(60000, 8), _us(938, 64)
    print("8 x 8: %.1f us, 64 x 64: %.1f us" % (small, large))
    assert small < 4 * large

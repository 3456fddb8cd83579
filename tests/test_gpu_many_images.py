"""Batches of more images than a wave has lanes: the searches for a tile's and for a primitive's image
narrow by 64 per step, and a workgroup of the binning whose primitives belong to many images finds
each in a few steps. Against the same images in batches of at most 64 (bit for bit), and in time."""
import math

import numpy as np
import pytest
import torch

from paper_2602_22625_amd import synth
from paper_2602_22625_amd.render import Renderer

pytestmark = pytest.mark.gpu


def _batch(n_images, seed, count, size):
    """(descriptors, parameters): image k is up to size(g) x size(g) with count(k) primitives."""
    g = np.random.default_rng(seed)
    descs, po, xo = [], 0, 0
    for k in range(n_images):
        H, W, n = size(g), size(g), count(k)
        descs.append((H, W, n, po, xo))
        po += n
        xo += H * W
    p = np.zeros((po, 8), np.float32)
    p[:, :2] = g.uniform(0, 16, (po, 2))
    p[:, 2], p[:, 3] = np.log(g.uniform(2, 8, po)), g.uniform(0, 6.28, po)
    p[:, 4], p[:, 5:] = g.normal(-1, 1, po), g.normal(0, 1, (po, 3))
    return descs, torch.tensor(p, device="cuda")


# around one and two steps of the search (64, 64^2 images) and past the second; one primitive per
# image (every workgroup of the binning meets many images), a few, long gaps of empty images (also
# before the first and after the last primitive), and 64 primitives per workgroup of the binning
@pytest.mark.parametrize("n_images,count", [
    (65, lambda k: 1), (127, lambda k: k % 3), (128, lambda k: 1), (129, lambda k: 1),
    (4095, lambda k: 1), (4096, lambda k: k % 2), (4097, lambda k: 1), (4160, lambda k: 1),
    (5000, lambda k: 3 * (k % 700 == 350)), (9000, lambda k: 2)])
def test_equals_small_batches(n_images, count):
    descs, P = _batch(n_images, n_images, count, lambda g: int(g.integers(1, 20)))
    atlas = torch.tensor(synth.soft_disk(16)[None], device="cuda")
    idx = torch.zeros(P.shape[0], dtype=torch.int32, device="cuda")
    bg = torch.rand(n_images, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    Rb, Rs = Renderer(), Renderer()
    img, alp = Rb.render_batched(descs, P, idx, atlas, bg, 1.0, 16)
    for k0 in range(0, n_images, 64):
        part = descs[k0:k0 + 64]
        p0, x0 = part[0][3], part[0][4]
        p1, x1 = part[-1][3] + part[-1][2], part[-1][4] + part[-1][0] * part[-1][1]
        if p1 == p0:  # (a render reads at least one row)
            assert torch.equal(alp[x0:x1], torch.zeros_like(alp[x0:x1])), k0
            continue
        i1, a1 = Rs.render_batched([(h, w, n, p - p0, x - x0) for h, w, n, p, x in part],
                                   P[p0:p1].contiguous(), idx[:p1 - p0].contiguous(), atlas,
                                   bg[k0:k0 + 64].contiguous(), 1.0, 16)
        assert torch.equal(img[3 * x0:3 * x1], i1), k0
        assert torch.equal(alp[x0:x1], a1), k0


def _graph_us(descs, P, atlas, calls=5):
    n = len(descs)
    idx = torch.zeros(P.shape[0], dtype=torch.int32, device="cuda")
    bg = torch.ones(n, 3, device="cuda")
    img = torch.empty(3 * (descs[-1][4] + descs[-1][0] * descs[-1][1]), device="cuda")
    R = Renderer(check=False)
    R.set_atlas(atlas)

    def call():
        R.render_batched(descs, P, idx, None, bg, 1.0, 8, image=img, with_alpha=False)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        call()
    torch.cuda.current_stream().wait_stream(s)
    R.check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(calls):
            call()
    t = []
    for _ in range(7):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3 / calls)
    return min(t)


def test_image_count_costs_little():
    """16,384 images of one tile and one primitive against the same number of tiles and primitives in
    64 images: the searches are the difference. 35 us each; 383 with a search through all images 64 at
    a time. The line is at 8 times."""
    g = np.random.default_rng(0)
    P = np.zeros((16384, 8), np.float32)
    P[:, :2], P[:, 2] = g.uniform(0, 8, (16384, 2)), math.log(3.0)
    P = torch.tensor(P, device="cuda")
    atlas = torch.tensor(synth.soft_disk(16)[None], device="cuda")
    many = _graph_us([(8, 8, 1, k, 64 * k) for k in range(16384)], P, atlas)
    P[:, :2] *= 16
    few = _graph_us([(128, 128, 256, 256 * k, 16384 * k) for k in range(64)], P, atlas)
    print("16,384 images %.1f us, 64 images %.1f us" % (many, few))
    assert many < 8 * few

"""Edges of the binning and of the rasteriser's list sort: images searched 64 at a time, lists
around the one-wave sort's 64 entries, Adam's bias corrections at any step count."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_22625_amd import capi, synth
from paper_2602_22625_amd.render import Renderer

pytestmark = pytest.mark.gpu


def _scene(n, H, W, seed, lo=4.0, hi=10.0):
    g = np.random.default_rng(seed)
    p = np.zeros((n, 8), dtype=np.float32)
    p[:, 0], p[:, 1] = g.uniform(0, W, n), g.uniform(0, H, n)
    p[:, 2], p[:, 3] = np.log(g.uniform(lo, hi, n)), g.uniform(0, 6.28, n)
    p[:, 4], p[:, 5:] = g.normal(-2, 1, n), g.normal(0, 1, (n, 3))
    return p


# one image (no search), one wave's worth and around it, more than two
@pytest.mark.parametrize("n_images", [1, 2, 63, 64, 65, 130])
def test_image_search(n_images):
    """Every image of a batch of small ones (some empty, gaps between primitive ranges, the first
    range not at 0; many share a workgroup of the binning) is bitwise its own render."""
    g = np.random.default_rng(n_images)
    atlas = torch.tensor(synth.soft_disk(16)[None], device="cuda")
    descs, ps, po, xo = [], [], 0, 0
    for k in range(n_images):
        gap = 5 if k == 0 else int(g.integers(0, 3))
        ps.append(np.zeros((gap, 8), np.float32))
        po += gap
        H, W, n = int(g.integers(1, 40)), int(g.integers(1, 40)), int(g.integers(0, 12))
        if k == n_images - 1:
            n += 70  # the last image spans workgroups
        descs.append((H, W, n, po, xo))
        ps.append(_scene(n, H, W, 1000 * n_images + k))
        po += n
        xo += H * W
    P = torch.tensor(np.concatenate(ps), device="cuda")
    idx = torch.zeros(P.shape[0], dtype=torch.int32, device="cuda")
    bg = torch.rand(n_images, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    Rb, Rs = Renderer(), Renderer()
    img, alp = Rb.render_batched(descs, P, idx, atlas, bg, 1.0, 16)
    Rb.check()
    for k, (H, W, n, p0, x0) in enumerate(descs):
        i1, a1 = Rs.render(P[p0:p0 + n].contiguous(), idx[:n].contiguous(), atlas, H, W,
                           bg[k].contiguous(), 1.0, 16)
        Rs.check()
        assert torch.equal(img[3 * x0:3 * (x0 + H * W)], i1.reshape(-1)), k
        assert torch.equal(alp[x0:x0 + H * W], a1.reshape(-1)), k


# around a list's smallest capacity (32), a wave, and the capacities that follow
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 96])
def test_short_lists(n, tile):
    """One tile whose list has n entries, at the smallest capacity that holds them: the pipelined
    build alone, the one-cell build beside a 1024 x 1024 canvas, both against float64."""
    p = _scene(n, tile, tile, 7 * n + tile, 2.0 * tile, 3.0 * tile)  # boxes over the whole tile
    atlas = synth.soft_disk(16)[None].astype(np.float32)
    ref, _ = oracle.render(p, np.zeros(n, np.int32), atlas, tile, tile)
    P, A = torch.tensor(p, device="cuda"), torch.tensor(atlas, device="cuda")
    idx = torch.zeros(n, dtype=torch.int32, device="cuda")
    bg = torch.ones(2, 3, device="cuda")
    R1, R2 = Renderer(list_capacity=n), Renderer(list_capacity=n)
    i1, _ = R1.render(P, idx, A, tile, tile, bg[0].contiguous(), 1.0, tile)
    R1.check()
    assert R1.longest_list() == n
    descs = [(tile, tile, n, 0, 0), (1024, 1024, 0, n, tile * tile)]
    i2, _ = R2.render_batched(descs, P, idx, A, bg, 1.0, tile)
    R2.check()
    assert torch.equal(i1.reshape(-1), i2[:3 * tile * tile])
    err = np.abs(i1.double().cpu().numpy() - ref).max() / max(np.abs(ref).max(), 1e-12)
    assert err <= 1e-5


@pytest.mark.parametrize("t", [1, 2, 1000, 123456, 2 ** 30])
def test_adam_bias_corrections(t):
    """The corrections 1 - beta^t at small, ordinary and very large t: parameters against float64
    with the kernel's own float32 moments, so that a handful of float32 roundings remain."""
    g = np.random.default_rng(t % 1000)
    n = 257
    p, gr = g.normal(size=n).astype(np.float32), g.normal(size=n).astype(np.float32)
    m, v = (0.1 * g.normal(size=n)).astype(np.float32), g.uniform(0, 1, n).astype(np.float32)
    d = [torch.tensor(x, device="cuda") for x in (p, gr, m, v)]
    step = torch.tensor([t - 1, 0], dtype=torch.int32, device="cuda")
    capi.dbmp_adam_step(capi.stream_handle(), *d, n, 1e-2, 0.9, 0.999, 1e-8, step, zero_grad=0)
    torch.cuda.synchronize()
    assert step.tolist() == [t, 0]
    m1, v1 = d[2].double().cpu().numpy(), d[3].double().cpu().numpy()
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    upd = float(np.float32(1e-2)) * (m1 / (1 - b1 ** t)) / (np.sqrt(v1 / (1 - b2 ** t)) + 1e-8)
    # corrections, two quotients, root, sum, product and quotient: under 16 roundings of 2^-24
    err = np.abs(d[0].double().cpu().numpy() - (p - upd))
    assert np.all(err <= 2.0 ** -20 * np.abs(upd) + 2.0 ** -24 * np.maximum(np.abs(p), np.abs(p - upd)))

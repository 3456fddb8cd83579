"""The structure-aware initialisation and the blur at the edges of their tiles, windows and strips:
single pixels and rows, odd sizes around a strip and a 128-column tile, every window size, both
strip heights. Against the float64 oracle, with the
tolerances of test_gpu_aids.py."""
import numpy as np
import pytest
import torch

from oracle import aids as oaids
from paper_2602_22625_amd import aids

pytestmark = pytest.mark.gpu


def _check(t, win, N, seed, base=0.1):
    _, H, W = t.shape
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    d = torch.tensor(t, device="cuda")
    params, nlv, (u, ut, z) = aids.sa_init(d, N, 2.0, 20.0, win=win, base=base, generator=g)
    torch.cuda.synchronize()
    got_nlv = nlv.double().cpu().numpy()
    assert np.max(np.abs(got_nlv - oaids.nlv(oaids.local_variance(t, win)))) <= 1e-6
    ref = oaids.sa_init(got_nlv, t, u.cpu().numpy(), ut.cpu().numpy(), z.cpu().numpy(), 2.0, 20.0,
                        base=base)
    got = params.double().cpu().numpy()
    assert np.array_equal(got[:, :2], ref[:, :2])
    assert np.max(np.abs(got[:, 2:] - ref[:, 2:]) / np.maximum(np.abs(ref[:, 2:]), 1.0)) <= 1e-6


@pytest.mark.parametrize("H,W,win", [(1, 1, 7), (1, 300, 7), (130, 1, 5), (16, 128, 7), (17, 129, 7),
                                     (5, 127, 15), (65, 131, 1), (65, 131, 3), (33, 260, 9),
                                     (40, 70, 11), (40, 70, 13), (67, 140, 15)])
def test_sa_init_edges(H, W, win):
    g = np.random.default_rng(H * 1000 + W + win)
    _check(g.uniform(0, 1, (3, H, W)).astype(np.float32), win, 257, H + W)


@pytest.mark.parametrize("win", [3, 7, 15])
def test_nlv_of_a_large_target(win):
    """The taller strips (at least 512 workgroups), a last strip and column tile partly empty. The
    reference sums shifted float64 planes (two-pass variance)."""
    H, W, h = 2041, 2043, win // 2
    g = torch.Generator(device="cuda")
    g.manual_seed(win)
    t = torch.rand(3, H, W, generator=g, device="cuda")
    _, nlv, _ = aids.sa_init(t, 16, 2.0, 20.0, win=win)
    d = torch.nn.functional.pad(t.double(), (h, h, h, h))
    n = torch.nn.functional.pad(torch.ones(1, H, W, device="cuda", dtype=torch.float64), (h, h, h, h))
    shifts = [(slice(i, i + H), slice(j, j + W)) for i in range(win) for j in range(win)]
    cnt = sum(n[:, a, b] for a, b in shifts)
    mean = sum(d[:, a, b] for a, b in shifts) / cnt
    lv = (sum(n[:, a, b] * (d[:, a, b] - mean) ** 2 for a, b in shifts) / cnt).mean(0)
    ref = (lv - lv.min()) / (lv.max() - lv.min())
    assert float((nlv.double() - ref).abs().max()) <= 1e-6


@pytest.mark.parametrize("value", [0.5, 0.3, 1.0])
def test_flat_target_has_zero_nlv(value):
    t = torch.full((3, 70, 200), value, device="cuda")
    _, nlv, _ = aids.sa_init(t, 64, 2.0, 20.0)
    torch.cuda.synchronize()
    assert float(nlv.abs().max()) == 0.0


@pytest.mark.parametrize("B,Hb,Wb,sigma", [(1, 1, 1, 1.0), (1, 9, 65, 1.0), (3, 8, 64, 2.2),
                                           (2, 70, 33, 5.0), (600, 17, 20, 1.0), (1, 5, 1024, 0.5)])
def test_blur_edges(B, Hb, Wb, sigma):
    g = np.random.default_rng(B + Hb + Wb)
    a = g.uniform(0, 1, (B, Hb, Wb)).astype(np.float32)
    out = aids.blur_atlas(torch.tensor(a, device="cuda"), sigma)
    torch.cuda.synchronize()
    assert np.max(np.abs(out.double().cpu().numpy() - oaids.gaussian_blur(a, sigma))) <= 1e-6

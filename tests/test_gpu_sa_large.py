"""The start of a fit on large targets: every window size with the taller strips of the local variance, and
a target of more blocks than the sampler scans itself and more extremes than a workgroup reads, whose
draws must equal exact integer sums."""
import numpy as np
import pytest
import torch

from paper_2602_22625_amd import aids

pytestmark = pytest.mark.gpu


# (3, 7 and 15 are in test_gpu_sa_init.py); the reference sums shifted float64 planes (two passes)
@pytest.mark.parametrize("win", [1, 5, 9, 11, 13])
def test_windows(win):
    H, W, h = 1030, 1085, win // 2  # 17 x 33 workgroups: at least 512, the last of each partly empty
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
    span = lv.max() - lv.min()
    ref = (lv - lv.min()) / span if span > 0 else torch.zeros_like(lv)
    assert float((nlv.double() - ref).abs().max()) <= 1e-6


@pytest.mark.parametrize("base", [0.0, 0.1])
def test_draws_from_nine_million_pixels(base):
    H, W, N = 3001, 2999, 5000
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    t = torch.rand(3, H, W, generator=g, device="cuda")
    t[:, :900] = 0.25  # a flat part
    params, nlv, (u, _, _) = aids.sa_init(t, N, 2.0, 20.0, base=base, generator=g)
    nf = nlv.cpu().numpy().reshape(-1).astype(np.float64)
    assert nf.min() == 0.0 and nf.max() == 1.0
    cdf = np.cumsum(np.floor((base + (1.0 - base) * nf) * 16777216.0).astype(np.int64))
    k = np.floor(u.cpu().numpy().astype(np.float64) * float(cdf[-1])).astype(np.int64)
    p = np.searchsorted(cdf, np.minimum(k, cdf[-1] - 1), side="right")
    got = params[:, :2].cpu().numpy()
    assert np.array_equal(got[:, 0], (p % W).astype(np.float32))
    assert np.array_equal(got[:, 1], (p // W).astype(np.float32))

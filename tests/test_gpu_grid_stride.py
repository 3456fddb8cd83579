"""Kernels that stride a bounded grid over their values, four at a time where the buffers allow:
counts around the vector width, the workgroup and the whole grid, and buffers off 16-byte
alignment (which take the one-value form), against float64."""
import numpy as np
import pytest
import torch

from paper_2602_22625_amd import aids, capi

pytestmark = pytest.mark.gpu


def _buf(a, off):
    """A device float32 copy of `a` that starts `off` values past a 16-byte boundary."""
    b = torch.zeros(a.size + off, device="cuda")
    b[off:] = torch.tensor(a.reshape(-1), device="cuda")
    return b[off:]


# one thread's share, a remainder, one workgroup, the whole grid (256 x 1,024 x 4) and past it
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 4, 1027, 4096, 256 * 4096 + 5])
def test_adam_step(n, off):
    g = np.random.default_rng(n + off)
    p, gr = g.normal(size=n).astype(np.float32), g.normal(size=n).astype(np.float32)
    m, v = (0.1 * g.normal(size=n)).astype(np.float32), g.uniform(0, 1, n).astype(np.float32)
    bufs = [_buf(x, off) for x in (p, gr, m, v)]
    step = torch.tensor([4, 0], dtype=torch.int32, device="cuda")
    capi.dbmp_adam_step(capi.stream_handle(), *bufs, n, 1e-2, 0.9, 0.999, 1e-8, step, zero_grad=1)
    torch.cuda.synchronize()
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    m64 = b1 * m.astype(np.float64) + (1 - b1) * gr
    v64 = b2 * v.astype(np.float64) + (1 - b2) * gr.astype(np.float64) ** 2
    upd = 1e-2 * (m64 / (1 - b1 ** 5)) / (np.sqrt(v64 / (1 - b2 ** 5)) + 1e-8)
    got = [b.double().cpu().numpy() for b in bufs]
    assert step.tolist() == [5, 0]
    assert np.all(got[1] == 0)
    # float32: 1 - beta2 is 1e-3 off one float32 ulp of 1 (6e-5 relative), which v and the root carry
    assert np.max(np.abs(got[2] - m64)) <= 1e-6
    assert np.max(np.abs(got[3] - v64) / (v64 + 1e-3)) <= 1e-4
    assert np.max(np.abs(got[0] - (p - upd))) <= 1e-4 * np.max(np.abs(upd)) + 2.0 ** -22


# both forms (planes of a multiple of 4 pixels or not, aligned or not) and more than the grid
# takes at once (256 workgroups of 256 threads)
@pytest.mark.parametrize("H,W,off", [(1, 1, 0), (3, 5, 0), (4, 7, 0), (4, 7, 1), (601, 880, 0),
                                     (601, 881, 0)])
def test_constraint_loss(H, W, off):
    g = np.random.default_rng(H * W + off)
    I, t = g.uniform(0, 1, (3, H, W)).astype(np.float32), g.uniform(0, 1, (3, H, W)).astype(np.float32)
    A = g.uniform(0, 1, (H, W)).astype(np.float32)
    ta = np.maximum(g.uniform(-1, 1, (H, W)), 0).astype(np.float32)
    d = [_buf(x, off) for x in (I, A, t, ta)]
    gI, gA = _buf(np.full(I.size, 9, np.float32), off), _buf(np.full(A.size, 9, np.float32), off)
    loss = torch.tensor([0.5], device="cuda")
    aids.dbmp_constraint_loss(capi.stream_handle(), d[0], d[1], d[2], d[3], H, W, 0.7, gI, gA, loss)
    torch.cuda.synchronize()
    D = (I.astype(np.float64) - t) * (ta > 0)
    E = A.astype(np.float64) - ta
    L = 0.5 + np.mean(D * D) + 0.7 * np.mean(E * E)
    # one subtraction, two or three roundings per value; the sum's rounding grows with its depth
    assert np.max(np.abs(gI.double().cpu().numpy().reshape(I.shape) - 2 * D / D.size)) <= 3e-7 / D.size
    assert np.max(np.abs(gA.double().cpu().numpy().reshape(A.shape) - 1.4 * E / E.size)) <= 4e-7 / E.size
    assert abs(float(loss) - L) <= 1e-5


@pytest.mark.parametrize("n", [8, 2056, 256 * 256 * 3 + 64])
def test_param_loss(n):
    g = np.random.default_rng(n)
    pred, tgt = g.normal(size=n).astype(np.float32), g.normal(size=n).astype(np.float32)
    ex = g.normal(size=n).astype(np.float32)
    w = np.array([1, 1, 1, 0.1, 1, 2, 1, 1], np.float32)
    xs = [0.5, 1, 2, 3, 4, 5, 6, 7]
    dp = torch.empty(n, device="cuda", dtype=torch.bfloat16)
    loss = torch.zeros(1, device="cuda")
    c = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    capi.dbmp_cnn_param_loss(capi.stream_handle(), c(pred), c(tgt), c(w), n, 1.0 / n, dp, loss,
                             c(ex), xs)
    torch.cuda.synchronize()
    d = pred.astype(np.float64) - tgt
    q = np.arange(n) % 8
    wq = w.astype(np.float64)[q]
    L = np.where(q == 3, wq * (1 - np.cos(d)), wq * d * d).sum() / n
    G = np.where(q == 3, wq * np.sin(d), 2 * wq * d) / n + ex * np.array(xs)[q]
    got = dp.double().cpu().numpy()
    assert abs(float(loss) - L) <= 1e-5 * (1 + L)
    assert np.max(np.abs(got - G) - 2.0 ** -8 * np.abs(G)) <= 1e-6   # one bf16 rounding

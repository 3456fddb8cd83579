"""Bias gradients as column sums (the layers that the matrix kernels have no build for): exact on dyadic
inputs at the edges of the rows dealt to a workgroup, and no slower for few columns or many rows than
a split into 2,048 rows was."""
import numpy as np
import pytest
import torch

from paper_2602_22625_amd import capi

pytestmark = pytest.mark.gpu


# (rows, columns): one row, around a workgroup's 2,048 rows and its passes, few and many columns, a row
# count that the number of workgroups does not divide, and above 200 MB (twice the workgroups)
@pytest.mark.parametrize("M,N", [(1, 8), (2047, 8), (2049, 16), (6000, 24), (127, 520), (129, 520),
                                 (65537, 40), (600011, 16), (210001, 488)])
def test_exact(M, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    dz = (torch.randint(-2, 3, (M, N), generator=g, device="cuda") / 4).to(torch.bfloat16)
    x = torch.zeros(M, 8, device="cuda", dtype=torch.bfloat16)
    dw, db = torch.zeros(N, 8, device="cuda"), torch.full((N,), 0.5, device="cuda")
    capi.dbmp_cnn_linear_backward_weight(capi.stream_handle(), x, dz, M, 8, N, dw, db)
    want = torch.zeros(N, device="cuda", dtype=torch.float64)
    for k in range(0, M, 1 << 16):
        want += dz[k:k + (1 << 16)].double().sum(0)
    assert float(want.abs().max()) < 2 ** 22  # quarters: exact in float32
    assert torch.equal(db.double(), want + 0.5)


def _us(M, N):
    """Time of the sums: the layer with its bias less the layer without, in graphs of 20."""
    dz = torch.randn(M, N, device="cuda").to(torch.bfloat16)
    x = torch.zeros(M, 8, device="cuda", dtype=torch.bfloat16)
    dw, db = torch.zeros(N, 8, device="cuda"), torch.zeros(N, device="cuda")
    t = []
    for b in (db, None):
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            capi.dbmp_cnn_linear_backward_weight(capi.stream_handle(), x, dz, M, 8, N, dw, b)
        torch.cuda.current_stream().wait_stream(s)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                capi.dbmp_cnn_linear_backward_weight(capi.stream_handle(), x, dz, M, 8, N, dw, b)
        v = []
        for _ in range(15):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            g.replay()
            e[1].record()
            e[1].synchronize()
            v.append(e[0].elapsed_time(e[1]) * 50)
        t.append(float(np.median(v)))
    return t[0] - t[1]


def test_many_rows_are_read_fast():
    """1,048,576 x 264 (554 MB) against a copy of them, which reads and writes as much: 90 us of about 210, 129
    with a workgroup per compute unit. The line is at half."""
    us = _us(1 << 20, 264)
    a = torch.empty(1 << 20, 264, device="cuda", dtype=torch.bfloat16)
    b = torch.empty_like(a)
    t = []
    for _ in range(15):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(5):
            b.copy_(a)
        e[1].record()
        e[1].synchronize()
        t.append(e[0].elapsed_time(e[1]) * 200)
    print("sums %.1f us, copy %.1f us" % (us, min(t)))
    assert us < 0.5 * min(t)

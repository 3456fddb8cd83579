"""The layer export where its forms meet: bitmaps of odd and smallest sizes, each texel type, boxes on
both sides of the rule that copies a bitmap to LDS, bitmaps too large for it, boxes of one row or
column, and counts around the offset scan's pass of 8,192 primitives."""
import math

import numpy as np
import pytest
import torch

from paper_2602_22625_amd import aids, synth
from test_gpu_export import _check_layers

pytestmark = pytest.mark.gpu


# (Hb, Wb, dtype, half-extent): 130 x 131 float32 does not fit the LDS copy; half-extents around
# sqrt(Hb Wb / 2) / 2 give boxes on both sides of half as many values as texels
@pytest.mark.parametrize("Hb,Wb,dtype,s", [(2, 2, "f32", 5.0), (2, 37, "f32", 9.0), (31, 2, "f16", 6.0),
                                           (33, 63, "f32", 14.0), (33, 63, "bf16", 14.0),
                                           (64, 65, "f16", 22.0), (64, 64, "f32", 2.0),
                                           (130, 131, "f32", 30.0), (130, 131, "bf16", 45.0)])
def test_bitmap_shapes(Hb, Wb, dtype, s):
    g = np.random.default_rng(Hb * 1000 + Wb)
    td = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    a = torch.tensor(g.uniform(0, 1, (3, Hb, Wb)).astype(np.float32)).to(td)
    H, W, N = 61, 83, 40
    params, idx = synth.init_params(N, H, W, math.log(s), 0.3, 3, Hb + Wb)
    params[0, :2] = (0.4, -s - 0.2)          # reaches the canvas by a row or not at all
    params[1, :2] = (W - 1.0 + s, H / 2.0)
    out = aids.export_layers(torch.tensor(params, device="cuda"), torch.tensor(idx, device="cuda"),
                             a.cuda(), H, W, 1.5, 0.9)
    torch.cuda.synchronize()
    _check_layers(params.astype(np.float64), idx, a.double().numpy(), H, W, 1.5, *out, 0.9)


@pytest.mark.parametrize("N", [1, 7, 8191, 8193, 20000])
def test_offsets_scan(N):
    g = np.random.default_rng(N)
    params, idx = synth.init_params(N, 300, 200, math.log(4.0), 0.5, 1, N)
    a = torch.tensor(g.uniform(0.1, 1, (1, 8, 8)).astype(np.float32), device="cuda")
    boxes, offsets, alpha, _ = aids.export_layers(torch.tensor(params, device="cuda"),
                                                  torch.tensor(idx, device="cuda"), a, 300, 200, 1.0)
    torch.cuda.synchronize()
    b = boxes.cpu().numpy().astype(np.int64)
    want = np.concatenate([[0], np.cumsum(b[:, 2] * b[:, 3])])
    assert np.array_equal(offsets.cpu().numpy(), want)
    assert alpha.numel() == max(want[-1], 0)

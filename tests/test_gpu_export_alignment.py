"""The layer export with boxes at a 4-byte address, as an int32 array may lie: the kernels that move a box
as one 16-byte access do not ask for more."""
import math

import pytest
import torch

from paper_2602_22625_amd import aids, capi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [50, 20000])  # a workgroup per primitive, several primitives each
@pytest.mark.parametrize("off", [1, 2, 3])
def test_boxes_at_any_word(N, off):
    H, W = 130, 170
    params, idx = synth.init_params(N, H, W, math.log(5.0), 0.5, 3, N)
    P, I = torch.tensor(params, device="cuda"), torch.tensor(idx, device="cuda")
    a = torch.rand(3, 20, 20, device="cuda")
    boxes, offsets, alpha, colours = aids.export_layers(P, I, a, H, W, 1.0)
    words = torch.full((4 * N + 8,), -7, dtype=torch.int32, device="cuda")
    moved = words[off:off + 4 * N]
    assert moved.data_ptr() % 16 == 4 * off
    offs = torch.empty(N + 1, dtype=torch.int64, device="cuda")
    wh = torch.empty(2, dtype=torch.int32, device="cuda")
    st = capi.stream_handle()
    aids.dbmp_export_boxes(st, P, N, 20, 20, H, W, 1.0, moved, offs, wh)
    alpha2, colours2 = torch.empty_like(alpha), torch.empty_like(colours)
    mw, mh = (int(v) for v in wh.cpu())
    aids.dbmp_export_layers(st, P, I, N, a, 3, 20, 20, aids._atlas_code(a), H, W, 1.0, 1.0, moved, offs,
                            mw, mh, alpha2, colours2)
    assert torch.equal(moved.view(N, 4), boxes) and torch.equal(offs, offsets)
    assert torch.equal(alpha2, alpha) and torch.equal(colours2, colours)
    assert (words[:off] == -7).all() and (words[off + 4 * N:] == -7).all()

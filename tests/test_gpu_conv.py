"""The direct convolution kernels at the edges of their tiles and dispatch: pixel counts that leave
a tile partly empty, one output row or column (every tap at a border), channel counts on each side
of the wave tile's rules, batches that select each wave tile. Dyadic inputs as in test_gpu_cnn.py:
every sum is exact in float32, so results must equal the float64 layer oracle (bf16 outputs: its
value rounded to nearest even)."""
import numpy as np
import pytest
import torch

from oracle import cnn_oracle as co
from paper_2602_22625_amd import capi, synth

pytestmark = pytest.mark.gpu


def dyadic(g, shape, num, den):
    return (g.integers(-num, num + 1, size=shape) / den).astype(np.float32)


def bf(a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda").to(torch.bfloat16)


def bf16_round(a):
    return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.asarray(a, np.float32)))


# (B, H, W, Cin, Cout): borders only; odd pixel counts; Cout of one, two, three and four fragments
SHAPES = [(1, 2, 2, 8, 16), (3, 6, 10, 8, 32), (1, 2, 2, 32, 64), (1, 2, 18, 64, 32),
          (5, 6, 14, 32, 48), (2, 10, 22, 128, 64), (1, 6, 6, 256, 16), (2, 4, 4, 256, 256)]


@pytest.mark.parametrize("shape", SHAPES)
def test_forward_and_input_gradient_exact(shape):
    B, H, W, Ci, Co = shape
    g = np.random.default_rng(sum(shape))
    st = capi.stream_handle()
    x, w, b = dyadic(g, (B, H, W, Ci), 4, 4), dyadic(g, (Co, 3, 3, Ci), 4, 8), dyadic(g, (Co,), 8, 16)
    ref = co.conv_forward(x, w, b)
    for relu in (0, 1):
        r = np.maximum(ref, 0) if relu else ref
        y = torch.empty(B, H // 2, W // 2, Co, device="cuda", dtype=torch.bfloat16)
        y32 = torch.empty(B, H // 2, W // 2, Co, device="cuda")
        capi.dbmp_cnn_conv_forward(st, bf(x), B, H, W, Ci, bf(w), torch.tensor(b, device="cuda"), Co,
                                   relu, y, y32)
        torch.cuda.synchronize()
        assert np.array_equal(y32.cpu().numpy(), r.astype(np.float32))
        assert np.array_equal(y.float().cpu().numpy(), bf16_round(r))
    if Ci < 16:
        return
    dz, mask = dyadic(g, (B, H // 2, W // 2, Co), 4, 16), dyadic(g, (B, H, W, Ci), 2, 2)
    wt = torch.empty(Ci, 3, 3, Co, device="cuda", dtype=torch.bfloat16)
    capi.dbmp_cnn_cast_weights(st, torch.tensor(w, device="cuda"), Co, 9, Ci, None, wt)
    dx = torch.empty(B, H, W, Ci, device="cuda", dtype=torch.bfloat16)
    for m in (None, mask):
        capi.dbmp_cnn_conv_backward_data(st, bf(dz), B, H, W, Ci, wt, Co,
                                         None if m is None else bf(m), dx)
        torch.cuda.synchronize()
        want = bf16_round(co.conv_backward_data(dz, w, H, W, mask=m))
        assert np.array_equal(dx.float().cpu().numpy(), want)


# (B, H, W, Cin, Cout): output rows of 8 k and of 4 pixels, pixel counts that leave the last 32-pixel
# step partly empty, one step, several pixel splits, each channel tile; the last two take the general
# product (an output row of 9 pixels, 24 channels)
WSHAPES = [(1, 2, 16, 8, 32), (3, 6, 16, 8, 64), (1, 2, 16, 32, 64), (3, 10, 8, 32, 32),
           (5, 6, 24, 64, 96), (2, 16, 8, 128, 64), (1, 8, 8, 256, 256), (4, 64, 64, 32, 64),
           (4, 64, 64, 8, 32), (1, 4, 18, 32, 64), (1, 4, 16, 32, 24)]


@pytest.mark.parametrize("shape", WSHAPES)
def test_weight_and_bias_gradient_exact(shape):
    B, H, W, Ci, Co = shape
    g = np.random.default_rng(sum(shape))
    x, dz = dyadic(g, (B, H, W, Ci), 4, 4), dyadic(g, (B, H // 2, W // 2, Co), 4, 16)
    rw, rb = co.conv_backward_weight(x, dz)
    for with_bias in (True, False):
        dw = torch.full((Co, 3, 3, Ci), 0.5, device="cuda")
        db = torch.full((Co,), -0.25, device="cuda") if with_bias else None
        capi.dbmp_cnn_conv_backward_weight(capi.stream_handle(), bf(x), bf(dz), B, H, W, Ci, Co, dw,
                                           db)
        torch.cuda.synchronize()
        assert np.array_equal(dw.cpu().numpy(), (rw + 0.5).astype(np.float32))
        if with_bias:
            assert np.array_equal(db.cpu().numpy(), (rb - 0.25).astype(np.float32))


@pytest.mark.parametrize("B,S,Ci,Co", [(70, 32, 32, 64), (33, 32, 32, 64), (9, 64, 64, 32)])
def test_wave_tiles_agree(B, S, Ci, Co):
    """Batches that take the larger wave tiles equal the same images one at a time (the smallest
    tile), bit for bit: the K order does not depend on the tile."""
    g = torch.Generator(device="cuda")
    g.manual_seed(B)
    st = capi.stream_handle()
    r = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    x, w, wt, dz = r(B, S, S, Ci), r(Co, 9, Ci), r(Ci, 9, Co), r(B, S // 2, S // 2, Co)
    bias = torch.randn(Co, generator=g, device="cuda")
    y, dx = torch.empty_like(dz), torch.empty_like(x)
    capi.dbmp_cnn_conv_forward(st, x, B, S, S, Ci, w, bias, Co, 1, y)
    capi.dbmp_cnn_conv_backward_data(st, dz, B, S, S, Ci, wt, Co, x, dx)
    y1, dx1 = torch.empty_like(y), torch.empty_like(dx)
    for i in range(B):
        capi.dbmp_cnn_conv_forward(st, x[i], 1, S, S, Ci, w, bias, Co, 1, y1[i])
        capi.dbmp_cnn_conv_backward_data(st, dz[i], 1, S, S, Ci, wt, Co, x[i], dx1[i])
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y1.view(torch.int16))
    assert torch.equal(dx.view(torch.int16), dx1.view(torch.int16))

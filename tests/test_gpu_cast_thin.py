"""Weight copies of thin layers (few rows or few channels), which are taken value by value: on both sides
of the rule, alone and beside layers taken in tiles, and in time."""
import numpy as np
import pytest
import torch

from paper_2602_22625_amd import capi, synth

pytestmark = pytest.mark.gpu


def _round(a):
    return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))


# (R, T, C): an eighth of a 64 x 64 tile in use is 512 values (8 x 64), a quarter 1,024 (16 x 64); above and
# up to 65,536 values; a last workgroup of one value
@pytest.mark.parametrize("shapes", [[(1, 1, 1)], [(257, 1, 1)], [(1, 700, 1)], [(7, 3, 2000)], [(8, 3, 2000)],
                                    [(3000, 9, 7)], [(3000, 9, 8)], [(15, 1, 4000)], [(16, 1, 4000)],
                                    [(5000, 1, 12)], [(5000, 2, 12)],
                                    [(3, 5, 100), (64, 9, 32), (1, 1, 9), (128, 1, 256), (32, 9, 8)]])
@pytest.mark.parametrize("off", [0, 1])
def test_copies(shapes, off):
    g = np.random.default_rng(len(shapes) + shapes[0][0])
    layers, want = [], []
    for R, T, C in shapes:
        w = g.standard_normal((R, T, C)).astype(np.float32)
        d = torch.zeros(w.size + off, device="cuda")
        d[off:] = torch.tensor(w.reshape(-1), device="cuda")
        wb, wt = (torch.zeros(w.size + 8, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        layers.append((d[off:], R, T, C, wb[off:], wt[off:]))
        want.append(_round(w))
    capi.dbmp_cnn_cast_layers(capi.stream_handle(), layers)
    torch.cuda.synchronize()
    for k, ((d, R, T, C, wb, wt), r) in enumerate(zip(layers, want)):
        n = R * T * C
        assert np.array_equal(wb[:n].float().cpu().numpy(), r.reshape(-1)), k
        assert np.array_equal(wt[:n].float().cpu().numpy(), r.transpose(2, 1, 0).reshape(-1)), k
        assert not wb[n:].any() and not wt[n:].any()
        one = torch.zeros_like(wt)
        capi.dbmp_cnn_cast_weights(capi.stream_handle(), d, R, T, C, None, one)
        assert torch.equal(one, wt), k


def _us(R, T, C):
    w = torch.rand(R, T, C, device="cuda")
    wb, wt = (torch.empty(R * T * C, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    t = []
    for _ in range(15):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(10):
            capi.dbmp_cnn_cast_weights(0, w, R, T, C, wb, wt)
        e[1].record()
        e[1].synchronize()
        t.append(e[0].elapsed_time(e[1]) * 100)
    return min(t)


def test_thin_layers_are_fast():
    """300,000 weights as 1 x 300,000 x 1 and as 550 x 1 x 550: each within 10 us of launches (511 for the
    former as tiles). The line is at 10 times."""
    thin, square = _us(1, 300000, 1), _us(550, 1, 550)
    print("thin %.1f us, square %.1f us" % (thin, square))
    assert thin < 10 * square

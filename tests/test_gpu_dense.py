"""The dense layers' kernels at the edges of their tiles and dispatch: rows that leave a tile partly
empty, every run length of the inputs, channel and row counts that select each wave tile, shapes and
alignments that take the general product. Dyadic inputs: every sum is exact in float32, so results
must equal the float64 layer oracle (bf16 outputs: its value rounded to nearest even)."""
import numpy as np
import pytest
import torch

from oracle import cnn_oracle as co
from paper_2602_22625_amd import capi, synth

pytestmark = pytest.mark.gpu


def dyadic(g, shape, num, den):
    return (g.integers(-num, num + 1, size=shape) / den).astype(np.float32)


def bf(a, off=0):
    """A device bfloat16 copy that starts `off` values past a 16-byte boundary."""
    a = np.asarray(a, np.float32)
    b = torch.zeros(a.size + off, device="cuda", dtype=torch.bfloat16)
    b[off:] = torch.tensor(a.reshape(-1), device="cuda").to(torch.bfloat16)
    return b[off:]


def bf16_round(a):
    return synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(np.asarray(a, np.float32)))


# (rows, inputs, outputs, offset of the 16-bit buffers): runs of 32, 64, 128 and 256 inputs, one and
# several; tiles 1 x 1, 1 x 2, 1 x 4 and 2 x 4; inputs or outputs the kernels refuse; misaligned
SHAPES = [(1, 32, 16, 0), (3, 64, 48, 0), (16, 96, 32, 0), (65, 128, 64, 0), (72, 160, 96, 0),
          (1000, 256, 512, 0), (2048, 512, 512, 0), (4104, 512, 512, 0), (5480, 32, 96, 0),
          (40, 40, 24, 0), (24, 256, 64, 1)]


@pytest.mark.parametrize("shape", SHAPES)
def test_dense_layers_exact(shape):
    B, K, N, off = shape
    g = np.random.default_rng(sum(shape))
    st = capi.stream_handle()
    x, w, b = dyadic(g, (B, K), 4, 4), dyadic(g, (N, K), 4, 8), dyadic(g, (N,), 8, 16)
    # (16-byte loads of a plain product need alignment: only the gradients accept the offset)
    if not off:
        for relu in (0, 1):
            ref = co.linear_forward(x, w, b, relu=bool(relu))
            y = torch.empty(B, N, device="cuda", dtype=torch.bfloat16)
            y32 = torch.empty(B, N, device="cuda")
            capi.dbmp_cnn_linear_forward(st, bf(x), B, K, bf(w), torch.tensor(b, device="cuda"), N,
                                         relu, y, y32)
            torch.cuda.synchronize()
            assert np.array_equal(y32.cpu().numpy(), ref.astype(np.float32))
            assert np.array_equal(y.float().cpu().numpy(), bf16_round(ref))
    dz = dyadic(g, (B, N), 4, 16)
    if not off:
        wt = torch.empty(K, N, device="cuda", dtype=torch.bfloat16)
        capi.dbmp_cnn_cast_weights(st, torch.tensor(w, device="cuda"), N, 1, K, None, wt)
        dx = torch.empty(B, K, device="cuda", dtype=torch.bfloat16)
        for m in (None, x):
            capi.dbmp_cnn_linear_backward_data(st, bf(dz), B, N, wt, K,
                                               None if m is None else bf(m), dx)
            torch.cuda.synchronize()
            want = bf16_round(co.linear_backward_data(dz, w, mask=m))
            assert np.array_equal(dx.float().cpu().numpy(), want)
    rw, rb = co.linear_backward_weight(x, dz)
    for bias in (True, False):  # added to what is there
        dw = torch.full((N, K), 0.5, device="cuda")
        db = torch.full((N,), -0.25, device="cuda") if bias else None
        capi.dbmp_cnn_linear_backward_weight(st, bf(x, off), bf(dz, off), B, K, N, dw, db)
        torch.cuda.synchronize()
        assert np.array_equal(dw.cpu().numpy(), (rw + 0.5).astype(np.float32))
        if bias:
            assert np.array_equal(db.cpu().numpy(), (rb - 0.25).astype(np.float32))


# one layer off the vector forms; all of them at once (R, T, C around the 64 x 64 tile; more layers
# than one launch takes)
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("shapes", [[(5, 1, 3)], [(64, 9, 64)],
                                    [(32, 9, 8), (65, 1, 130), (1, 9, 64), (512, 1, 256), (24, 3, 20)],
                                    [(8 * k, 1 + k % 3, 4 * k) for k in range(1, 20)]])
def test_cast_layers(shapes, off):
    g = np.random.default_rng(len(shapes))
    layers, want = [], []
    for R, T, C in shapes:
        w = g.standard_normal((R, T, C)).astype(np.float32)
        d = torch.zeros(w.size + off, device="cuda")
        d[off:] = torch.tensor(w.reshape(-1), device="cuda")
        wb, wt = (torch.zeros(w.size + 8, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        layers.append((d[off:], R, T, C, wb[off:], wt[off:]))
        want.append(bf16_round(w))
    layers[0] = layers[0][:4] + (None,) + layers[0][5:]
    capi.dbmp_cnn_cast_layers(capi.stream_handle(), layers)
    torch.cuda.synchronize()
    for k, ((_, R, T, C, wb, wt), r) in enumerate(zip(layers, want)):
        n = R * T * C
        assert np.array_equal(wt[:n].float().cpu().numpy(), r.transpose(2, 1, 0).reshape(-1)), k
        assert not wt[n:].any()
        if wb is not None:
            assert np.array_equal(wb[:n].float().cpu().numpy(), r.reshape(-1)), k
            assert not wb[n:].any()

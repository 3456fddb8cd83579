"""Every build of the learned initialiser's kernels: the wave tiles of the forward and the input gradient
(1 x 1, 1 x 2, 1 x 4 and 2 x 4 fragments; the larger ones are for layers of many pixels) for each channel
count, those of the dense layers for each run of inputs, the first layer's walk over several tiles per workgroup, and the weight gradient's
channel tiles, row splits and pixel splits. The sizes follow from the launch rules in conv.hip and
wgrad.hip, which the tests restate to be sure of the build they reach. Dyadic inputs: every sum is
exact in float32, so results equal the float64 reference (bf16 outputs: rounded to nearest even)."""
import pytest
import torch
import torch.nn.functional as F

from paper_2602_22625_amd import capi

pytestmark = pytest.mark.gpu


def _dyadic(g, shape, num, den):
    return torch.randint(-num, num + 1, shape, generator=g, device="cuda").double() / den


def _gen(*key):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(key))
    return g


def _bf(a):
    return a.to(torch.bfloat16)


def _patches(x):
    """[B, H, W, C] -> [P, 9 C] in the weights' order (tap, channel), float64."""
    B, H, W, C = x.shape
    xp = F.pad(x.permute(0, 3, 1, 2), (1, 1, 1, 1))
    u = xp.unfold(2, 3, 2).unfold(3, 3, 2)  # [B, C, OH, OW, 3, 3]
    return u.permute(0, 2, 3, 4, 5, 1).reshape(B * (H // 2) * (W // 2), 9 * C)


def _input_gradient(dz, w, H, W):
    """dz [B, OH, OW, Co], w [Co, 9, Ci] -> [B, H, W, Ci], float64."""
    B, OH, OW, Co = dz.shape
    Ci = w.shape[2]
    out = torch.zeros(B, H + 2, W + 2, Ci, device="cuda", dtype=torch.float64)
    for t in range(9):
        y, x = t // 3, t % 3
        part = (dz.reshape(-1, Co) @ w[:, t]).view(B, OH, OW, Ci)
        out[:, y:y + 2 * OH:2, x:x + 2 * OW:2] += part
    return out[:, 1:H + 1, 1:W + 1]


def _tile(P, N):
    """launch_mn's rule: fragments of pixels and channels of a wave."""
    def waves(mt, nt):
        return -(-P // (16 * mt)) * (N // (16 * nt))
    if N % 64 == 0 and waves(2, 4) >= 1024:
        return 2, 4
    if N % 64 == 0 and waves(1, 4) >= 1024:
        return 1, 4
    if N % 64 and N % 32 == 0 and waves(1, 2) >= 1024:
        return 1, 2
    return 1, 1


# the tile, output pixels per image, images, and the channels that a wave's fragments divide (N); no pixel
# count fills the last workgroup
TILES = [((2, 4), 8, 33, 31, 256), ((1, 4), 5, 29, 29, 256), ((1, 2), 7, 28, 28, 96),
         ((2, 4), 33, 33, 31, 64), ((1, 1), 3, 5, 7, 112)]


@pytest.mark.parametrize("C", [32, 64, 128, 256])
@pytest.mark.parametrize("tile,B,OH,OW,N", TILES)
def test_forward(tile, B, OH, OW, N, C):
    P = B * OH * OW
    assert _tile(P, N) == tile and P % (64 * tile[0])
    g = _gen(P, N, C)
    x, w, b = _dyadic(g, (B, 2 * OH, 2 * OW, C), 4, 4), _dyadic(g, (N, 9, C), 4, 8), _dyadic(g, (N,), 8, 16)
    y = torch.empty(B, OH, OW, N, device="cuda", dtype=torch.bfloat16)
    y32 = torch.empty(B, OH, OW, N, device="cuda")
    capi.dbmp_cnn_conv_forward(capi.stream_handle(), _bf(x), B, 2 * OH, 2 * OW, C, _bf(w), b.float(), N,
                               1, y, y32)
    ref = (_patches(x) @ w.reshape(N, -1).t() + b).clamp(min=0).view(B, OH, OW, N)
    assert torch.equal(y32.double(), ref)
    assert torch.equal(y, _bf(ref.float()))


@pytest.mark.parametrize("C", [32, 64, 128, 256])
@pytest.mark.parametrize("tile,B,OH,OW,N", TILES)
def test_input_gradient(tile, B, OH, OW, N, C):
    P = B * OH * OW
    assert _tile(P, N) == tile
    g = _gen(P, N, C, 1)
    dz, w = _dyadic(g, (B, OH, OW, C), 4, 16), _dyadic(g, (C, 9, N), 4, 8)
    mask = _dyadic(g, (B, 2 * OH, 2 * OW, N), 2, 2)
    wt = _bf(w).permute(2, 1, 0).contiguous()  # [N][9][C]
    dx = torch.empty(B, 2 * OH, 2 * OW, N, device="cuda", dtype=torch.bfloat16)
    capi.dbmp_cnn_conv_backward_data(capi.stream_handle(), _bf(dz), B, 2 * OH, 2 * OW, N, wt, C,
                                     _bf(mask), dx)
    ref = _input_gradient(dz, w, 2 * OH, 2 * OW) * (mask > 0)
    assert torch.equal(dx.double(), _bf(ref.float()).double())  # (either zero)


# the tile, rows and outputs; one run of C inputs and three
@pytest.mark.parametrize("runs", [1, 3])
@pytest.mark.parametrize("C", [32, 64, 128, 256])
@pytest.mark.parametrize("tile,B,N", [((2, 4), 8185, 256), ((1, 4), 4205, 256), ((1, 2), 5489, 96),
                                      ((2, 4), 32740, 64), ((1, 1), 105, 112)])
def test_dense(tile, B, N, C, runs):
    K = C * runs
    assert _tile(B, N) == tile and min(K & -K, 256) == C and B % (64 * tile[0])
    g = _gen(B, N, K)
    x, w, b = _dyadic(g, (B, K), 4, 4), _dyadic(g, (N, K), 4, 8), _dyadic(g, (N,), 8, 16)
    y = torch.empty(B, N, device="cuda", dtype=torch.bfloat16)
    y32 = torch.empty(B, N, device="cuda")
    st = capi.stream_handle()
    capi.dbmp_cnn_linear_forward(st, _bf(x), B, K, _bf(w), b.float(), N, 1, y, y32)
    ref = (x @ w.t() + b).clamp(min=0)
    assert torch.equal(y32.double(), ref)
    assert torch.equal(y, _bf(ref.float()))
    # as the input gradient of a layer of N inputs and K outputs (w as its transposed weights)
    mask = _dyadic(g, (B, N), 2, 2)
    dx = torch.empty(B, N, device="cuda", dtype=torch.bfloat16)
    capi.dbmp_cnn_linear_backward_data(st, _bf(x), B, K, _bf(w), N, _bf(mask), dx)
    assert torch.equal(dx.double(), _bf(((x @ w.t()) * (mask > 0)).float()).double())


@pytest.mark.parametrize("N", [16, 32])
def test_first_layer_many_tiles(N):
    """More tiles than workgroups (2,048 are resident), the last one partly empty."""
    B, OH, OW = 33, 127, 129
    P = B * OH * OW
    assert -(-P // 256) > 2048 and P % 256
    g = _gen(N)
    x, w, b = _dyadic(g, (B, 2 * OH, 2 * OW, 8), 4, 4), _dyadic(g, (N, 9, 8), 4, 8), _dyadic(g, (N,), 8, 16)
    y32 = torch.empty(B, OH, OW, N, device="cuda")
    capi.dbmp_cnn_conv_forward(capi.stream_handle(), _bf(x), B, 2 * OH, 2 * OW, 8, _bf(w), b.float(), N,
                               0, None, y32)
    for i in range(B):
        ref = (_patches(x[i:i + 1]) @ w.reshape(N, -1).t() + b).view(OH, OW, N)
        assert torch.equal(y32[i].double(), ref), i


def _wgrad(B, H, W, Ci, Co):
    """conv_backward_weight_direct's choice: (channels of dz per lane, rows of 8 pixels, pixel splits),
    or None for the general product."""
    OW, P = W // 2, B * (H // 2) * (W // 2)
    if Co % 32 or (Ci != 8 and Ci % 32) or OW % 4 or P % 8:
        return None
    wm = 4 if Co % 64 == 0 and Ci != 8 else 2
    tiles = Co // (16 * wm) * (1 if Ci == 8 else Ci // 32 * 3)
    s = min(max(1, 512 // tiles), max(1, -(-(P // 8) // 4) // 16))
    return wm, 2 if OW % 8 else 1, s // 8 * 8 if s >= 8 else 4 if s >= 4 else 2 if s >= 2 else 1


# (the build, then B, H, W, Ci, Co); Ci = 8 is the first layer's kernel
@pytest.mark.parametrize("build,shape", [
    ((2, 1, 1), (2, 8, 32, 32, 32)), ((2, 1, 2), (4, 32, 32, 64, 96)), ((2, 1, 8), (9, 64, 32, 32, 32)),
    ((2, 2, 1), (2, 12, 8, 32, 32)), ((2, 2, 1), (2, 8, 24, 64, 96)), ((2, 2, 4), (8, 32, 40, 32, 32)),
    ((4, 1, 1), (1, 8, 16, 64, 64)), ((4, 1, 2), (4, 32, 32, 128, 256)), ((4, 1, 4), (8, 32, 32, 32, 64)),
    ((4, 1, 32), (16, 64, 64, 32, 64)), ((4, 2, 1), (2, 16, 8, 128, 64)), ((4, 2, 2), (8, 32, 24, 64, 64)),
    ((4, 2, 16), (10, 64, 56, 32, 128)),
    ((2, 2, 1), (2, 8, 8, 8, 32)), ((2, 2, 2), (8, 32, 24, 8, 32)), ((2, 1, 4), (8, 32, 32, 8, 64)),
    ((2, 1, 1), (1, 6, 16, 8, 32)), ((2, 2, 8), (12, 64, 24, 8, 96)),
    (None, (3, 10, 8, 32, 32)), (None, (5, 6, 24, 64, 96)), (None, (1, 4, 18, 32, 64))])
def test_weight_gradient(build, shape):
    B, H, W, Ci, Co = shape
    assert _wgrad(*shape) == build
    g = _gen(*shape)
    x, dz = _dyadic(g, (B, H, W, Ci), 4, 4), _dyadic(g, (B, H // 2, W // 2, Co), 4, 16)
    rw = (dz.reshape(-1, Co).t() @ _patches(x)).view(Co, 9, Ci)
    for bias in (True, False):
        dw = torch.full((Co, 9, Ci), 0.5, device="cuda")
        db = torch.full((Co,), -0.25, device="cuda") if bias else None
        capi.dbmp_cnn_conv_backward_weight(capi.stream_handle(), _bf(x), _bf(dz), B, H, W, Ci, Co, dw, db)
        assert torch.equal(dw.double(), rw + 0.5)
        if bias:
            assert torch.equal(db.double(), dz.reshape(-1, Co).sum(0) - 0.25)

"""The calls whose time counts: what a user of this package has it do, through its public entry
points, over the range of sizes, types and options that the package's workloads span.

listed() gives the named cases, draw(rng) one more case of the same ranges, prepare(case, seed)
what a program holds before the call, run(state) one call, work(case) the bytes and operations
one call cannot do without, and exact(case, seed) the call's result in float64, formed with plain
torch and numpy (None where that would take too long).

Kinds:
  fit        one Adam iteration of a fit, replayed from its captured graph (forward, MSE
             backward, Adam), every iteration from the same primitives (`hold`)
  fit_batch  the same over many images of uneven size advanced together
  autograd   differentiable render: forward, then the backward of gradients of image and alpha
  render     forward only, the atlas stored once
  constrain  one iteration with a noise canvas and the spatial-constraint loss
  start      the start of a fit: bitmaps blurred, structure-aware initial primitives
  export     every primitive as a layer of its own
  conv       one convolution layer of the learned initialiser: forward and both gradients
  train      one training step of the learned initialiser
  predict    its prediction
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_22625_amd import aids, capi, cnn_init, synth
from paper_2602_22625_amd.fit import BatchFitter, Fitter
from paper_2602_22625_amd.render import Renderer, render

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SCHED = {"grid": 0, "sorted": 1}
# bitmaps of an atlas (count, edge) and the share of a primitive's square that its support box
# covers on average (stars and strokes have tight boxes)
ATLAS = {"disk32": (1, 32, 1.0), "ss64x16": (16, 64, 0.45), "ss128x64": (64, 128, 0.43)}
EXACT_PRIMS = 9000      # most primitives that exact() composites one by one
FWD_FLOP, BWD_FLOP = 31, 85   # operations of one (pixel, primitive) pair, Eqs. 1-5 and S1-S5


# ------------------------------------------------------------------------------------------
# Cases
# ------------------------------------------------------------------------------------------
def _fit(H, W, N, atlas, dtype, s, std, bg="white", sched="grid", tile=16, **kw):
    return dict(kw, kind="fit", H=H, W=W, N=N, atlas=atlas, dtype=dtype, s=s, std=std, bg=bg,
                sched=sched, tile=tile)


def listed():
    return [
        # a small icon fit: one soft disk, 64 primitives; a step is two short launches
        _fit(128, 128, 64, "disk32", "f32", 8.0, 0.3, name="fit_128"),
        # the ordinary fit: 4,096 primitives on 512 x 512, tiles dealt longest list first
        _fit(512, 512, 4096, "ss64x16", "f32", 12.0, 0.5, sched="sorted", name="fit_512"),
        # the headline workload: 65,536 primitives on 2048 x 2048, bfloat16 bitmaps
        _fit(2048, 2048, 65536, "ss128x64", "bf16", 10.0, 0.6, name="fit_2048_bf16"),
        # a photograph's odd size with the reduced-precision raster and a background image
        _fit(751, 1000, 6000, "ss64x16", "f16", 12.0, 0.5, bg="pixel", name="fit_odd_f16"),
        # 64 fits of uneven size and primitive count advanced together
        dict(kind="fit_batch", images=64, smin=256, smax=1024, nmin=512, nmax=16384,
             atlas="ss64x16", dtype="f32", sched="sorted", tile=16, name="fit_batch_64"),
        # a caller's own loss through torch.autograd, gradients of image and alpha, odd size
        dict(kind="autograd", H=301, W=417, N=1500, atlas="ss64x16", dtype="f32", s=12.0, std=0.5,
             tile=16, name="autograd_odd"),
        # rendering fitted primitives, no gradients
        dict(kind="render", H=1024, W=1024, N=16384, atlas="ss128x64", dtype="bf16", s=10.0,
             std=0.6, tile=16, name="render_1024_bf16"),
        # spatially constrained fit (a shape on a transparent ground): noise canvas, render,
        # constraint loss, backward with a gradient of alpha
        dict(kind="constrain", H=768, W=640, N=4096, atlas="ss64x16", dtype="f32", s=12.0,
             std=0.5, tile=16, name="constrain_768"),
        # what precedes a large fit: blurred bitmaps, structure-aware primitives
        dict(kind="start", H=2048, W=2048, N=65536, atlas="ss128x64", dtype="bf16", win=7,
             name="start_2048"),
        # layers of a finished fit at twice the canvas resolution
        dict(kind="export", H=1024, W=1024, N=8192, atlas="ss64x16", dtype="f32", s=12.0, std=0.5,
             rho=2.0, name="export_1024_x2"),
        # the learned initialiser: its second convolution at the training batch, and a whole step
        dict(kind="conv", B=64, S=128, cin=32, cout=64, name="conv_32_64"),
        dict(kind="train", B=64, name="train_64"),
    ]


def _lu(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def draw(rng):
    kind = rng.choice(["fit", "fit", "fit", "fit_batch", "autograd", "render", "constrain",
                       "start", "export", "conv", "train", "predict"])
    if kind == "fit_batch":
        smin = int(_lu(rng, 64, 512))
        nmin = int(_lu(rng, 64, 1024))
        return dict(kind=kind, images=rng.randint(2, 48), smin=smin,
                    smax=min(1024, int(smin * rng.uniform(1.0, 4.0))), nmin=nmin,
                    nmax=int(nmin * rng.uniform(1.0, 8.0)), atlas=rng.choice(["disk32", "ss64x16"]),
                    dtype=rng.choice(["f32", "bf16", "f16"]), sched=rng.choice(["grid", "sorted"]),
                    tile=rng.choice([16, 16, 16, 8, 32]))
    if kind in ("train", "predict"):
        return dict(kind=kind, B=int(_lu(rng, 1, 64.99)))
    if kind == "conv":
        l = rng.randrange(len(cnn_init.CONV))
        ci, co = cnn_init.CONV[l]
        return dict(kind=kind, B=int(_lu(rng, 1, 64.99)), S=cnn_init.IMG >> l, cin=ci, cout=co)
    atlas = rng.choice(["disk32", "ss64x16", "ss64x16", "ss128x64"])
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    H, W = int(_lu(rng, 96, 2048.99)), int(_lu(rng, 96, 2048.99))
    N = max(16, min(65536, int(H * W * _lu(rng, 1 / 400, 1 / 60))))
    if kind == "start":
        return dict(kind=kind, H=H, W=W, N=N, atlas=atlas, dtype=dtype,
                    win=rng.choice([3, 5, 7, 7, 7, 9, 15]))
    size = dict(H=H, W=W, N=N, atlas=atlas, dtype=dtype, s=rng.uniform(8.0, 13.0),
                std=rng.uniform(0.2, 0.6))
    if kind == "export":
        rho = rng.choice([1.0, 1.5, 2.0])
        return dict(size, kind=kind, N=min(N, 16384), rho=rho)
    size["tile"] = rng.choice([16, 16, 16, 8, 32])
    if kind == "fit":
        return dict(size, kind=kind, bg=rng.choice(["white", "pixel"]),
                    sched=rng.choice(["grid", "sorted"]))
    return dict(size, kind=kind)


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, stream):
    g = torch.Generator(device=_dev())
    g.manual_seed((int(seed) * 1000003 + stream * 7919 + 17) & 0x7FFFFFFF)
    return g


_atlases = {}


def _atlas(kind, dtype):
    """The package's synthetic bitmaps: the same for every seed, as a user's templates are."""
    if (kind, dtype) not in _atlases:
        a = torch.tensor(synth.make_atlas(kind), device=_dev())
        _atlases[kind, dtype] = a.to(DTYPES[dtype]).contiguous()
    return _atlases[kind, dtype]


def _params(N, H, W, s, std, B, seed):
    """Initial primitives: uniform positions and angles, log-normal sizes, normal opacity logits,
    logits of uniform colours, uniform bitmaps."""
    dev, g = _dev(), _gen(seed, 1)
    u = torch.rand(N, 6, generator=g, device=dev)
    z = torch.randn(N, 2, generator=g, device=dev)
    p = torch.empty(N, 8, device=dev)
    p[:, 0], p[:, 1] = u[:, 0] * W, u[:, 1] * H
    p[:, 2] = math.log(s) + std * z[:, 0]
    p[:, 3] = 2.0 * math.pi * u[:, 2]
    p[:, 4] = z[:, 1]
    c = u[:, 3:6].clamp(1e-3, 1 - 1e-3)
    p[:, 5:8] = torch.log(c / (1 - c))
    idx = torch.randint(0, B, (N,), generator=g, device=dev).to(torch.int32)
    return p, idx


def _image(H, W, seed, stream=2, blobs=24):
    """A smooth target in [0, 1] with anti-aliased ellipses, odd sizes included."""
    dev, g = _dev(), _gen(seed, stream)
    low = torch.rand(1, 3, max(2, H // 64) + 1, max(2, W // 64) + 1, generator=g, device=dev)
    img = torch.nn.functional.interpolate(low, size=(H, W), mode="bilinear", align_corners=True)[0]
    u = torch.rand(blobs, 8, generator=g, device=dev).cpu().double()
    ys = torch.arange(H, device=dev, dtype=torch.float32)[:, None]
    xs = torch.arange(W, device=dev, dtype=torch.float32)[None, :]
    L = float(min(H, W))
    for e in range(blobs):
        cx, cy = float(u[e, 0]) * W, float(u[e, 1]) * H
        ax, ay = L * (0.02 + 0.13 * float(u[e, 2])), L * (0.02 + 0.13 * float(u[e, 3]))
        c, s = math.cos(math.pi * float(u[e, 4])), math.sin(math.pi * float(u[e, 4]))
        dx, dy = xs - cx, ys - cy
        r = torch.sqrt(((c * dx + s * dy) / ax) ** 2 + ((c * dy - s * dx) / ay) ** 2)
        cov = torch.clamp(0.5 - (r - 1.0) * min(ax, ay), 0.0, 1.0)
        col = torch.tensor([float(v) for v in u[e, 5:8]], device=dev)[:, None, None]
        img = img + (col - img) * cov
    return img.clamp(0.0, 1.0).contiguous()


def _bg(case, seed):
    if case.get("bg") == "pixel":
        return torch.rand(3, case["H"], case["W"], generator=_gen(seed, 3), device=_dev())
    return torch.ones(3, device=_dev())


def _scene(case, seed):
    B = ATLAS[case["atlas"]][0]
    p, idx = _params(case["N"], case["H"], case["W"], case["s"], case["std"], B, seed)
    return p, idx, _atlas(case["atlas"], case["dtype"])


def _batch(case, seed):
    """[(params, idx, target)] of a batch: sizes spread over the case's ranges (primitive counts
    over their logarithm), the same for every seed, odd ones among them."""
    fits = []
    B = ATLAS[case["atlas"]][0]
    for k in range(case["images"]):
        S, N = _batch_size(case, k)
        p, idx = _params(N, S, S, 12.0 if case["atlas"] != "disk32" else 8.0, 0.5, B,
                         seed * 131 + k)
        fits.append((p, idx, _image(S, S, seed * 131 + k, blobs=4)))
    return fits


def _batch_size(case, k):
    S = case["smin"] + (case["smax"] - case["smin"]) * ((k * 7) % 16 + 0.5) / 16
    N = case["nmin"] * (case["nmax"] / case["nmin"]) ** ((k + 0.5) / case["images"])
    return int(round(S)), int(round(N))


def _export_scene(case, seed):
    """Fitted primitives to export: the seed deals a fixed set of positions, sizes and angles to
    the rows (so that the layers of every seed have the same total size) and draws the rest."""
    p, idx, atlas = _scene(case, seed)
    geo = _scene(case, 0)[0][:, :4]
    p[:, :4] = geo[torch.randperm(case["N"], generator=_gen(seed, 10), device=_dev())]
    return p, idx, atlas


def _shape_alpha(H, W, seed):
    """Target alpha of a shape: an opaque ellipse with a soft rim on a transparent ground."""
    u = torch.rand(2, generator=_gen(seed, 5), device=_dev()).tolist()
    ys = torch.arange(H, device=_dev(), dtype=torch.float32)[:, None]
    xs = torch.arange(W, device=_dev(), dtype=torch.float32)[None, :]
    r = torch.sqrt(((xs - W / 2) / (W * (0.3 + 0.1 * u[0]))) ** 2 +
                   ((ys - H / 2) / (H * (0.3 + 0.1 * u[1]))) ** 2)
    return torch.clamp((1.05 - r) * 10.0, 0.0, 1.0).contiguous()


LAMBDA = 1.0
NOISE_ITERATION = 7
LR_TRAIN = 1e-5
WIDTHS = [(8, 32), (32, 64), (64, 128), (128, 256), (256, 256), (256, 256)]
LOSS_W = (1.0, 1.0, 1.0, 0.1, 1.0, 1.0, 1.0, 1.0)
LAYERS = [(co, 9, ci) for ci, co in WIDTHS] + [(512, 1, 256), (512, 1, 512)]


def _net_weights(seed):
    """All weights and biases of the initialiser as one vector, layer by layer (a network some
    way into its training: He-scaled weights, small biases)."""
    g = _gen(seed, 6)
    parts = []
    for l, (R, T, C) in enumerate(LAYERS):
        fan = T * (3 if l == 0 else C)
        w = torch.randn(R, T, C, generator=g, device=_dev()) * math.sqrt(2.0 / fan)
        if l == 0:
            w[:, :, 3:] = 0.0
        parts += [w.reshape(-1), 0.05 * torch.randn(R, generator=g, device=_dev())]
    return torch.cat(parts)


def _net_data(case, seed):
    B = case["B"]
    base = [_image(256, 256, seed * 31 + k, blobs=8) for k in range(min(B, 8))]
    img = torch.stack([base[k % 8].roll(17 * (k // 8), 2) for k in range(B)]).contiguous()
    codes = torch.randn(B, 1024, 8, generator=_gen(seed, 7), device=_dev()).clamp(-4, 4)
    return img, codes


def _conv_data(case, seed):
    B, S, ci, co = case["B"], case["S"], case["cin"], case["cout"]
    g, dev, bf = _gen(seed, 8), _dev(), torch.bfloat16
    x = torch.randn(B, S, S, ci, generator=g, device=dev).relu().to(bf)
    if ci == 8:
        x[..., 3:] = 0.0
    w = (torch.randn(co, 9, ci, generator=g, device=dev) * math.sqrt(2.0 / (9 * ci)))
    b = 0.05 * torch.randn(co, generator=g, device=dev)
    dz = torch.randn(B, S // 2, S // 2, co, generator=g, device=dev) * 1e-3
    dz = (dz * (torch.rand(dz.shape, generator=g, device=dev) < 0.5)).to(bf)
    return x, w, b, dz


class _State:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "fit":
        p, idx, atlas = _scene(case, seed)
        f = Fitter(p, idx, atlas, _image(case["H"], case["W"], seed), bg=_bg(case, seed),
                   tile=case["tile"])
        f.R.set_schedule(SCHED[case["sched"]])
        f.capture(hold=p)
        return _State(kind=kind, f=f)
    if kind == "fit_batch":
        f = BatchFitter(_batch(case, seed), _atlas(case["atlas"], case["dtype"]),
                        tile=case["tile"])
        f.R.set_schedule(SCHED[case["sched"]])
        f.capture(hold=f.params.clone())
        return _State(kind=kind, f=f)
    if kind == "autograd":
        p, idx, atlas = _scene(case, seed)
        H, W = case["H"], case["W"]
        gI = torch.randn(3, H, W, generator=_gen(seed, 4), device=_dev()) / (H * W)
        gA = torch.randn(H, W, generator=_gen(seed, 5), device=_dev()) / (H * W)
        return _State(kind=kind, p=p.requires_grad_(True), idx=idx, atlas=atlas, H=H, W=W, gI=gI,
                      gA=gA, R=Renderer(), bg=_bg(case, seed), tile=case["tile"])
    if kind == "render":
        p, idx, atlas = _scene(case, seed)
        R = Renderer(check=False, list_capacity=1024)
        R.set_atlas(atlas)
        return _State(kind=kind, p=p, idx=idx, R=R, bg=_bg(case, seed), H=case["H"], W=case["W"],
                      tile=case["tile"])
    if kind == "constrain":
        p, idx, atlas = _scene(case, seed)
        H, W = case["H"], case["W"]
        R = Renderer(check=False, list_capacity=1024)
        R.set_atlas(atlas)
        e = lambda *s: torch.empty(*s, device=_dev())  # noqa: E731
        return _State(kind=kind, p=p, idx=idx, R=R, H=H, W=W, tile=case["tile"], seed=int(seed),
                      target=_image(H, W, seed), talpha=_shape_alpha(H, W, seed), bg=e(3, H, W),
                      image=e(3, H, W), alpha=e(H, W), gI=e(3, H, W), gA=e(H, W),
                      grad=e(case["N"], 8), loss=e(1))
    if kind == "start":
        N, dev, g = case["N"], _dev(), _gen(seed, 9)
        draws = (torch.rand(N, generator=g, device=dev), torch.rand(N, generator=g, device=dev),
                 torch.randn(N, 3, generator=g, device=dev))
        return _State(kind=kind, atlas=_atlas(case["atlas"], case["dtype"]), N=N, draws=draws,
                      target=_image(case["H"], case["W"], seed), win=case["win"])
    if kind == "export":
        p, idx, atlas = _export_scene(case, seed)
        return _State(kind=kind, p=p, idx=idx, atlas=atlas, H=case["H"], W=case["W"],
                      rho=case["rho"])
    if kind == "conv":
        x, w, b, dz = _conv_data(case, seed)
        B, S, ci, co = case["B"], case["S"], case["cin"], case["cout"]
        e = lambda *s, **k: torch.empty(*s, device=_dev(), **k)  # noqa: E731
        bf = torch.bfloat16
        wb, wt = e(co, 9, ci, dtype=bf), e(ci, 9, co, dtype=bf)
        capi.dbmp_cnn_cast_weights(capi.stream_handle(), w, co, 9, ci, wb, wt)
        return _State(kind=kind, x=x, b=b, dz=dz, wb=wb, wt=wt, B=B, S=S, ci=ci, co=co,
                      y=e(B, S // 2, S // 2, co, dtype=bf), dx=e(B, S, S, ci, dtype=bf),
                      dw=e(co, 9, ci), db=e(co))
    if kind in ("train", "predict"):
        net = cnn_init.InitNet()
        net.P.copy_(_net_weights(seed))
        net.cast()
        img, codes = _net_data(case, seed)
        return _State(kind=kind, net=net, img=img, codes=codes)
    raise ValueError(kind)


# ------------------------------------------------------------------------------------------
# One call
# ------------------------------------------------------------------------------------------
def run(s):
    if s.kind in ("fit", "fit_batch"):
        f = s.f
        f.step()
        return {"image": f.image, "grad": f.grad, "params": f.params, "m": f.m, "v": f.v}
    if s.kind == "autograd":
        image, alpha = render(s.p, s.R, s.idx, s.atlas, s.H, s.W, s.bg, 1.0, s.tile)
        (g,) = torch.autograd.grad((image, alpha), s.p, (s.gI, s.gA))
        return {"image": image.detach(), "alpha": alpha.detach(), "grad": g}
    if s.kind == "render":
        image, alpha = s.R.render(s.p, s.idx, None, s.H, s.W, s.bg, tile=s.tile)
        return {"image": image, "alpha": alpha}
    if s.kind == "constrain":
        st = capi.stream_handle()
        aids.dbmp_noise_canvas(st, s.seed, NOISE_ITERATION, s.H, s.W, s.bg)
        s.R.render(s.p, s.idx, None, s.H, s.W, s.bg, tile=s.tile, image=s.image, alpha=s.alpha)
        s.loss.zero_()
        aids.dbmp_constraint_loss(st, s.image, s.alpha, s.target, s.talpha, s.H, s.W, LAMBDA,
                                  s.gI, s.gA, s.loss)
        s.R.backward(s.gI, s.gA, out=s.grad)
        return {"bg": s.bg, "image": s.image, "alpha": s.alpha, "grad": s.grad, "loss": s.loss}
    if s.kind == "start":
        soft = aids.blur_atlas(s.atlas, 1.0)
        params, nlv, _ = aids.sa_init(s.target, s.N, 4.0, 24.0, win=s.win, draws=s.draws)
        return {"soft": soft, "params": params, "nlv": nlv}
    if s.kind == "export":
        boxes, offsets, alpha, colours = aids.export_layers(s.p, s.idx, s.atlas, s.H, s.W, s.rho)
        return {"boxes": boxes, "offsets": offsets, "alpha": alpha, "colours": colours}
    if s.kind == "conv":
        st = capi.stream_handle()
        capi.dbmp_cnn_conv_forward(st, s.x, s.B, s.S, s.S, s.ci, s.wb, s.b, s.co, 1, s.y)
        s.dw.zero_()
        s.db.zero_()
        capi.dbmp_cnn_conv_backward_weight(st, s.x, s.dz, s.B, s.S, s.S, s.ci, s.co, s.dw, s.db)
        capi.dbmp_cnn_conv_backward_data(st, s.dz, s.B, s.S, s.S, s.ci, s.wt, s.co, s.x, s.dx)
        return {"y": s.y, "dx": s.dx, "dw": s.dw, "db": s.db}
    if s.kind == "train":
        net = s.net
        net.train_step(s.img, s.codes, LR_TRAIN)
        return {"out": net.out, "P": net.P, "m": net.m, "v": net.v}
    return {"params": s.net.predict(s.img)}


# ------------------------------------------------------------------------------------------
# What a call cannot do without
# ------------------------------------------------------------------------------------------
def _pairs(N, s, std, atlas):
    return N * 4.0 * s * s * math.exp(2.0 * std * std) * ATLAS[atlas][2]


def _atlas_bytes(case):
    n, e, _ = ATLAS[case["atlas"]]
    return n * e * e * (4 if case["dtype"] == "f32" else 2)


def work(case):
    kind = case["kind"]
    if kind in ("fit", "autograd", "render", "constrain"):
        px, N = case["H"] * case["W"], case["N"]
        pairs = _pairs(N, case["s"], case["std"], case["atlas"])
        by = 36.0 * N + _atlas_bytes(case)          # parameters and bitmap indices, bitmaps
        fl = pairs * (FWD_FLOP if kind == "render" else FWD_FLOP + BWD_FLOP)
        if kind == "render":
            by += 16.0 * px                          # image and alpha
        elif kind == "fit":                          # target in, image out; gradient and state
            by += 24.0 * px + 224.0 * N + (12.0 * px if case["bg"] == "pixel" else 0.0)
        elif kind == "autograd":                     # image, alpha and their gradients
            by += 32.0 * px + 32.0 * N
        else:                                        # target and alpha in; canvas, image, alpha out
            by += 44.0 * px + 32.0 * N
        return {"bytes": by, "flops": fl}
    if kind == "fit_batch":
        by = fl = 0.0
        for k in range(case["images"]):
            S, N = _batch_size(case, k)
            by += 24.0 * S * S + 260.0 * N
            fl += _pairs(N, 12.0 if case["atlas"] != "disk32" else 8.0, 0.5, case["atlas"]) * \
                (FWD_FLOP + BWD_FLOP)
        return {"bytes": by + _atlas_bytes(case), "flops": fl}
    if kind == "start":
        px, N = case["H"] * case["W"], case["N"]
        return {"bytes": 2.0 * _atlas_bytes(case) + 16.0 * px + 52.0 * N,
                "flops": 3.0 * px * 8 * case["win"]}
    if kind == "export":
        n, e, _ = ATLAS[case["atlas"]]
        k = (e + 1) / (e - 1)
        # the axis-aligned box of a randomly rotated square: (|cos| + |sin|)^2 = 1 + 2 / pi
        vals = case["N"] * 4.0 * case["s"] ** 2 * math.exp(2.0 * case["std"] ** 2) * k * k * \
            (1.0 + 2.0 / math.pi) * case["rho"] ** 2
        return {"bytes": 4.0 * vals + 72.0 * case["N"] + _atlas_bytes(case), "flops": 20.0 * vals}
    if kind == "conv":
        B, S, ci, co = case["B"], case["S"], case["cin"], case["cout"]
        x, y, w = 2.0 * B * S * S * ci, 0.5 * B * S * S * co, 9.0 * ci * co
        return {"bytes": 2 * x + 2 * y + 8.0 * w, "flops": 3 * 2.0 * (B * S * S / 4) * w}
    n = sum(R * T * C + R for R, T, C in LAYERS)
    B, fl, act, S = case["B"], 0.0, 0.0, 256
    for l, (ci, co) in enumerate(WIDTHS):
        S //= 2
        f = 2.0 * B * S * S * co * 9 * (3 if l == 0 else ci)
        fl += f if kind == "predict" else f * (2 if l == 0 else 3)
        act += 2.0 * B * S * S * co
    f = 2.0 * B * 16 * (256 * 512 + 512 * 512)
    fl += f if kind == "predict" else 3 * f
    io = 12.0 * B * 65536 + 4.0 * B * 8192
    if kind == "predict":
        return {"bytes": io + 2.0 * n, "flops": fl}
    # activations written and read back for the gradients; weights, gradients and moments
    return {"bytes": io + 4.0 * B * 8192 + 2 * act + 28.0 * n, "flops": fl}


# ------------------------------------------------------------------------------------------
# The results in float64
# ------------------------------------------------------------------------------------------
def _composite(p, idx, atlas, H, W, bg, grads):
    """Image, alpha and the gradient table of one scene: the over operator front to back, one
    primitive at a time over its bounding box (Eqs. 1-5), then back to front with the
    division-free recurrence (Eq. 7, S4-S5). grads(image, alpha) -> (dL/dI, dL/dA or None), or
    None for a forward alone."""
    dev, f8 = p.device, torch.float64
    p = p.detach().to(f8)
    tex = torch.nn.functional.pad(atlas.to(f8), (1, 2, 1, 2))  # zero border
    Hb, Wb = atlas.shape[1], atlas.shape[2]
    cu, cv = 0.5 * (Wb - 1), 0.5 * (Hb - 1)
    s, ct, st = p[:, 2].exp(), p[:, 3].cos(), p[:, 3].sin()
    sig, col = torch.sigmoid(p[:, 4]), torch.sigmoid(p[:, 5:8])
    ex = s * (1 + 1 / cu) * ct.abs() + s * (1 + 1 / cv) * st.abs()
    ey = s * (1 + 1 / cu) * st.abs() + s * (1 + 1 / cv) * ct.abs()
    box = torch.stack([(p[:, 0] - ex).ceil().clamp(0, W), (p[:, 0] + ex).floor().clamp(-1, W - 1) + 1,
                       (p[:, 1] - ey).ceil().clamp(0, H), (p[:, 1] + ey).floor().clamp(-1, H - 1) + 1],
                      1).to(torch.int64).cpu().tolist()
    host = torch.stack([p[:, 0], p[:, 1], s, ct, st, sig], 1).cpu().tolist()
    kk = idx.cpu().tolist()
    hcol = col.cpu().tolist()
    xs, ys = torch.arange(W, device=dev, dtype=f8), torch.arange(H, device=dev, dtype=f8)
    T = torch.ones(H, W, device=dev, dtype=f8)
    C = torch.zeros(3, H, W, device=dev, dtype=f8)
    b = bg.to(f8) if bg.dim() == 3 else bg.to(f8)[:, None, None].expand(3, H, W)

    def sample(i):
        x0, x1, y0, y1 = box[i]
        x, y, si, c, sn, _ = host[i]
        dx, dy = (xs[x0:x1] - x)[None, :], (ys[y0:y1] - y)[:, None]
        u, v = (c * dx + sn * dy) / si, (c * dy - sn * dx) / si
        U, V = cu * (u + 1), cv * (v + 1)
        iu, iv = U.floor(), V.floor()
        wu, wv = U - iu, V - iv
        ok = (iu >= -1) & (iu <= Wb - 1) & (iv >= -1) & (iv <= Hb - 1)
        ju = torch.where(ok, iu + 1, torch.full_like(iu, Wb + 1)).long()
        jv = torch.where(ok, iv + 1, torch.full_like(iv, Hb + 1)).long()
        t, pitch = tex[kk[i]].reshape(-1), Wb + 3
        at = jv * pitch + ju
        p00, p01 = t[at], t[(at + 1).clamp_max(t.numel() - 1)]
        p10, p11 = t[(at + pitch).clamp_max(t.numel() - 1)], \
            t[(at + pitch + 1).clamp_max(t.numel() - 1)]
        z = ok.to(f8)
        p00, p01, p10, p11 = p00 * z, p01 * z, p10 * z, p11 * z
        top, bot = p00 + wu * (p01 - p00), p10 + wu * (p11 - p10)
        M = top + wv * (bot - top)
        MU = (p01 - p00) + wv * ((p11 - p10) - (p01 - p00))
        return M, MU, bot - top, u, v

    saved = [None] * len(kk)
    for i in range(len(kk)):
        x0, x1, y0, y1 = box[i]
        if x0 >= x1 or y0 >= y1:
            continue
        smp = sample(i)
        a = host[i][5] * smp[0]
        Tw = T[y0:y1, x0:x1]
        saved[i] = (smp, Tw.clone())
        w = Tw * a
        for ch in range(3):
            C[ch, y0:y1, x0:x1] += w * hcol[i][ch]
        Tw *= 1 - a
    image, alpha = C + T * b, 1 - T
    if grads is None:
        return image, alpha, None
    gI, gA = grads(image, alpha)
    gI = gI.to(f8)
    gA = torch.zeros(H, W, device=dev, dtype=f8) if gA is None else gA.to(f8)
    G, Bk = b.clone(), torch.ones(H, W, device=dev, dtype=f8)
    rows = []
    for i in range(len(kk) - 1, -1, -1):
        if saved[i] is None:
            rows.append(torch.zeros(8, device=dev, dtype=f8))
            continue
        (M, MU, MV, u, v), Tw = saved[i]
        saved[i] = None
        x0, x1, y0, y1 = box[i]
        _, _, si, c, sn, sg = host[i]
        a = sg * M
        Gw, gw = G[:, y0:y1, x0:x1], gI[:, y0:y1, x0:x1]
        ci = col[i][:, None, None]
        Bw = Bk[y0:y1, x0:x1]
        dal = Tw * ((gw * (ci - Gw)).sum(0) + gA[y0:y1, x0:x1] * Bw)
        dM = sg * dal
        gU, gV = dM * MU, dM * MV
        r = [(-gU * cu * c + gV * cv * sn).sum() / si, (-gU * cu * sn - gV * cv * c).sum() / si,
             -(gU * cu * u + gV * cv * v).sum(), (gU * cu * v - gV * cv * u).sum(),
             (dal * M).sum() * sg * (1 - sg)]
        dc = (gw * (Tw * a)).sum((1, 2)) * col[i] * (1 - col[i])
        rows.append(torch.cat([torch.stack(r), dc]))
        Gw += a * (ci - Gw)
        Bw *= 1 - a
    rows.reverse()
    return image, alpha, torch.stack(rows)


def _mse_grads(target):
    t = target.double()
    return lambda image, alpha: (2.0 * (image - t) / image.numel(), None)


def _noise(H, W, seed, iteration):
    """The noise canvas from numpy's Philox (whose counter steps before its first block)."""
    start = np.array([2 ** 64 - 1, iteration - 1, 0, 0], dtype=np.uint64)
    g = np.random.Philox(counter=start, key=np.array([seed, 0], dtype=np.uint64))
    w = g.random_raw(4 * H * W).reshape(H * W, 4)[:, :3]
    v = (w >> np.uint64(40)).astype(np.float64) * 2.0 ** -24
    return torch.tensor(v.T.reshape(3, H, W).copy(), device=_dev())


def _exact_start(case, seed):
    f8 = torch.float64
    a = _atlas(case["atlas"], case["dtype"]).to(f8)
    k = torch.tensor([math.exp(-d * d / 2.0) for d in range(-3, 4)], device=_dev(), dtype=f8)
    k = k / k.sum()
    pad = torch.nn.functional.pad(a, (3, 3, 3, 3))
    h = sum(k[d] * pad[:, :, d:d + a.shape[2]] for d in range(7))
    soft = sum(k[d] * h[:, d:d + a.shape[1], :] for d in range(7))
    H, W, hw = case["H"], case["W"], case["win"] // 2
    t = _image(H, W, seed).to(f8)
    st = prepare(case, seed)
    ones = torch.ones(1, H, W, device=_dev(), dtype=f8)

    def box_sum(x):
        q = torch.nn.functional.pad(x, (hw, hw, hw, hw))
        q = sum(q[:, :, d:d + W] for d in range(2 * hw + 1))
        return sum(q[:, d:d + H, :] for d in range(2 * hw + 1))

    n = box_sum(ones)
    m = box_sum(t) / n
    lv = (box_sum(t * t) / n - m * m).mean(0).clamp_min(0.0)
    nlv = (lv - lv.min()) / (lv.max() - lv.min())
    nf = nlv.float().double()
    w = torch.floor((0.1 + 0.9 * nf) * float(1 << 24)).to(torch.int64).reshape(-1)
    cdf = torch.cumsum(w, 0)
    u, ut, z = (d.to(f8) for d in st.draws)
    at = torch.searchsorted(cdf, torch.floor(u * float(cdf[-1])).to(torch.int64), right=True)
    rows = torch.empty(case["N"], 8, device=_dev(), dtype=f8)
    rows[:, 0], rows[:, 1] = (at % W).to(f8), (at // W).to(f8)
    rows[:, 2] = torch.log(24.0 - 20.0 * nf.reshape(-1)[at])
    rows[:, 3] = 2.0 * math.pi * ut
    rows[:, 4] = -2.0
    c = (t.reshape(3, -1)[:, at].T + 0.02 * z).clamp(1e-3, 1 - 1e-3)
    rows[:, 5:8] = torch.log(c / (1 - c))
    return {"soft": soft, "params": rows, "nlv": nlv}


def _exact_export(case, seed):
    f8 = torch.float64
    p, idx, atlas = _export_scene(case, seed)
    p, H, W, rho = p.to(f8), case["H"], case["W"], case["rho"]
    Hb, Wb = atlas.shape[1], atlas.shape[2]
    cu, cv = 0.5 * (Wb - 1), 0.5 * (Hb - 1)
    s, ct, st = p[:, 2].exp(), p[:, 3].cos(), p[:, 3].sin()
    HH, WW = round(H * rho), round(W * rho)
    X, Y = [], []
    for U in (-1.0, float(Wb)):
        for V in (-1.0, float(Hb)):
            u, v = U / cu - 1, V / cv - 1
            X.append(rho * (p[:, 0] + s * (ct * u - st * v) + 0.5) - 0.5)
            Y.append(rho * (p[:, 1] + s * (st * u + ct * v) + 0.5) - 0.5)
    X, Y = torch.stack(X), torch.stack(Y)
    x0 = (X.amin(0) - 1e-3).ceil().clamp_min(0)
    x1 = (X.amax(0) + 1e-3).floor().clamp_max(WW - 1)
    y0 = (Y.amin(0) - 1e-3).ceil().clamp_min(0)
    y1 = (Y.amax(0) + 1e-3).floor().clamp_max(HH - 1)
    ok = (x0 <= x1) & (y0 <= y1)
    w = torch.where(ok, x1 - x0 + 1, torch.zeros_like(x0)).long()
    h = torch.where(ok, y1 - y0 + 1, torch.zeros_like(x0)).long()
    off = torch.cumsum(w * h, 0) - w * h
    n = int((w * h).sum())
    tex = torch.nn.functional.pad(atlas.to(f8), (1, 2, 1, 2)).reshape(-1)
    pitch, page = Wb + 3, (Wb + 3) * (Hb + 3)
    ka = torch.sigmoid(p[:, 4])
    out = torch.empty(n, device=p.device, dtype=f8)
    prim = torch.repeat_interleave(torch.arange(case["N"], device=p.device), w * h)
    for a in range(0, n, 1 << 23):
        i = prim[a:a + (1 << 23)]
        j = torch.arange(a, a + i.numel(), device=p.device) - off[i]
        x = (x0[i] + (j % w[i]) + 0.5) / rho - 0.5
        y = (y0[i] + (j // w[i]) + 0.5) / rho - 0.5
        dx, dy = x - p[i, 0], y - p[i, 1]
        U = cu * ((ct[i] * dx + st[i] * dy) / s[i] + 1)
        V = cv * ((ct[i] * dy - st[i] * dx) / s[i] + 1)
        iu, iv = U.floor(), V.floor()
        inside = (iu >= -1) & (iu <= Wb - 1) & (iv >= -1) & (iv <= Hb - 1)
        at = idx[i].long() * page + (iv.clamp(-1, Hb - 1).long() + 1) * pitch + \
            iu.clamp(-1, Wb - 1).long() + 1
        wu, wv = U - iu, V - iv
        top = tex[at] + wu * (tex[at + 1] - tex[at])
        bot = tex[at + pitch] + wu * (tex[at + pitch + 1] - tex[at + pitch])
        out[a:a + i.numel()] = ka[i] * (top + wv * (bot - top)) * inside
    return {"boxes": None, "offsets": None, "alpha": out, "colours": torch.sigmoid(p[:, 5:8])}


def _conv64(x, w, b):
    """3 x 3 stride-2 convolution, x [B, C, S, S] float64, w [R, 9, C]."""
    B, C, S, _ = x.shape
    cols = torch.nn.functional.unfold(x, 3, padding=1, stride=2)        # [B, C * 9, L]
    k = w.permute(0, 2, 1).reshape(w.shape[0], -1)
    y = torch.matmul(k, cols) + b[None, :, None]
    return y.view(B, w.shape[0], S // 2, S // 2)


def _exact_conv(case, seed):
    f8 = torch.float64
    x, w, b, dz = _conv_data(case, seed)
    w = w.to(torch.bfloat16).to(f8).requires_grad_(True)
    x8 = x.to(f8).permute(0, 3, 1, 2).contiguous().requires_grad_(True)
    b8 = b.to(f8).requires_grad_(True)
    y = _conv64(x8, w, b8)
    dz8 = dz.to(f8).permute(0, 3, 1, 2).contiguous()
    dx, dw, db = torch.autograd.grad(y, (x8, w, b8), dz8)
    dx = dx.permute(0, 2, 3, 1) * (x > 0)
    return {"y": y.detach().relu().permute(0, 2, 3, 1).contiguous(), "dx": dx.contiguous(),
            "dw": dw, "db": db}


def _exact_net(case, seed):
    f8 = torch.float64
    P = _net_weights(seed).to(f8).requires_grad_(True)
    img, codes = _net_data(case, seed)
    at, h = 0, img.to(f8)
    for l, (R, T, C) in enumerate(LAYERS):
        w = P[at:at + R * T * C].view(R, T, C)
        b = P[at + R * T * C:at + R * T * C + R]
        at += R * T * C + R
        if T == 9:
            h = _conv64(h, w[:, :, :h.shape[1]], b).relu()
        else:
            if h.dim() == 4:
                h = h.permute(0, 2, 3, 1).reshape(-1, C)
            h = h @ w[:, 0].T + b
            if l == len(LAYERS) - 2:
                h = h.relu()
    out = h.view(case["B"], 1024, 8)
    if case["kind"] == "predict":
        i = torch.arange(1024, device=out.device)
        blk, pos = i // 64, i % 64
        cx = ((blk % 4) * 8 + pos % 8 + 0.5) * 8.0
        cy = ((blk // 4) * 8 + pos // 8 + 0.5) * 8.0
        t = out.detach().clone()
        keep = t[..., 3].clone()
        t = t.clamp(-4, 4)
        t[..., 3] = keep
        t *= torch.tensor([8.0, 8.0, 0.5, 1.0, 2.0, 2.0, 2.0, 2.0], device=t.device, dtype=f8)
        t[..., 0] += cx
        t[..., 1] += cy
        t[..., 2] += math.log(12.0)
        return {"params": t}
    d = out - codes.to(f8)
    wts = torch.tensor(LOSS_W, device=out.device, dtype=f8)
    sq = d * d
    terms = torch.cat([sq[..., :3], (1 - torch.cos(d[..., 3:4])), sq[..., 4:]], -1)
    loss = (terms * wts).sum() / (case["B"] * 1024)
    (g,) = torch.autograd.grad(loss, P)
    c1, c2 = 1.0 - 0.9, 1.0 - 0.999
    m, v = c1 * g, c2 * g * g
    P1 = P.detach() - LR_TRAIN * (m / c1) / ((v / c2).sqrt() + 1e-8)
    return {"out": out.detach().reshape(case["B"], 8192), "P": P1, "m": m, "v": v}


def exact(case, seed):
    kind = case["kind"]
    if kind == "fit":
        if case["N"] > EXACT_PRIMS:
            return None
        p, idx, atlas = _scene(case, seed)
        t = _image(case["H"], case["W"], seed)
        image, _, g = _composite(p, idx, atlas, case["H"], case["W"], _bg(case, seed),
                                 _mse_grads(t))
        z = torch.zeros_like(g)
        return {"image": image, "grad": g, "params": p.double(), "m": z, "v": z}
    if kind == "fit_batch":
        fits = _batch(case, seed)
        if sum(f[0].shape[0] for f in fits) > EXACT_PRIMS:
            return None
        atlas, bg = _atlas(case["atlas"], case["dtype"]), torch.ones(3, device=_dev())
        imgs, gs = [], []
        for p, idx, t in fits:
            image, _, g = _composite(p, idx, atlas, t.shape[1], t.shape[2], bg, _mse_grads(t))
            imgs.append(image.reshape(-1))
            gs.append(g)
        g = torch.cat(gs)
        z = torch.zeros_like(g)
        return {"image": torch.cat(imgs), "grad": g,
                "params": torch.cat([f[0] for f in fits]).double(), "m": z, "v": z}
    if kind in ("autograd", "render", "constrain"):
        if case["N"] > EXACT_PRIMS * (2 if kind == "render" else 1):
            return None
        p, idx, atlas = _scene(case, seed)
        H, W = case["H"], case["W"]
        if kind == "render":
            image, alpha, _ = _composite(p, idx, atlas, H, W, _bg(case, seed), None)
            return {"image": image, "alpha": alpha}
        if kind == "autograd":
            st = prepare(case, seed)
            image, alpha, g = _composite(p, idx, atlas, H, W, st.bg, lambda i, a: (st.gI, st.gA))
            return {"image": image, "alpha": alpha, "grad": g}
        bg = _noise(H, W, int(seed), NOISE_ITERATION)
        t, ta = _image(H, W, seed).double(), _shape_alpha(H, W, seed).double()
        loss = []

        def grads(image, alpha):
            d, e = (image - t) * (ta > 0), alpha - ta
            loss.append((d * d).mean() + LAMBDA * (e * e).mean())
            return 2.0 * d / d.numel(), 2.0 * LAMBDA * e / e.numel()

        image, alpha, g = _composite(p, idx, atlas, H, W, bg, grads)
        return {"bg": bg, "image": image, "alpha": alpha, "grad": g, "loss": loss[0].reshape(1)}
    if kind == "start":
        return _exact_start(case, seed)
    if kind == "export":
        return _exact_export(case, seed)
    if kind == "conv":
        return _exact_conv(case, seed)
    return _exact_net(case, seed)

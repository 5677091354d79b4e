"""The work that users of this framework have it do, as cases that can be timed.

Nine kinds of work, each through the public entry points of the package:

  render      one forward pass of every view (a viewer, evaluation images)
  grad        render through autograd and back-propagate dL/d(image)
  train       one optimisation step of every per-Gaussian parameter (TrainStep)
  decode      rendered compact features to codes or distributions
  language    decoder distribution, then the language feature map F = M S
  quantize    hybrid features against the discrete feature space
  smooth      the spatial smoothing loss and its gradients
  fit         one training step of the decoder on sampled pixels
  semantic    the uncertainty-weighted semantic loss of one view

A case is a dict of plain values. Inputs are made on the GPU from the seed
alone: Gaussians uniform in a volume with log-scales N(-3, 0.5), opacity logits
and semantic features N(0, 1), as in the benchmark's scenes.
"""
from __future__ import annotations

import math

import torch

from paper_2311_18482_amd import decode as D
from paper_2311_18482_amd import raster as R
from paper_2311_18482_amd.train import GROUPS, TrainStep

DEV = "cuda:0"
PARAMS = ("mean", "log_scale", "quat", "opacity_logit", "channels")
VOLUMES = {"front": ((-4.0, 4.0), (-4.0, 4.0), (2.0, 12.0)), "near": ((-1.0, 1.0), (-1.0, 1.0), (2.0, 6.0)),
           "rig": ((-4.0, 4.0), (-4.0, 4.0), (-4.0, 4.0))}
RIG_SIZES = ((640, 480), (960, 540), (1080, 720), (1280, 720), (1920, 1080))


# ---- the cases -------------------------------------------------------------------

def listed():
    return [
        # the smallest render: a 10k-Gaussian object in a 128 px thumbnail, default options; launches count
        dict(name="render_128px_10k", kind="render", scene="near", n=10_000, C=12, views=1, width=128, height=128,
             sizes="same", tile=16, lds_batch=256, persistent=False, ids_only=False),
        # an ordinary viewer frame: 300k Gaussians at 1080x720, default options
        dict(name="render_720p_300k", kind="render", scene="front", n=300_000, C=12, views=1, width=1080, height=720,
             sizes="same", tile=16, lds_batch=256, persistent=False, ids_only=False),
        # forward and backward of a small odd-sized crop, default options (early training, unit experiments)
        dict(name="grad_333x217_25k", kind="grad", scene="near", n=25_000, C=12, views=1, width=333, height=217,
             sizes="same", tile=16, lds_batch=256, persistent=False, ids_only=False),
        # the benchmark's view: 1M Gaussians at 1920x1080 with its options, through autograd
        dict(name="grad_1080p_1m", kind="grad", scene="rig", n=1_000_000, C=12, views=1, width=1920, height=1080,
             sizes="same", tile=32, lds_batch=256, persistent=False, ids_only=True),
        # a batch of 16 views of uneven size, as the multi-view objective renders them
        dict(name="grad_16views_1m", kind="grad", scene="rig", n=1_000_000, C=12, views=16, width=1920, height=1080,
             sizes="rig", tile=32, lds_batch=128, persistent=True, ids_only=True),
        # the largest: one training step of 3M Gaussians with 16 semantic channels over four 1080p views
        dict(name="train_4views_3m", kind="train", scene="rig", n=3_000_000, C=20, views=4, width=1920, height=1080,
             sizes="same", tile=32, lds_batch=256, persistent=False, ids_only=True),
        # codes of one rendered 1080p frame, read in place from the planar image (open-vocabulary viewing)
        dict(name="decode_codes_1080p", kind="decode", how="mlp", outputs="codes", P=1920 * 1080, K=128, planar=True,
             normalize=True),
        # language feature map of one 1080x720 frame, half precision, 512 dimensions
        dict(name="language_720p", kind="language", P=1080 * 720, K=128, d=512, half=True, planar=True),
        # quantisation of a scene's hybrid CLIP + DINO features with the gradient of the feature space
        dict(name="quantize_grad_1m", kind="quantize", P=1 << 20, K=128, d_clip=512, d_dino=384, grad=True),
        # smoothing loss over the Gaussians of the benchmark's scene
        dict(name="smooth_1m", kind="smooth", n=1_000_000, C=12),
        # one decoder training step on the batch that the benchmark trains with
        dict(name="fit_64k", kind="fit", P=65_536, K=128, normalize=True),
        # semantic loss of one 1080x720 training view, features and gradients in the rendered planes
        dict(name="semantic_720p", kind="semantic", P=1080 * 720, K=128, normalize=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("render", "render", "render", "grad", "grad", "grad", "train", "decode", "decode", "language",
                       "quantize", "smooth", "fit", "semantic"))
    if kind in ("render", "grad", "train"):
        views = rng.choice((1, 1, 1, 2, 3))
        scene = rng.choice(("near", "front", "rig"))   # the closer the volume, the wider the footprints
        c = dict(kind=kind, scene=scene, n=_log(rng, 2_000, {"near": 80_000, "front": 500_000, "rig": 1_000_000}[scene]),
                 C=rng.choice((4, 12, 12, 20)), views=views, width=_log(rng, 64, 1920), height=_log(rng, 64, 1080),
                 sizes="same", tile=rng.choice((16, 16, 32)), lds_batch=rng.choice((128, 256)),
                 persistent=rng.random() < 0.25, ids_only=rng.random() < 0.5)
        if kind == "train":
            c["C"] = rng.choice((12, 20))
        return c
    if kind == "decode":
        return dict(kind=kind, how=rng.choice(("mlp", "mlp", "table3", "folded", "plain")),
                    outputs=rng.choice(("codes", "codes", "probs")), P=_log(rng, 5_000, 4_000_000),
                    K=rng.choice((32, 64, 128, 128)), planar=rng.random() < 0.5, normalize=rng.random() < 0.5)
    if kind == "language":
        return dict(kind=kind, P=_log(rng, 5_000, 2_000_000), K=rng.choice((32, 64, 128, 128)),
                    d=rng.choice((256, 384, 512, 768)), half=rng.random() < 0.5, planar=rng.random() < 0.5)
    if kind == "quantize":
        return dict(kind=kind, P=_log(rng, 2_000, 1_000_000), K=rng.choice((32, 64, 128, 128)), d_clip=512,
                    d_dino=rng.choice((384, 768)), grad=rng.random() < 0.5)
    if kind == "smooth":
        return dict(kind=kind, n=_log(rng, 5_000, 2_000_000), C=rng.choice((12, 12, 20)))
    return dict(kind=kind, P=_log(rng, 4_000, 300_000 if kind == "fit" else 1_000_000),
                K=rng.choice((32, 64, 128, 128)), normalize=rng.random() < 0.5)


# ---- inputs ----------------------------------------------------------------------

class Cam:
    """A pinhole camera as views_build takes it."""

    def __init__(self, w, h, rot, t):
        self.w, self.h, self.f, self.rot, self.t = w, h, float(w), rot, t

    def as_tuple(self):
        return (self.w, self.h, self.f, self.f, self.w / 2.0, self.h / 2.0, tuple(self.rot), tuple(self.t))


def _cameras(case, seed):
    """Front cameras look down +z from the origin (further ones a little to the
    side); the rig's look at the origin from a sphere of radius 8."""
    g = torch.Generator().manual_seed(seed * 2 + 1)
    cams = []
    for v in range(case["views"]):
        w, h = case["width"], case["height"]
        if case["sizes"] == "rig":
            w, h = RIG_SIZES[3 * v % len(RIG_SIZES)]
        if case["scene"] != "rig":
            cams.append(Cam(w, h, (1.0, 0, 0, 0, 1.0, 0, 0, 0, 1.0), (0.05 * v, 0.0, 0.0)))
            continue
        pos = torch.randn(3, generator=g, dtype=torch.float64)
        pos = 8.0 * pos / pos.norm()
        z = -pos / pos.norm()
        up = torch.tensor([0.0, 1.0, 0.0] if abs(float(z[1])) < 0.99 else [0.0, 0.0, 1.0], dtype=torch.float64)
        y = -(up - up.dot(z) * z)
        y = y / y.norm()
        rot = torch.stack([torch.linalg.cross(y, z), y, z])
        cams.append(Cam(w, h, rot.reshape(-1).tolist(), (-(rot @ pos)).tolist()))
    return cams


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _scene(case, seed):
    g, n, C = _gen(seed), case["n"], case["C"]
    vol = VOLUMES[case["scene"]]
    lo = torch.tensor([v[0] for v in vol], device=DEV)
    hi = torch.tensor([v[1] for v in vol], device=DEV)
    q = torch.randn((n, 4), generator=g, device=DEV)
    ch = torch.cat([torch.rand((n, 3), generator=g, device=DEV), torch.randn((n, C - 4), generator=g, device=DEV),
                    torch.sigmoid(torch.randn((n, 1), generator=g, device=DEV))], dim=1)
    return dict(mean=lo + (hi - lo) * torch.rand((n, 3), generator=g, device=DEV),
                log_scale=-3.0 + 0.5 * torch.randn((n, 3), generator=g, device=DEV),
                quat=q / q.norm(dim=1, keepdim=True), opacity_logit=torch.randn(n, generator=g, device=DEV),
                channels=ch.contiguous())


def _layers(sizes, g):
    """Uniform(+-1/sqrt(fan_in)) weights and biases, in layer order."""
    ws, bs = [], []
    for fi, fo in zip(sizes[:-1], sizes[1:]):
        k = 1.0 / math.sqrt(fi)
        ws.append((2 * torch.rand((fo, fi), generator=g, device=DEV) - 1) * k)
        bs.append((2 * torch.rand(fo, generator=g, device=DEV) - 1) * k)
    return ws, bs


def _features(case, g):
    """(feature argument, [P][8] values): row-major, or planes as the image has them."""
    P = case["P"]
    if not case.get("planar", True):
        f = torch.randn((P, 8), generator=g, device=DEV)
        return D.rowmajor_features(f), f
    planes = torch.randn((12, P), generator=g, device=DEV)   # RGB | 8 semantic | u
    return (planes.view(-1)[3 * P:], P, P, 1), planes[3:11].t()


def _opts(case):
    return R.opts(tile=case["tile"], lds_batch=case["lds_batch"], persistent=case["persistent"],
                  ids_only=case["ids_only"])


def _target(case, cams, g):
    out = []
    for c in cams:
        t = torch.randn((case["C"], c.h * c.w), generator=g, device=DEV)
        t[:3].uniform_(generator=g)
        t[-1].zero_()
        out.append(t.view(-1))
    return torch.cat(out)


LR_LATE = 1e-4   # the step size of late training: repeated passes stay near the drawn scene


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed + 7919)
    if kind in ("render", "grad", "train"):
        cams, p = _cameras(case, seed), _scene(case, seed)
        s = dict(kind=kind, p=p)
        if kind == "train":
            s["step"] = TrainStep(cams, p, _target(case, cams, g), case["C"] - 4, o=_opts(case), lr=LR_LATE,
                                  capacity_slack=1.3)
            return s
        s["rast"] = R.Rasterizer(cams, _opts(case))
        if kind == "grad":
            for t in p.values():
                t.requires_grad_(True)
            s["d_out"] = torch.randn(case["C"] * sum(c.w * c.h for c in cams), generator=g, device=DEV)
        return s
    ctx = R.Context(0)
    if kind == "decode":
        f, values = _features(case, g)
        s = dict(kind=kind, ctx=ctx, f=f, K=case["K"], probs=case["outputs"] == "probs", how=case["how"],
                 normalize=case["normalize"])
        if case["how"] in ("mlp", "table3"):
            s["ws"], s["bs"] = _layers((8, 64, 64, case["K"]) if case["how"] == "mlp" else (8, 128, 256, case["K"]), g)
            s["params"] = D.mlp_pack(s["ws"], s["bs"])
        else:
            s["proj"] = torch.randn((512, 8), generator=g, device=DEV) / math.sqrt(8.0)
            cb = torch.randn((case["K"], 512), generator=g, device=DEV)
            s["codebook"] = (cb / cb.norm(dim=1, keepdim=True)).contiguous()
            if case["how"] == "folded":
                s["folded"] = D.decode_fold(ctx, s["proj"], s["codebook"])
        return s
    if kind == "language":
        f, values = _features(case, g)
        ws, bs = _layers((8, 128, 256, case["K"]), g)
        S = torch.randn((case["K"], case["d"]), generator=g, device=DEV)
        return dict(kind=kind, ctx=ctx, f=f, ws=ws, bs=bs, params=D.mlp_pack(ws, bs), K=case["K"],
                    S=(S / S.norm(dim=1, keepdim=True)).contiguous(), half=case["half"])
    if kind == "quantize":
        d = case["d_clip"] + case["d_dino"]
        S = torch.randn((case["K"], d), generator=g, device=DEV)
        at = torch.randint(0, case["K"], (case["P"],), generator=g, device=DEV)
        feat = torch.empty((case["P"], d), dtype=torch.float16, device=DEV)
        for i in range(0, case["P"], 1 << 17):   # features scattered around the codes
            k = at[i:i + (1 << 17)]
            feat[i:i + (1 << 17)] = S[k] + 1.5 * torch.randn((k.numel(), d), generator=g, device=DEV)
        ws = int(R.L.lib().legs_quantize_workspace_bytes(case["P"], case["K"], d))
        return dict(kind=kind, ctx=ctx, feat=feat, S=S, d_clip=case["d_clip"], grad=case["grad"],
                    workspace=torch.empty(max(ws, 16), dtype=torch.uint8, device=DEV))
    if kind == "smooth":
        p = _scene(dict(case, scene="rig"), seed)
        ws, bs = _layers((3, 128, 128, 128, 8), g)
        return dict(kind=kind, ctx=ctx, p=p, ws=ws, bs=bs, params=D.mlp_pack(ws, bs),
                    workspace=D.smooth_workspace(ctx, case["n"]), grad=torch.zeros(D.smooth_param_count(), device=DEV),
                    d_channels=torch.zeros_like(p["channels"]), loss=torch.zeros(1, device=DEV))
    K, P = case["K"], case["P"]
    ws, bs = _layers((8, 64, 64, K), g)
    labels = torch.randint(0, K, (P,), generator=g, device=DEV, dtype=torch.int32)
    if kind == "fit":
        f = torch.randn((P, 8), generator=g, device=DEV)
        return dict(kind=kind, f=D.rowmajor_features(f), labels=labels, ws=ws, bs=bs,
                    trainer=D.MlpTrainer(ctx, D.mlp_pack(ws, bs), K, P, normalize=case["normalize"]))
    planes = torch.randn((12, P), generator=g, device=DEV)
    planes[11].uniform_(generator=g)
    return dict(kind=kind, ctx=ctx, planes=planes, labels=labels, ws=ws, bs=bs, params=D.mlp_pack(ws, bs), K=K,
                normalize=case["normalize"], workspace=D.workspace(ctx, P, K),
                grad=torch.zeros(D.mlp_param_count(K), device=DEV), loss=torch.zeros(1, device=DEV),
                d_out=torch.zeros_like(planes))


# ---- one pass --------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "render":
        p = s["p"]
        _, _, out, T, _ = s["rast"].forward(p["mean"], p["log_scale"], p["quat"], p["opacity_logit"], p["channels"])
        return dict(out=out, T=T)
    if kind == "grad":
        p = s["p"]
        out, T = R.rasterize(p["mean"], p["log_scale"], p["quat"], p["opacity_logit"], p["channels"], s["rast"])
        grads = torch.autograd.grad(out, [p[k] for k in PARAMS], s["d_out"])
        return dict(out=out.detach(), T=T, grads=dict(zip(PARAMS, grads)))
    if kind == "train":
        t = s["step"]
        loss = t.step()
        return dict(loss=loss, grads=dict(t.g), params={k: t.p[k] for k in GROUPS})
    if kind == "decode":
        if s["how"] == "mlp":
            codes, probs = D.decode_mlp(s["ctx"], s["f"], s["params"], s["K"], probs=s["probs"],
                                        normalize=s["normalize"])
        elif s["how"] == "table3":
            codes, probs, _ = D.decode_dmlp(s["ctx"], s["f"], s["params"], s["K"], probs=s["probs"],
                                            normalize=s["normalize"])
        elif s["how"] == "folded":
            codes, probs = D.decode_folded(s["ctx"], s["f"], s["folded"], s["K"], probs=s["probs"])
        else:
            codes, probs = D.decode_plain(s["ctx"], s["f"], s["proj"], s["codebook"], probs=s["probs"])
        return dict(codes=codes, probs=probs)
    if kind == "language":
        _, _, M = D.decode_dmlp(s["ctx"], s["f"], s["params"], s["K"], probs_f16=True, top1=False)
        return dict(M=M, F=D.language_features(s["ctx"], M, s["S"], out_f16=s["half"]))
    if kind == "quantize":
        return D.quantize(s["ctx"], s["feat"], s["S"], s["d_clip"], grad=s["grad"], workspace=s["workspace"])
    if kind == "smooth":
        for k in ("grad", "d_channels", "loss"):   # the call adds to these
            s[k].zero_()
        ch = s["p"]["channels"]
        D.smooth_loss_grad(s["ctx"], s["p"]["mean"], ch, 3, ch.shape[1] - 1, s["params"], s["grad"], s["d_channels"],
                           s["loss"], workspace=s["workspace"])
        return dict(loss=s["loss"], grad=s["grad"], d_channels=s["d_channels"])
    if kind == "fit":
        t = s["trainer"]
        loss = t.step(s["f"], s["labels"])
        return dict(loss=loss, grad=t.grad, params=t.params)
    P = s["planes"].shape[1]
    s["grad"].zero_()
    s["loss"].zero_()
    D.semantic_loss_grad(s["ctx"], (s["planes"][3:], P, P, 1), s["planes"][11], s["labels"], s["params"], s["K"],
                         1.0 / P, s["workspace"], s["grad"], (s["d_out"][3:], P, 1), s["d_out"][11], s["loss"],
                         normalize=s["normalize"])
    return dict(loss=s["loss"], grad=s["grad"], d_out=s["d_out"])


# ---- what a pass cannot do without ------------------------------------------------

def work(case):
    """Each input read once and each output written once; the products of the
    decoders. A renderer's arithmetic depends on the scene: a nominal 64 blended
    entries per pixel."""
    kind = case["kind"]
    if kind in ("render", "grad", "train"):
        n, C = case["n"], case["C"]
        if case["sizes"] == "rig":
            px = sum(w * h for w, h in (RIG_SIZES[3 * v % len(RIG_SIZES)] for v in range(case["views"])))
        else:
            px = case["views"] * case["width"] * case["height"]
        b = 4 * (n * (11 + C) + px * (C + 1))
        f = px * 64 * (20 + 2 * C)
        if kind == "grad":
            b += 4 * (px * C + n * (11 + C))
            f += px * 64 * (56 + 7 * C)
        elif kind == "train":
            b += 4 * (px * C + n * (11 + C) * 6)
            f += px * 64 * (56 + 7 * C)
        return dict(bytes=b, flops=f)
    if kind in ("decode", "language"):
        P, K = case["P"], case["K"]
        if kind == "language":
            o = 2 if case["half"] else 4
            return dict(bytes=P * (32 + 2 * K + o * case["d"]),
                        flops=2 * P * (8 * 128 + 128 * 256 + 256 * K + K * case["d"]))
        b = P * (32 + 4 + (4 * K if case["outputs"] == "probs" else 0))
        f = {"mlp": 8 * 64 + 64 * 64 + 64 * K, "table3": 8 * 128 + 128 * 256 + 256 * K, "folded": 8 * K + 64,
             "plain": 8 * 512 + 512 * K}[case["how"]]
        return dict(bytes=b, flops=2 * P * f)
    if kind == "quantize":
        d = case["d_clip"] + case["d_dino"]
        return dict(bytes=case["P"] * (2 * d + 4), flops=(4 if case["grad"] else 2) * case["P"] * case["K"] * d)
    if kind == "smooth":
        return dict(bytes=4 * case["n"] * (3 + 9 + case["C"]), flops=6 * case["n"] * (3 * 128 + 2 * 128 * 128 + 128 * 8))
    macs = 8 * 64 + 64 * 64 + 64 * case["K"]
    return dict(bytes=case["P"] * (36 if kind == "fit" else 76), flops=6 * case["P"] * macs)


# ---- the same results in 64 bits ---------------------------------------------------

A_MAX, A_MIN, T_MIN = (float(torch.tensor(v, dtype=torch.float32)) for v in (0.99, 1.0 / 255.0, 1e-4))


def _project64(p, cam):
    """Camera-space depth, 2D mean, conic, pixel box and opacity of every
    Gaussian in float64: EWA projection with 0.3 px^2 on the diagonal, the
    Jacobian at the mean clamped to 1.3 times the field of view, and the box
    |pixel centre - mean| <= ceil(3 sqrt(largest eigenvalue))."""
    W, H, fx, fy, cx, cy, rot, t = cam.as_tuple()
    Rm = torch.tensor(rot, dtype=torch.float64, device=DEV).view(3, 3)
    tc = p["mean"] @ Rm.t() + torch.tensor(t, dtype=torch.float64, device=DEV)
    x, y, z = tc.unbind(1)
    seen = z > 0.2
    zs = torch.where(seen, z, torch.ones_like(z))
    qw, qx, qy, qz = (p["quat"] / p["quat"].norm(dim=1, keepdim=True)).unbind(1)
    rq = torch.stack([1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                      2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                      2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)], 1).view(-1, 3, 3)
    M = rq * p["log_scale"].exp()[:, None, :]
    lx, ly = 1.3 * 0.5 * W / fx, 1.3 * 0.5 * H / fy
    u, v = (x / zs).clamp(-lx, lx), (y / zs).clamp(-ly, ly)
    T0 = (fx / zs)[:, None] * Rm[0] - (fx * u / zs)[:, None] * Rm[2]
    T1 = (fy / zs)[:, None] * Rm[1] - (fy * v / zs)[:, None] * Rm[2]
    A0, A1 = (T0[:, :, None] * M).sum(1), (T1[:, :, None] * M).sum(1)     # rows of J W R S
    a, b, c = (A0 * A0).sum(1) + 0.3, (A0 * A1).sum(1), (A1 * A1).sum(1) + 0.3
    det = a * c - b * b
    mx, my = fx * x / zs + cx, fy * y / zs + cy
    with torch.no_grad():
        r = torch.ceil(3 * torch.sqrt(0.5 * (a + c) + torch.sqrt((0.5 * (a - c)) ** 2 + b * b)))
        box = torch.stack([torch.ceil(mx - r - 0.5).clamp(min=0), torch.floor(mx + r - 0.5).clamp(max=W - 1),
                           torch.ceil(my - r - 0.5).clamp(min=0), torch.floor(my + r - 0.5).clamp(max=H - 1)], 1)
        ok = seen & (box[:, 0] <= box[:, 1]) & (box[:, 2] <= box[:, 3])
        order = torch.argsort(z.float(), stable=True)
        order = order[ok[order]]
    rec = torch.stack([mx, my, c / det, -b / det, a / det, torch.sigmoid(p["opacity_logit"])], 1)
    return rec, box, order


def _tile64(rec, ch, x0, y0, w, h, box):
    """Colours [h w][C] and transmittance of one block of pixels over its
    depth-ordered Gaussians."""
    px = x0 + torch.arange(w, dtype=torch.float64, device=DEV)
    py = y0 + torch.arange(h, dtype=torch.float64, device=DEV)
    dx = (rec[:, 0:1] - (px + 0.5))[:, None, :]
    dy = (rec[:, 1:2] - (py + 0.5))[:, :, None]
    A, B, Cc, op = (rec[:, k][:, None, None] for k in (2, 3, 4, 5))
    power = -0.5 * (A * dx * dx + Cc * dy * dy) - B * dx * dy
    alpha = (op * torch.exp(power.clamp(max=0))).clamp(max=A_MAX)
    with torch.no_grad():
        inx = (px >= box[:, 0:1]) & (px <= box[:, 1:2])
        iny = (py >= box[:, 2:3]) & (py <= box[:, 3:4])
        keep = inx[:, None, :] & iny[:, :, None] & (alpha >= A_MIN)
        kept = torch.where(keep, alpha, torch.zeros_like(alpha)).flatten(1)
        through = torch.cumprod(1 - kept, 0)
        blend = keep.flatten(1) & (through >= T_MIN)
    alpha = torch.where(blend, alpha.flatten(1), torch.zeros_like(kept))
    after = torch.cumprod(1 - alpha, 0)
    before = torch.cat([torch.ones_like(after[:1]), after[:-1]])
    return (alpha * before).t() @ ch, after[-1]


def _render64(p, cams, C, d_out=None, block=32):
    """(out, T, gradient leaves): with d_out (a function of the image in 64
    bits) the gradients of sum(out * d_out) reach the parameters' .grad."""
    outs, Ts = [], []
    for v, cam in enumerate(cams):
        rec, box, order = _project64(p, cam)
        r2 = rec[order].detach().requires_grad_(d_out is not None)
        ch = p["channels"].detach()
        cacc = torch.zeros_like(ch)
        bx = box[order]
        out = torch.zeros((C, cam.h, cam.w), dtype=torch.float64, device=DEV)
        T = torch.ones((cam.h, cam.w), dtype=torch.float64, device=DEV)
        jobs = []
        for y0 in range(0, cam.h, block):
            iny = (bx[:, 2] < y0 + block) & (bx[:, 3] >= y0)
            for x0 in range(0, cam.w, block):
                idx = torch.nonzero(iny & (bx[:, 0] < x0 + block) & (bx[:, 1] >= x0)).flatten()
                if idx.numel():
                    jobs.append((x0, y0, min(block, cam.w - x0), min(block, cam.h - y0), idx))
        with torch.no_grad():
            for x0, y0, w, h, idx in jobs:
                col, t = _tile64(r2[idx], ch[order[idx]], x0, y0, w, h, bx[idx])
                out[:, y0:y0 + h, x0:x0 + w] = col.t().reshape(C, h, w)
                T[y0:y0 + h, x0:x0 + w] = t.view(h, w)
        if d_out is not None:
            G = d_out(v, out)
            racc = torch.zeros_like(r2)
            for x0, y0, w, h, idx in jobs:
                rt, ct = r2[idx].detach().requires_grad_(True), ch[order[idx]].requires_grad_(True)
                col, _ = _tile64(rt, ct, x0, y0, w, h, bx[idx])
                gr, gc = torch.autograd.grad(col, (rt, ct), G[:, y0:y0 + h, x0:x0 + w].reshape(C, -1).t())
                racc.index_add_(0, idx, gr)
                cacc.index_add_(0, order[idx], gc)
            torch.autograd.backward(rec, torch.zeros_like(rec).index_copy_(0, order, racc))
            p["channels"].grad = cacc if p["channels"].grad is None else p["channels"].grad + cacc
        outs.append(out.reshape(-1))
        Ts.append(T.reshape(-1))
    return torch.cat(outs), torch.cat(Ts)


def _bf16(x):
    """Nearest bfloat16 of float64 values (ties to even), in float64."""
    m, e = torch.frexp(x)
    return torch.ldexp(torch.round(torch.ldexp(m, torch.tensor(8, device=x.device))), e - 8)


def _mlp64(x, ws, bs, round_input=True):
    """The layers with bf16 weights and activations and 64-bit sums: (inputs of
    each layer, logits)."""
    h = _bf16(x) if round_input else x
    hs = [h]
    for i, (w, b) in enumerate(zip(ws, bs)):
        z = h @ _bf16(w.double()).t() + b.double()
        if i + 1 < len(ws):
            h = _bf16(z.clamp(min=0))
            hs.append(h)
    return hs, z


def _mlp_back64(dz, hs, ws):
    """Packed parameter gradient and the gradient at the input, straight through the roundings."""
    parts = []
    for i in range(len(ws) - 1, -1, -1):
        parts = [(dz.t() @ hs[i]).reshape(-1), dz.sum(0)] + parts
        dz = dz @ _bf16(ws[i].double())
        if i:
            dz = dz * (hs[i] > 0)
    return torch.cat(parts), dz


def _unit(f):
    n = f.norm(dim=1, keepdim=True)
    return f / torch.where(n > 0, n, torch.ones_like(n)), n


def _chunks(P, step=1 << 18):
    return [slice(i, min(P, i + step)) for i in range(0, P, step)]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("render", "grad", "train"):
        cams = _cameras(case, seed)
        px = sum(c.w * c.h for c in cams)
        if px * case["n"] > (3e11 if kind == "render" else 4e10):
            return None      # more than some seconds
        p = {k: v.double().requires_grad_(kind != "render") for k, v in _scene(case, seed).items()}
        C = case["C"]
        if kind == "render":
            out, T = _render64(p, cams, C)
            return dict(out=out, T=T)
        g = _gen(seed + 7919)
        if kind == "grad":
            flat = torch.randn(C * px, generator=g, device=DEV).double()
            at = [0]
            for c in cams:
                at.append(at[-1] + C * c.w * c.h)
            out, T = _render64(p, cams, C, lambda v, o: flat[at[v]:at[v + 1]].view_as(o))
            return dict(out=out, T=T, grads={k: p[k].grad for k in PARAMS})
        target, loss, at = _target(case, cams, g).double(), [], [0]
        for c in cams:
            at.append(at[-1] + C * c.w * c.h)

        def l1(v, o):
            hw = cams[v].w * cams[v].h
            t = target[at[v]:at[v + 1]].view_as(o)
            d = (o - t)[:C - 1]
            loss.append(d.abs().sum() / ((C - 1) * hw) + o[C - 1].sum() / hw)
            return torch.cat([d.sign() / ((C - 1) * hw), torch.full_like(o[C - 1:], 1.0 / hw)])
        _render64(p, cams, C, l1)
        # the projected records' gradients and the parameters after the step (a sign at the first one) have no value here
        return dict(loss=sum(loss).view(1), grads=dict(grad2d=None, **{k: p[k].grad for k in PARAMS}),
                    params={k: None for k in GROUPS})
    s = prepare(case, seed)
    if kind in ("decode", "language"):
        f, P, cs, ps = s["f"]
        x = torch.as_strided(f, (P, 8), (ps, cs))
        if kind == "language":
            M = torch.empty((P, case["K"]), dtype=torch.float64, device=DEV)
            for c in _chunks(P):
                M[c] = torch.softmax(_mlp64(x[c].double(), s["ws"], s["bs"])[1], 1)
            if P * case["d"] > 1_000_000_000:
                return None
            F = torch.empty((case["d"], P), dtype=torch.float64, device=DEV)
            for c in _chunks(P):
                F[:, c] = s["S"].double().t() @ M[c].t()
            return dict(M=M, F=F)
        if case["outputs"] != "probs":
            return None          # codes alone
        probs = torch.empty((P, case["K"]), dtype=torch.float64, device=DEV)
        for c in _chunks(P):
            v = x[c].double()
            if case["how"] in ("mlp", "table3"):
                z = _mlp64(_unit(v)[0] if case["normalize"] else v, s["ws"], s["bs"])[1]
            else:
                z = _unit(v @ s["proj"].double().t())[0] @ _unit(s["codebook"].double())[0].t()
            probs[c] = torch.softmax(z, 1)
        return dict(codes=None, probs=probs)
    if kind == "quantize":
        K, P, dc, d = case["K"], case["P"], case["d_clip"], case["d_clip"] + case["d_dino"]
        S = s["S"].half().double()
        parts = ((slice(0, dc), 1.0), (slice(dc, d), 0.5))
        codes = [_unit(S[:, q]) for q, _ in parts]
        counts, psum, lcos = torch.zeros(K, device=DEV, dtype=torch.float64), 0.0, 0.0

        def cosines(c):
            F = s["feat"][c].double()
            us = [_unit(F[:, q])[0] for q, _ in parts]
            return us, [u @ e[0].t() for u, e in zip(us, codes)]
        for c in _chunks(P, 1 << 16):
            _, cos = cosines(c)
            Dm = cos[0] + 0.5 * cos[1]
            best, m = Dm.max(1)
            counts += torch.bincount(m, minlength=K)
            psum = psum + torch.softmax(Dm, 1).sum(0)
            lcos = lcos + (1.5 - best).sum()
        r, pm = counts / P, psum / P
        lc, lb = lcos / P, (r * pm).sum()
        out = dict(index=None, counts=None, prob_mean=pm, losses=torch.stack([lc, lb, lc + 0.5 * lb]), grad=None)
        if case["grad"]:
            gs = [torch.zeros((K, e[0].shape[1]), dtype=torch.float64, device=DEV) for e in codes]
            for c in _chunks(P, 1 << 16):
                us, cos = cosines(c)
                Dm = cos[0] + 0.5 * cos[1]
                sm = torch.softmax(Dm, 1)
                dD = 0.5 / P * sm * (r - (sm @ r)[:, None])
                dD.scatter_add_(1, Dm.argmax(1, keepdim=True), torch.full_like(Dm[:, :1], -1.0 / P))
                for g, u, co, e, (_, lam) in zip(gs, us, cos, codes, parts):
                    g += lam * (dD.t() @ u - (dD * co).sum(0)[:, None] * e[0]) / e[1]
            out["grad"] = torch.cat(gs, 1)
        return out
    if kind == "smooth":
        n, grad, loss = case["n"], 0.0, 0.0
        ch = s["p"]["channels"]
        dch = torch.zeros(ch.shape, dtype=torch.float64, device=DEV)
        for c in _chunks(n):
            hs, z = _mlp64(s["p"]["mean"][c].double(), s["ws"], s["bs"], round_input=False)
            diff = z - ch[c, 3:11].double()
            u, nrm = _unit(diff)
            wgt = ch[c, -1].double().clamp(min=float(torch.tensor(0.1, dtype=torch.float32)))
            loss = loss + (nrm[:, 0] * (1 + wgt)).sum() / n
            dch[c, 3:11] = -(wgt / n)[:, None] * u
            grad = grad + _mlp_back64(u / n, hs, s["ws"])[0]
        return dict(loss=loss.view(1), grad=grad, d_channels=dch)
    P, K = case["P"], case["K"]
    x = (s["f"][0] if kind == "fit" else s["planes"][3:11].t())
    grad, loss = 0.0, 0.0
    d_out = None if kind == "fit" else torch.zeros((12, P), dtype=torch.float64, device=DEV)
    for c in _chunks(P):
        v = x[c].double()
        u, nrm = _unit(v)
        hs, z = _mlp64(u if case["normalize"] else v, s["ws"], s["bs"])
        lp = torch.log_softmax(z, 1)
        y = s["labels"][c].long()[:, None]
        ce = -lp.gather(1, y)[:, 0]
        ru = None if kind == "fit" else s["planes"][11, c].double()
        wpx = torch.full_like(ce, 1.0 / P) if kind == "fit" else (1 - ru) / P
        loss = loss + (wpx * ce).sum() + (0 if kind == "fit" else ru.sum() / P)
        dz = lp.exp().scatter_add(1, y, -torch.ones_like(lp[:, :1])) * wpx[:, None]
        gr, dh = _mlp_back64(dz, hs, s["ws"])
        grad = grad + gr
        if kind != "fit":
            if case["normalize"]:
                dh = (dh - (dh * u).sum(1, keepdim=True) * u) / nrm
            d_out[3:11, c] = dh.t()
            d_out[11, c] = (1 - ce) / P
    out = dict(loss=loss.view(1), grad=grad)
    if kind == "fit":
        return dict(out, params=None)   # a sign at the first step
    return dict(out, d_out=d_out)

"""The workloads this package is measured on: rendering, the rasterizer's forward + backward step, whole training
iterations and the multi-view score pass, from a few thousand Gaussians to three million.

`listed()` names twelve of them, `draw(rng)` makes more over the same ranges.  A case is a dict of plain values:

    kind        render   preprocess + bin_sort + render_fwd, as a viewer or a test-time evaluation calls them
                step     preprocess + bin_sort + render_fwd_loss + render_bwd + mask_score_fused, outputs allocated once
                train    Trainer.step: activations, the path, photometric loss, absolute gradient, Adam
                score    Trainer.score_views: error masks and counts of `views` views, summed, and the pruning score
    gaussians, sh, width, height
    views       cameras (1 except for score)
    compact     pairs from the Compact Box (the method's own rule) instead of the 3-sigma square
    scale_mean, scale_sd    of the logarithm of the Gaussians' scales
    late        train: iteration 16 000, where the method sums 32 iterations' gradients before an Adam update

Scenes are drawn on the GPU from the seed alone with the recipes of paper_2511_04283_amd/scenes.py: anisotropic clusters
inside (and a little outside) the frustum for one camera, clusters round the origin for cameras on an arc; opacities
sigmoid(N(0, 1.5)), SH coefficients N(0, 0.5) and N(0, 0.05); target images U[0, 1].
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_04283_amd import binding as B
from paper_2511_04283_amd import scenes
from paper_2511_04283_amd.trainer import TrainConfig, Trainer

DEVICE = "cuda:0"


def _case(kind, gaussians, sh, width, height, compact, scale_mean, scale_sd, views=1, late=False, name=None):
    c = dict(kind=kind, gaussians=gaussians, sh=sh, width=width, height=height, views=views, compact=compact,
             scale_mean=scale_mean, scale_sd=scale_sd, late=late)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest frame: a thumbnail of a small scene, where launches and the one read-back are all there is
        _case("render", 4096, 0, 128, 128, False, -3.5, 0.3, name="render_4k_128"),
        # a novel view of a trained scene at evaluation resolution (frames per second at test time)
        _case("render", 300_000, 3, 1332, 876, True, -4.0, 0.5, name="render_300k_1332x876_cb"),
        # the rasterizer's step at the five benchmark sizes: a unit-test-sized scene ...
        _case("step", 4096, 0, 128, 128, False, -3.5, 0.3, name="step_4k_128"),
        # ... an indoor scene early in training (odd image height: the last row of tiles is one pixel high)
        _case("step", 100_000, 3, 980, 545, False, -4.0, 0.5, name="step_100k_980x545"),
        # ... the headline: a trained outdoor scene, footprints from below a pixel to tens of tiles
        _case("step", 500_000, 3, 1600, 1064, False, -4.5, 0.7, name="step_500k_1600x1064"),
        # ... a dense unpruned model, 10 M pairs
        _case("step", 3_000_000, 3, 1920, 1080, False, -5.0, 0.8, name="step_3m_1920x1080"),
        # ... and the same with a heavy tail of large splats: tens of millions of pairs, lists of thousands
        _case("step", 3_000_000, 3, 1920, 1080, False, -5.0, 1.2, name="step_3m_wide_1920x1080"),
        # a whole training iteration on a sparse start: low resolution, low SH degree, odd sizes throughout
        _case("train", 12_347, 1, 509, 337, True, -3.7, 0.4, name="train_12k_509x337"),
        # a whole training iteration in the densification phase (an Adam update every iteration)
        _case("train", 500_000, 3, 1600, 1064, True, -4.5, 0.7, name="train_500k_1600x1064"),
        # ... and in the last third of the schedule, where gradients are summed between updates
        _case("train", 300_000, 3, 1332, 876, True, -4.0, 0.5, late=True, name="train_300k_1332x876_late"),
        # the multi-view consistency pass over ten sampled views
        _case("score", 300_000, 3, 1332, 876, False, -4.0, 0.5, views=10, name="score_300k_10x1332x876"),
        # ... and of a scene that is still growing, in the method's own pair rule
        _case("score", 100_000, 3, 980, 545, True, -4.0, 0.5, views=10, name="score_100k_10x980x545_cb"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["render", "render", "step", "step", "train", "train", "score"])
    most = {"render": 3e6, "step": 3e6, "train": 1e6, "score": 3e5}[kind]
    n = int(_log_uniform(rng, 3e3, most))
    # images hold between two thirds of a pixel and ten pixels per Gaussian, as in the benchmark sizes; any aspect ratio
    # between upright and wide
    pixels = min(1920 * 1080, max(96 * 96, n / _log_uniform(rng, 0.1, 1.5)))
    aspect = rng.uniform(0.7, 1.9)
    width, height = int(math.sqrt(pixels * aspect)), int(math.sqrt(pixels / aspect))
    # the more Gaussians, the smaller and the more varied they are (N(-3.5, 0.3) at 4 k, N(-5, 0.8) at 3 M)
    x = min(1.0, max(0.0, math.log(n / 4096) / math.log(3e6 / 4096)))
    scale_sd = 0.3 + 0.5 * x
    if kind in ("render", "step") and rng.random() < 0.15:
        scale_sd *= 1.5
    views = rng.randint(2, 10) if kind == "score" else 1
    # the late schedule draws from the same sizes as the early one; the Compact Box is the method's default
    return _case(kind, n, rng.choice([0, 1, 2, 3, 3, 3]), width, height, rng.random() < 0.6,
                 -3.5 - 1.5 * x + rng.uniform(-0.1, 0.1), scale_sd, views, kind == "train" and rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------------------------------
def _rotations(q):
    w, x, y, z = q.unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).view(-1, 3, 3)


def _scene(case, gen):
    """Activated parameters on the GPU; clusters as in scenes.config2 .. config5."""
    n, dev = case["gaussians"], torch.device(DEVICE)
    rand = lambda *s: torch.rand(s, device=dev, generator=gen)
    randn = lambda *s: torch.randn(s, device=dev, generator=gen)
    unit = lambda m: torch.nn.functional.normalize(randn(m, 4), dim=1)
    k = 32 if n < 200_000 else (64 if n < 1_000_000 else 256)
    if case["views"] > 1:
        centre = randn(k, 3) * torch.tensor([1.5, 1.0, 1.5], device=dev)
        spread = torch.full((k, 1), 3.0, device=dev) * (0.03 + 0.12 * rand(k, 3))
    else:
        half = 0.5 * torch.tensor([case["width"], case["height"]], device=dev) / (0.8 * case["width"])
        depth = 2.0 + 28.0 * rand(k, 1)
        centre = torch.cat([(2.0 * rand(k, 2) - 1.0) * 1.1 * half, torch.ones(k, 1, device=dev)], 1) * depth
        spread = depth * (0.02 + 0.10 * rand(k, 3))
    turn = _rotations(unit(k))
    which = torch.randint(0, k, (n,), device=dev, generator=gen)
    means = (turn[which] @ (randn(n, 3) * spread[which]).unsqueeze(-1)).squeeze(-1) + centre[which]
    scales = torch.exp(case["scale_mean"] + case["scale_sd"] * randn(n, 3))
    opacities = torch.sigmoid(1.5 * randn(n))
    sh = 0.05 * randn(n, (case["sh"] + 1) ** 2, 3)
    sh[:, 0] *= 10.0
    return means.contiguous(), scales, unit(n), opacities, sh


def _cameras(case):
    W, H, v = case["width"], case["height"], case["views"]
    f = 0.8 * W
    cams = []
    for j in range(v):
        a = math.radians(-15.0 + 30.0 * j / (v - 1)) if v > 1 else 0.0
        R = np.array([[math.cos(a), 0.0, math.sin(a)], [0.0, 1.0, 0.0], [-math.sin(a), 0.0, math.cos(a)]], np.float32)
        t = np.array([0.0, 0.0, 8.0 if v > 1 else 0.0], np.float32)   # on an arc: the origin eight units ahead
        cams.append(scenes.Camera(W, H, f, f, W / 2.0, H / 2.0, R, t))
    return cams


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    dev = torch.device(DEVICE)
    n, K, W, H = case["gaussians"], (case["sh"] + 1) ** 2, case["width"], case["height"]
    means, scales, quats, opacities, sh = _scene(case, gen)
    cams = _cameras(case)
    targets = [torch.rand((3, H, W), device=dev, generator=gen) for _ in cams] if case["kind"] != "render" else []
    config = B.default_config()
    config.compact_box = 1 if case["compact"] else 0
    ctx = B.Context(DEVICE, config)
    state = dict(kind=case["kind"], ctx=ctx, cams=cams, targets=targets)
    if case["kind"] in ("render", "step"):
        e = lambda *s, dt=torch.float32: torch.empty(s, dtype=dt, device=dev)
        state.update(g=B.Gaussians(means, scales, quats, opacities, sh, case["sh"]), cam=B.make_camera(cams[0]),
                     proj=B.Projected(e(n, 2), e(n), e(n, 4), e(n, 3), e(n, 4, dt=torch.int16), e(n, dt=torch.int32),
                                      e(n, 3, dt=torch.uint8)),
                     image=e(3, H, W), final_T=e(H, W), n_contrib=e(H, W, dt=torch.int32))
        if case["kind"] == "render":
            ctx.fs_set_score_record(False)   # no count pass follows
        else:
            state.update(dL=e(3, H, W), loss=torch.zeros(1, dtype=torch.float64, device=dev),
                         grads=dict(means=e(n, 3), scales=e(n, 3), quats=e(n, 4), opacities=e(n), sh=e(n, K, 3), mean2d=e(n, 2)),
                         mask=e(H, W, dt=torch.uint8), thr=e(1), counts=torch.zeros(n, dtype=torch.int32, device=dev))
        return state
    # a trainer in the middle of its run: the moments of many updates, and the learning rates they end with (every pass
    # changes the parameters, but little enough for one pass to be like the next)
    lr = dict(means=1e-5, sh=1e-5, raw_scales=1e-5, raw_quats=1e-5, raw_opacities=1e-5)
    trainer = Trainer(ctx, means, scales, quats, opacities, sh, case["sh"], TrainConfig(lr=lr, seed=int(seed) & 0x7fffffff))
    for k in trainer.p:
        trainer.m[k].normal_(0.0, 1e-7, generator=gen)
        trainer.v[k].uniform_(0.5e-14, 2e-14, generator=gen)
    trainer.iteration, trainer.updates = (16_000, 15_031) if case["late"] else (5_000, 5_000)
    state["trainer"] = trainer
    return state


# ---- one pass -----------------------------------------------------------------------------------------------------
def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind in ("render", "step"):
        s, cam, proj = state, state["cam"], state["proj"]
        ctx.fs_preprocess(s["g"], cam, proj)
        bins = ctx.fs_bin_sort(proj, cam)
        if kind == "render":
            ctx.fs_render_fwd(proj, bins, cam, s["image"], s["final_T"], s["n_contrib"])
            return dict(image=s["image"], final_T=s["final_T"], n_contrib=s["n_contrib"], pairs=bins.num_pairs)
        ctx.fs_render_fwd_loss(proj, bins, cam, s["targets"][0], s["image"], s["final_T"], s["n_contrib"], s["dL"], s["loss"])
        ctx.fs_render_bwd(s["g"], cam, proj, bins, s["final_T"], s["n_contrib"], s["dL"], s["grads"])
        s["counts"].zero_()
        ctx.fs_mask_score_fused(proj, bins, cam, s["n_contrib"], s["counts"], B.FS_MASK_MEAN_STD, 1.0, s["mask"], s["thr"])
        return dict(image=s["image"], final_T=s["final_T"], n_contrib=s["n_contrib"], loss=s["loss"], grads=s["grads"],
                    mask=s["mask"], threshold=s["thr"], counts=s["counts"], touched=proj.tiles_touched, pairs=bins.num_pairs)
    tr = state["trainer"]
    if kind == "train":
        loss = tr.step(state["cams"][0], state["targets"][0])
        return dict(loss=loss, p=tr.p, m=tr.m, v=tr.v, acc=tr.acc, grad_accum=tr.grad_accum, abs_accum=tr.abs_accum,
                    denom=tr.denom)
    counts, s_p = tr.score_views(state["cams"], state["targets"])
    return dict(counts=counts, s_p=s_p)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def work(case):
    """Bytes: parameters and targets read once, the projected splats (public outputs of fs_preprocess), images, gradients
    and state written once.  Flops: a pixel blends about 18 Gaussians of these scenes before it is opaque; 37 operations
    for each (distance, exponent, exponential, blend), 77 more for its gradient; the projection's 250 and the gradient's
    600 for each Gaussian; two separable 11-tap filters over the planes that SSIM needs (4 forward, 3 backward)."""
    n, K, px, v = case["gaussians"], (case["sh"] + 1) ** 2, case["width"] * case["height"], case["views"]
    params, projected, frame = 4 * (11 + 3 * K) * n, 55 * n, 20 * px
    blends = 18 * px
    render = dict(bytes=params + projected + frame, flops=250 * n + 37 * blends)
    if case["kind"] == "render":
        return render
    ssim_fwd, ssim_bwd = 3 * px * 4 * 44, 3 * px * 3 * 44
    if case["kind"] in ("step", "train"):
        b = render["bytes"] + 12 * px + 2 * params - 4 * n + 8 * n    # target; parameters again, gradients out
        f = render["flops"] + 600 * n + 77 * blends
        if case["kind"] == "step":
            return dict(bytes=b + 12 * px + px + 4 * n, flops=f)      # dL/dimage, mask, counts
        state = 2 * params if case["late"] else 6 * params            # acc, or m, v and the parameters: read and written
        return dict(bytes=b + state + 24 * n, flops=f + ssim_fwd + ssim_bwd + 15 * (11 + 3 * K) * n)
    return dict(bytes=v * (render["bytes"] + 12 * px + px + 4 * n) + 8 * n, flops=v * (render["flops"] + ssim_fwd))


def tolerance(case):
    """Integers (n_contrib, pairs, mask, counts) are the same in every correct implementation: the single-precision
    operations that decide them are fixed.  Gradients are single-precision sums over the pixels of terms that carry the
    rounding of a chain of up to a few hundred products (the transmittance), and go through the inverse of a 2x2 matrix:
    some 1e-5 as a whole, and a sum whose terms cancel is off by more of itself.  A training iteration starts from
    parameters that such gradients have moved, so a Gaussian at an edge may be visible in one more view or one fewer."""
    if case["kind"] == "render":
        return {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "step":
        return {"rel": 5e-5, "max": 5e-3}
    if case["kind"] == "train":
        return {"rel": 5e-5, "max": 5e-3, "differ": 1e-6}
    return {"rel": 1e-6, "max": 1e-5}

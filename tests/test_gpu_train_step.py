"""fs_train_step against the calls it stands for, one after the other on copies of the same state: every array of the state bit
for bit the same (the arithmetic is the same, operation by operation) over iterations with an update each, iterations that only
sum, and the update on the sum, for every SH degree, both pair rules, dense and sparse records, and counts of
Gaussians off the wavefront, the workgroup and the 16-byte row."""
import numpy as np
import pytest

from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu
LR = dict(means=1e-3, sh=2e-3, raw_scales=5e-3, raw_quats=1e-3, raw_opacities=5e-2)


SCHEDULE = [(False, True), (False, True), (True, False), (True, False), (True, True), (False, True)]   # (sums, update)


def compare_with_the_calls(c, sc, deg, views):
    """A training iteration per (camera, sums, update), each way on its own copy of the state; the statistics' view counts."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd.trainer import GROUPS, TrainConfig, Trainer
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(c.device)
    tr = Trainer(c, t(sc.means), t(sc.scales), t(sc.quats * 1.7), t(sc.opacities), t(sc.sh), deg, TrainConfig(lr=LR, eps=1e-8))
    copy = lambda d: {k: v.clone() for k, v in d.items()}
    p, m, v, acc = copy(tr.p), copy(tr.m), copy(tr.v), copy(tr.acc)
    ga, aa, den = tr.grad_accum.clone(), tr.abs_accum.clone(), tr.denom.clone()
    updates = 0
    for it, (cam, sums, update) in enumerate(views):
        fcam = B.make_camera(cam)
        target = t(np.random.default_rng(sc.n).uniform(0, 1, (3, cam.height, cam.width)))
        s, q, o = c.fs_activate(p["raw_scales"], p["raw_quats"], p["raw_opacities"])
        g = B.Gaussians(p["means"], s, q, o, p["sh"], deg)
        proj = c.fs_preprocess(g, fcam)
        bins = c.fs_bin_sort(proj, fcam)
        image, fT, nc = c.fs_render_fwd(proj, bins, fcam)
        out3, dL = c.fs_photo_loss(image, target, 0.2)
        gr = c.fs_render_bwd(g, fcam, proj, bins, fT, nc, dL, want_abs=True)
        c.fs_densify_accumulate(gr["mean2d"], gr["mean2d_abs"], proj.tiles_touched, ga, aa, den)
        c.fs_activate_bwd(p["raw_scales"], p["raw_quats"], p["raw_opacities"], gr["scales"], gr["quats"], gr["opacities"])
        grads = dict(zip(GROUPS, (gr["means"], gr["sh"], gr["scales"], gr["quats"], gr["opacities"])))
        for k in GROUPS:
            if sums:
                c.fs_grad_accumulate(acc[k], grads[k])
            if update:
                c.fs_adam_step(p[k], acc[k] if sums else grads[k], m[k], v[k], updates + 1, LR[k], eps=1e-8, zero_grad=sums)
        got = c.fs_train_step(fcam, target, deg, *[[d[k] for k in GROUPS] for d in (tr.p, tr.m, tr.v, tr.acc)], tr.grad_accum,
                              tr.abs_accum, tr.denom, [LR[k] for k in GROUPS], eps=1e-8, step=updates + 1, sum=sums,
                              update=update)
        updates += update
        assert list(got) == out3.tolist(), it
        for a, b in ((tr.p, p), (tr.m, m), (tr.v, v), (tr.acc, acc)):
            for k in GROUPS:
                assert torch.equal(a[k], b[k]), (it, k)
        assert torch.equal(tr.grad_accum, ga) and torch.equal(tr.abs_accum, aa) and torch.equal(tr.denom, den), it
    return den


def context(compact, records):
    from paper_2511_04283_amd import binding as B
    cfg = B.default_config()
    cfg.compact_box = compact
    c = B.Context("cuda:0", cfg)
    c.fs_set_record_mode(B.FS_RECORDS_DENSE if records == "dense" else B.FS_RECORDS_SPARSE)
    return c


@pytest.mark.parametrize("compact,records", [(1, "dense"), (0, "sparse"), (1, "sparse"), (0, "dense")])
@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 33, 97, 611])
def test_train_step_equals_the_calls_it_replaces(n, deg, compact, records):
    c = context(compact, records)
    sc = scenes.tiny_scene(40 + n, n, 83, 50, sh_degree=deg, log_scale=(-2.3, 0.6), spread=1.3)
    den = compare_with_the_calls(c, sc, deg, [(sc.cameras[0], *it) for it in SCHEDULE])
    assert int(den.max().item()) == 6
    c.close()


@pytest.mark.parametrize("compact,records", [(1, "dense"), (0, "sparse"), (1, "sparse"), (0, "dense")])
@pytest.mark.parametrize("n", [0, 97])
def test_train_step_where_nothing_is_visible(n, compact, records):
    """No Gaussians at all, and views that see none of them, first and between others that do (moments decay and parameters
    move on all the same)."""
    c = context(compact, records)
    sc = scenes.tiny_scene(70, 97, 83, 50, sh_degree=1, log_scale=(-2.3, 0.6), spread=1.3)
    cam = sc.cameras[0]
    away = scenes.Camera(cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy, cam.R, cam.t - np.array([0, 0, 100.0], np.float32))
    if n == 0:
        sc = scenes.Scene("empty", 1, *(a[:0] for a in (sc.means, sc.scales, sc.quats, sc.opacities, sc.sh)), [cam], 0)
    den = compare_with_the_calls(c, sc, 1, [(away, *SCHEDULE[0])] + [(k, *it) for it in SCHEDULE for k in (cam, away)])
    assert den.numel() == n and (n == 0 or int(den.max().item()) == 6)
    c.close()


@pytest.mark.parametrize("compact,records", [(1, "dense"), (0, "sparse"), (1, "sparse"), (0, "dense")])
def test_train_step_on_frames_and_lists_that_grow(compact, records):
    """Frames of other sizes on one context, each with more pairs than its buffers hold, and back: they grow within an
    iteration."""
    c = context(compact, records)
    sc = scenes.tiny_scene(71, 611, 83, 50, sh_degree=2, log_scale=(-2.3, 0.6), spread=1.3)
    cam = sc.cameras[0]
    sized = lambda k: scenes.Camera(int(k * cam.width), int(k * cam.height), k * cam.fx, k * cam.fy, k * cam.cx, k * cam.cy, cam.R, cam.t)
    compare_with_the_calls(c, sc, 2, [(sized(k), *it) for k, it in zip((0.3, 1.0, 2.7, 6.1, 0.5, 2.7), SCHEDULE)])
    c.close()


@pytest.mark.parametrize("compact,records", [(1, "dense"), (0, "sparse"), (1, "sparse"), (0, "dense")])
@pytest.mark.parametrize("n, width, height, scale", [(16385, 83, 50, -3.2), (611, 650, 480, -2.3), (16384, 83, 50, -3.2), (16384, 40, 33, -1.2)])
def test_train_step_by_general_launches_and_by_the_largest_one_launch(n, width, height, scale, compact, records):
    """An iteration orders its pairs in one launch up to 16384 Gaussians and 1024 tiles, where the separate calls have left it: one more of
    either, and the most of it, with lists beyond 8192 entries as well."""
    from paper_2511_04283_amd import binding as B
    c = context(compact, records)
    sc = scenes.tiny_scene(72, n, width, height, sh_degree=1, log_scale=(scale, 0.5), spread=1.0)
    cam = sc.cameras[0]
    bins = c.fs_bin_sort(c.fs_preprocess(B.Gaussians.from_scene(sc, c.device), B.make_camera(cam)), B.make_camera(cam))
    ranges = bins.copy_ranges()
    longest = int((ranges[:, 1] - ranges[:, 0]).max().item())
    assert (8192 < longest <= n) if scale > -2 else longest > 0, longest
    compare_with_the_calls(c, sc, 1, [(cam, *it) for it in SCHEDULE[:1] + SCHEDULE[2:5]])
    c.close()


@pytest.mark.parametrize("shape", [(1, 3, 50, 83), (3 * 50 * 83,)])
def test_target_of_another_shape_and_too_small_a_target(shape):
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd.trainer import TrainConfig, Trainer
    c = B.Context("cuda:0")
    sc = scenes.tiny_scene(44, 61, 83, 50, sh_degree=1, log_scale=(-2.3, 0.6), spread=1.3)
    cam = sc.cameras[0]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(c.device)
    target = t(np.random.default_rng(5).uniform(0, 1, (3, 50, 83)))
    make = lambda: Trainer(c, t(sc.means), t(sc.scales), t(sc.quats), t(sc.opacities), t(sc.sh), 1, TrainConfig(lr=LR))
    a, b = make(), make()
    assert a.step(cam, target) == b.step(cam, target.view(shape))
    for k in a.p:
        assert torch.equal(a.p[k], b.p[k]), k
    with pytest.raises(ValueError):   # refused on the host, before anything is enqueued
        b.step(cam, target[:2])
    assert (b.iteration, b.pending, b.updates) == (a.iteration, a.pending, a.updates) == (1, 0, 1)
    c.close()

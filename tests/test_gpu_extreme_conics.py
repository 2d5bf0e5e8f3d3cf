"""Conics at the end of the single-precision range (a caller's own fs_projected, or splats far below a pixel without a
low-pass): the exponent is minus infinity at most pixels, and nothing is blended there, as in the oracle.  Every user of the
exponential: the forward pass, both backward passes, the count pass from its record and by its two walks."""
import numpy as np
import pytest

from gpu_common import assert_grads_close, assert_image_close
from oracle import Oracle
from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [5.0e37, 1.5e38, 3.0e38, np.inf])
def test_exponent_of_minus_infinity_blends_nothing(size):
    import torch
    from paper_2511_04283_amd import binding as B
    sc = scenes.tiny_scene(321, 400, 61, 43, sh_degree=0, log_scale=(-2.5, 0.5), spread=1.0)
    sc.opacities[:] = np.random.default_rng(3).uniform(0.2, 0.9, sc.n)
    cam, fcam = sc.cameras[0], B.make_camera(sc.cameras[0])
    o = Oracle(np.float32)
    p = o.preprocess(sc, cam)
    huge = (np.arange(sc.n) % 3 == 0) & (p.tiles_touched > 0)
    assert huge.sum() > 40
    p.conic_opacity[huge, :3] = np.array([size, 0.0, size], np.float32)
    p.conic_opacity[huge & (np.arange(sc.n) % 2 == 0), 0] = 0.7   # (in one direction only)
    if np.isfinite(size):   # one whose centre is a pixel's: blended there and nowhere else
        assert huge[0]
        p.mean2d[0] = np.floor(p.mean2d[0]) + 0.5
        p.conic_opacity[0, :3] = np.array([size, 0.0, size], np.float32)
    b = o.bin_sort(p, cam)
    image, T, nc = o.render_fwd(p, b, cam)
    rng = np.random.default_rng(4)
    dL = rng.normal(size=(3, cam.height, cam.width)).astype(np.float32)

    c = B.Context("cuda:0")
    t = lambda a, dt=np.float32: torch.from_numpy(np.ascontiguousarray(a).astype(dt)).to(c.device)
    g = B.Gaussians.from_scene(sc, c.device)
    proj = B.Projected(t(p.mean2d), t(p.depth), t(p.conic_opacity), t(p.rgb), t(p.rect.astype(np.uint16).view(np.int16), np.int16),
                       t(p.tiles_touched, np.int32), t(p.clamped, np.uint8))
    bins = c.fs_bin_sort(proj, fcam)
    assert bins.num_pairs == b.num_pairs
    got = c.fs_render_fwd(proj, bins, fcam)
    assert np.array_equal(got[2].cpu().numpy().view(np.uint32), nc)
    assert_image_close(got[0].cpu().numpy(), image)
    for share in (0.9, 0.2):   # of the pixels in the mask: the walk has one path for crowded tiles and one for sparse ones
        mask = (rng.uniform(size=(cam.height, cam.width)) < share).astype(np.uint8)
        want = o.score(p, b, cam, mask, np.zeros(sc.n, np.int32))
        for record in (True, False):
            c.fs_set_score_record(record)
            image2, T2, nc2 = c.fs_render_fwd(proj, bins, fcam)
            counts = torch.zeros(sc.n, dtype=torch.int32, device=c.device)
            c.fs_score_accumulate(proj, bins, fcam, T2, nc2, t(mask, np.uint8), counts)
            assert np.array_equal(counts.cpu().numpy(), want), (share, record)
    # (an infinite conic has no gradient of its place: infinity times the zero it receives)
    d_mean2d, d_conic, d_op, d_rgb, d_abs = o.render_bwd(p, b, cam, dL)
    ref = dict(conic=d_conic, opacities=d_op, rgb=d_rgb)
    if size < 1.7e38:   # (twice the conic is finite)
        ref.update(mean2d=d_mean2d)
    if size < 1.0e38:   # (... and its product with the distances that get that far)
        ref.update(mean2d_abs=d_abs)
    for mode in (B.FS_BWD_PER_PIXEL, B.FS_BWD_PER_SPLAT):
        c.fs_set_backward_mode(mode)
        for want_abs in (False, True):
            gr = c.fs_render_bwd(g, fcam, proj, bins, got[1], got[2], t(dL), want_2d=True, want_abs=want_abs)
            grads = {k: v.cpu().numpy() for k, v in gr.items()}
            grads["mean2d"][0] = d_mean2d[0]
            assert_grads_close(grads, ref)
    c.close()

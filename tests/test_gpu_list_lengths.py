"""The render kernels' walks over the tile lists where their steps begin and end: groups of 4 entries (forward), exchanges of
8 (backward), batches of 207, 231 (backward with and without the absolute gradient) and 255 (forward).  Every Gaussian
covers the whole image of two ragged tiles and is faint, so that all of every list is blended; and the same with
small ones, whose sub-tile lists have every length up to a few.  Integers bit for bit, image and gradients within the
benchmark's bars (1e-4; 1e-3 with its floor) of the oracle."""
import numpy as np
import pytest

from gpu_common import assert_grads_close, assert_image_close, gpu_pipeline
from oracle import Config, Oracle
from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want_abs", [False, True])
@pytest.mark.parametrize("large", [True, False])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 207, 208, 231, 232, 255, 256, 463])
def test_list_of_n_entries(n, large, want_abs):
    from paper_2511_04283_amd import binding as B
    sc = scenes.tiny_scene(900 + n, n, 29, 13, sh_degree=0, log_scale=(-0.5, 0.2) if large else (-3.2, 0.5), spread=0.6)
    sc.opacities[:] = np.random.default_rng(n).uniform(0.006, 0.02, n) if large else 0.7
    cam = sc.cameras[0]
    dL = np.random.default_rng(n + 1).normal(size=(3, cam.height, cam.width)).astype(np.float32)
    c = B.Context("cuda:0")
    out = gpu_pipeline(c, sc, cam, dL=dL, want_abs=want_abs)
    c.close()
    o = Oracle(np.float32)
    p, b, image, T, nc = o.forward(sc, cam)
    assert out["num_pairs"] == b.num_pairs
    assert np.array_equal(out["n_contrib"], nc)
    assert_image_close(out["image"], image)
    assert_grads_close(out["grads"], o.backward(sc, cam, p, b, dL))


@pytest.mark.parametrize("want_abs", [False, True])
@pytest.mark.parametrize("every", [1, 5])
def test_needles_among_other_splats(every, want_abs):
    """Splats more than thirty times as long as wide have their second moments added up another way (k_render_bwd): all of
    the splats, or every fifth.  What the render pass itself leaves (the screen-space gradients) within the benchmark's
    bar; the scales' gradients are the small difference of large moments, to a few parts in 10^4 of the largest."""
    from paper_2511_04283_amd import binding as B
    sc = scenes.tiny_scene(77, 300, 150, 83, sh_degree=0, log_scale=(-3.0, 0.3), spread=1.0)
    sc.scales[::every] *= np.array([40.0, 0.02, 0.02], np.float32)
    sc.opacities[::every] = 0.3
    cam = sc.cameras[0]
    dL = np.random.default_rng(5).normal(size=(3, cam.height, cam.width)).astype(np.float32)
    c = B.Context("cuda:0")
    out = gpu_pipeline(c, sc, cam, dL=dL, want_abs=want_abs)
    c.close()
    o = Oracle(np.float32)
    p, b, image, T, nc = o.forward(sc, cam)
    co = p.conic_opacity.astype(np.float64)
    needles = (co[:, 0] + co[:, 2]) ** 2 > 1000.0 * (co[:, 0] * co[:, 2] - co[:, 1] ** 2)
    assert needles[p.tiles_touched > 0].sum() > (100 if every == 1 else 20)
    assert np.array_equal(out["n_contrib"], nc)
    ref = o.backward(sc, cam, p, b, dL)
    assert_grads_close(out["grads"], {k: ref[k] for k in ("conic", "mean2d", "rgb", "opacities", "sh") + (("mean2d_abs",) if want_abs else ())})
    for k in ("scales", "quats", "means"):
        assert np.linalg.norm(out["grads"][k] - ref[k]) <= 1e-3 * np.linalg.norm(ref[k]), k


@pytest.mark.parametrize("mode", ["weight", "alpha"])
@pytest.mark.parametrize("large", [True, False])
@pytest.mark.parametrize("n", [1, 4, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 320, 463])
def test_counts_of_n_entries(n, large, mode):
    """The record of counted pixels leaves the forward kernel's registers after every 64 places of a list and at its end, also where
    all pixels have stopped before it: the counts of such lists, from the record and from a second walk, against the oracle's."""
    from paper_2511_04283_amd import binding as B
    sc = scenes.tiny_scene(1900 + n, n, 29, 13, sh_degree=0, log_scale=(-0.5, 0.2) if large else (-3.2, 0.5), spread=0.6)
    sc.opacities[:] = np.random.default_rng(n).uniform(0.006, 0.12, n) if large else 0.7
    cam = sc.cameras[0]
    target = np.random.default_rng(n + 1).uniform(size=(3, cam.height, cam.width)).astype(np.float32)
    config = B.default_config()
    config.score_mode = B.FS_SCORE_WEIGHT if mode == "weight" else B.FS_SCORE_ALPHA
    c = B.Context("cuda:0", config)
    out = gpu_pipeline(c, sc, cam, target=target)   # (which compares the record's counts with the walk's)
    c.close()
    o = Oracle(np.float32, Config(score_mode=config.score_mode))
    p, b, image, T, nc = o.forward(sc, cam)
    mask, thr, _ = o.error_mask(image, target)
    assert np.array_equal(out["n_contrib"], nc)
    assert np.array_equal(out["mask"], mask)
    assert np.array_equal(out["counts"], o.score(p, b, cam, mask, np.zeros(n, np.int32)))

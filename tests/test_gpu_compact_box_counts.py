"""The Compact Box's tile counts where the wavefront deals the boxes' tiles out to its lanes: boxes of one tile beside
boxes of the whole image, runs that end at and across windows of 64, empty runs, Gaussian counts off the wavefront size."""
import numpy as np
import pytest

from oracle import Config, Oracle
from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 300])
@pytest.mark.parametrize("big_every", [1, 5, 40])
def test_counts_of_mixed_boxes(n, big_every):
    from paper_2511_04283_amd import binding as B
    cfg = B.default_config()
    cfg.compact_box = 1
    c = B.Context("cuda:0", cfg)
    sc = scenes.tiny_scene(70 + n, n, 520, 260, sh_degree=0, log_scale=(-4.0, 0.5), spread=1.3)
    sc.scales[::big_every] *= 60.0
    sc.opacities[3::7] = 0.003                         # below 1/255: no tile at all
    cam = sc.cameras[0]
    proj = c.fs_preprocess(B.Gaussians.from_scene(sc, c.device), B.make_camera(cam))
    p = Oracle(np.float32, Config(compact_box=True)).preprocess(sc, cam)
    assert np.array_equal(proj.tiles_touched.cpu().numpy().view(np.uint32), p.tiles_touched)
    assert np.array_equal(proj.rect.cpu().numpy().view(np.uint16).astype(np.int32), p.rect)
    c.close()

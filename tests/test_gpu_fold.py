"""The fused forward pass's loss and error statistics: the tiles' partials are folded by one workgroup per quantity."""
import numpy as np
import pytest

from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 63, 65, 1024, 1025, 8192, 8193])
def test_statistics_of_so_many_tiles(tiles):
    """One tile, around a wavefront, a workgroup and a round of eight loads: the loss in 64 bits (terms of one sign and fewer than 3e6, so
    1e-12 leaves room for any order of them), and threshold and mask as the separate calls give them, with either rule,
    also where nobody asks for the loss.  Every call has a target of its own: the statistics of none before it will do."""
    import torch
    from paper_2511_04283_amd import binding as B
    W, H = 16 * tiles - 3, 7
    sc = scenes.tiny_scene(tiles, 60, W, H, sh_degree=0)
    c = B.Context("cuda:0")
    cam = B.make_camera(sc.cameras[0])
    g = B.Gaussians.from_scene(sc, c.device)
    proj = c.fs_preprocess(g, cam)
    bins = c.fs_bin_sort(proj, cam)
    image = c.fs_render_fwd(proj, bins, cam)[0]
    rng = np.random.default_rng(tiles)
    for rule, k in ((0, 1.0), (1, 0.35)):
        for loss in (None, torch.full((1,), -1.0, dtype=torch.float64, device=c.device), None):
            target = torch.from_numpy(rng.uniform(size=(3, H, W)).astype(np.float32)).to(c.device)
            mask, threshold = c.fs_error_mask(image, target, rule, k)
            fused = c.fs_render_fwd_loss(proj, bins, cam, target, loss_out=loss)[0]
            mask_f, threshold_f = c.fs_error_mask_fused(H, W, rule, k)
            assert torch.equal(fused, image) and torch.equal(mask_f, mask) and threshold_f.item() == threshold.item()
            if loss is not None:
                want = np.abs(image.cpu().numpy() - target.cpu().numpy()).astype(np.float64).mean()
                assert abs(loss.item() - want) <= 1e-12 * want
    c.close()

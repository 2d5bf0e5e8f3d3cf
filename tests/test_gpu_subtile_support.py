"""Which sub-tiles a splat's support reaches (support_strips, strip_mask): a sub-tile too few and its pixels miss a factor of their
transmittance.  Ellipses of every shape, thickness and direction -- needles up to 1e6 times as long as wide (in variance) among
them -- with their ends anywhere in the image, opacities down to the least that is blended, against the oracle, to the bit."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest", [0.31, 3.0, 1.0e2, 1.0e4, 3.0e5])
@pytest.mark.parametrize("origin", [0, 3008])   # (where coordinates have their coarse steps, too)
def test_no_sub_tile_is_missed(longest, origin):
    import torch
    from paper_2511_04283_amd import binding as B
    n, W, H = 700, origin + 61, 77
    rng = np.random.default_rng(int(longest) + origin)
    l1 = 0.3 * np.exp(rng.uniform(0, np.log(longest / 0.3), n))
    l2 = np.where(rng.random(n) < 0.5, 0.3, 0.3 * np.exp(rng.random(n) * np.log(l1 / 0.3)))
    th = np.where(rng.random(n) < 0.3, rng.integers(0, 4, n) * np.pi / 4 + rng.normal(0, 0.02, n), rng.uniform(0, np.pi, n))
    c, s = np.cos(th), np.sin(th)
    conic = np.stack([c * c / l1 + s * s / l2, c * s * (1 / l1 - 1 / l2), s * s / l1 + c * c / l2], 1).astype(np.float32)
    sigma = np.where(rng.random(n) < 0.3, (1 + 0.2 * rng.random(n)) / 255, np.exp(rng.uniform(np.log(0.005), np.log(0.05), n)))
    # a point just inside or outside the support's border, or anywhere within, comes to lie in the image's last columns
    reach = np.sqrt(2 * np.log(np.maximum(255 * sigma, 1.0001))) * np.where(rng.random(n) < 0.6, rng.normal(1, 0.02, n), rng.random(n))
    phi = rng.uniform(0, 2 * np.pi, n)
    u, v = np.sqrt(l1) * reach * np.cos(phi), np.sqrt(l2) * reach * np.sin(phi)
    border = np.stack([c * u - s * v, s * u + c * v], 1)
    mu = (np.stack([origin + rng.uniform(0, 61, n), rng.uniform(0, 77, n)], 1) - border).astype(np.float32)
    cam = scenes.Camera(W, H, 0.8 * W, 0.8 * W, W / 2, H / 2, np.eye(3), np.zeros(3))
    sc = scenes.tiny_scene(1, n, W, H, sh_degree=0)
    o = Oracle(np.float32)
    p = o.preprocess(sc, cam)
    p.mean2d[:], p.depth[:], p.rgb[:] = mu, np.arange(1, n + 1), rng.uniform(0.2, 1, (n, 3))
    p.conic_opacity[:] = np.concatenate([conic, sigma[:, None]], 1)
    p.rect[:] = [origin // 16, 0, (W + 15) // 16, (H + 15) // 16]
    p.tiles_touched[:] = 4 * 5
    b = o.bin_sort(p, cam)
    image, T, nc = o.render_fwd(p, b, cam)
    assert (nc[:, origin:] > 0).mean() > 0.2

    ctx = B.Context("cuda:0")
    t = lambda a, dt=np.float32: torch.from_numpy(np.ascontiguousarray(a).astype(dt)).to(ctx.device)
    proj = B.Projected(t(p.mean2d), t(p.depth), t(p.conic_opacity), t(p.rgb), t(p.rect.astype(np.uint16).view(np.int16), np.int16),
                       t(p.tiles_touched, np.int32), t(p.clamped, np.uint8))
    fcam = B.make_camera(cam)
    bins = ctx.fs_bin_sort(proj, fcam)
    assert bins.num_pairs == n * 20
    got = [a.cpu().numpy() for a in ctx.fs_render_fwd(proj, bins, fcam)]
    ctx.close()
    assert np.array_equal(got[2].view(np.uint32), nc)
    assert np.array_equal(got[1].view(np.uint32), T.view(np.uint32))


def test_the_least_opacity_that_is_blended():
    """A splat of opacity alpha_min whose centre is a pixel's is blended there: the bound's own rounding of their ratio does not decide."""
    import torch
    from paper_2511_04283_amd import binding as B
    rng = np.random.default_rng(4)
    cam = B.make_camera(scenes.Camera(96, 16, 50.0, 50.0, 48.0, 8.0))
    for alpha_min in [1 / 255, *np.exp(rng.uniform(np.log(1e-4), np.log(0.5), 60))]:
        cfg = B.default_config()
        cfg.alpha_min = alpha_min
        ctx = B.Context("cuda:0", cfg)
        least = np.float32(cfg.alpha_min)
        sigma = np.array([np.nextafter(least, np.float32(0)), least, np.nextafter(least, np.float32(1)), least * np.float32(1.01)], np.float32)
        x0 = np.arange(4)
        t = lambda a, dt=np.float32: torch.from_numpy(np.ascontiguousarray(a).astype(dt)).to(ctx.device)
        proj = B.Projected(t(np.stack([16 * x0 + 5.5, np.full(4, 9.5)], 1)), t(np.ones(4)), t(np.stack([np.full(4, 0.7), 0 * x0, np.full(4, 0.7), sigma], 1)),
                           t(np.ones((4, 3))), t(np.stack([x0, 0 * x0, x0 + 1, 0 * x0 + 1], 1).astype(np.uint16).view(np.int16), np.int16),
                           t(np.ones(4), np.int32), t(np.zeros((4, 3)), np.uint8))
        nc = ctx.fs_render_fwd(proj, ctx.fs_bin_sort(proj, cam), cam)[2].cpu().numpy()
        ctx.close()
        assert nc[9, 16 * x0 + 5].tolist() == [0, 1, 1, 1], alpha_min

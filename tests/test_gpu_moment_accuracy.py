"""How far k_render_bwd's screen-space gradients of small splats are from exact sums over their pixels.  Every splat has a
tile to itself, so that what a pixel contributes is known to a rounding or two (its weight is replayed in single precision,
operation by operation) and the sums can be formed in 64 bits."""
import numpy as np
import pytest

from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu
f32 = np.float32


def fma(a, b, c):
    return (np.multiply(a, b, dtype=np.float64) + c).astype(f32)


def exp_c(x):
    """The kernels' exponential for x <= 0."""
    t = x * f32(float.fromhex("0x1.715476p+0"))
    n = np.rint(t)
    r, p = t - n, np.full_like(t, float.fromhex("0x1.5bba14p-10"))
    for c in ("0x1.3cea88p-7", "0x1.c6b752p-5", "0x1.ebf9bcp-3", "0x1.62e42ap-1", "0x1p0"):
        p = fma(p, r, f32(float.fromhex(c)))
    return np.ldexp(p, n.astype(np.int32))


def gradient_errors(B, eigenvalues, one_sign, want_abs, tiles=64):
    """The 2-norm of the difference over that of the exact gradients (mean2d: of its contributions' magnitudes): conic, mean2d,
    opacity, rgb, and with want_abs the absolute mean2d."""
    import torch
    rng = np.random.default_rng(int(1000 * eigenvalues[1]) + one_sign)
    n, W, H = tiles * 24, 16 * tiles, 16 * 24
    th, (l1, l2) = rng.uniform(0, np.pi, n), eigenvalues
    c, s = np.cos(th), np.sin(th)
    conic = np.stack([c * c / l2 + s * s / l1, c * s * (1 / l2 - 1 / l1), s * s / l2 + c * c / l1], 1)
    sigma = rng.uniform(0.3, 0.9, n)
    reach = np.sqrt(2 * np.log(255 * 0.9) * l2)   # (beyond it nothing is blended: a splat stays within its tile)
    assert reach < 7.9
    tx, ty = np.arange(n) % tiles, np.arange(n) // tiles
    mu = (np.stack([tx, ty], 1) * 16 + rng.uniform(reach, 16 - reach, (n, 2))).astype(f32)
    co = np.concatenate([conic, sigma[:, None]], 1).astype(f32)
    rgb = rng.uniform(0.2, 1.0, (n, 3)).astype(f32)
    rect = np.stack([tx, ty, tx + 1, ty + 1], 1)
    dL = np.zeros((3, H, W), f32)
    dL[0] = rng.normal(size=(H, W)) if not one_sign else rng.uniform(0.9, 1.1, (H, W))

    ctx = B.Context("cuda:0")
    t = lambda a, dt=f32: torch.from_numpy(np.ascontiguousarray(a).astype(dt)).to(ctx.device)
    proj = B.Projected(t(mu), t(np.ones(n)), t(co), t(rgb), t(rect.astype(np.uint16).view(np.int16), np.int16), t(np.ones(n), np.int32),
                       t(np.zeros(n), np.uint8))
    g = B.Gaussians(t(np.tile([0, 0, 5.0], (n, 1))), t(np.full((n, 3), 0.1)), t(np.tile([1.0, 0, 0, 0], (n, 1))), t(sigma), t(np.zeros((n, 1, 3))), 0)
    cam = B.make_camera(scenes.Camera(W, H, 0.8 * W, 0.8 * W, W / 2, H / 2, np.eye(3), np.zeros(3)))
    bins = ctx.fs_bin_sort(proj, cam)
    assert bins.num_pairs == n
    image, T, nc = ctx.fs_render_fwd(proj, bins, cam)
    gr = {k: v.cpu().numpy().astype(np.float64) for k, v in
          ctx.fs_render_bwd(g, cam, proj, bins, T, nc, t(dL), want_2d=True, want_abs=want_abs).items()}
    ctx.close()

    # [splat, line, column]
    X = (16 * tx[:, None, None] + np.arange(16)[None, None, :] + 0.5).astype(f32)
    Y = (16 * ty[:, None, None] + np.arange(16)[None, :, None] + 0.5).astype(f32)
    ax = lambda v: v[:, None, None]
    dx, dy = X - ax(mu[:, 0]), Y - ax(mu[:, 1])
    power = fma(dx, fma(-ax(co[:, 1]), dy, (f32(-0.5) * ax(co[:, 0])) * dx), ((f32(-0.5) * ax(co[:, 2])) * dy) * dy)
    G = exp_c(power)
    alpha = np.minimum(f32(0.99), ax(co[:, 3]) * G)
    on = (power <= 0) & (alpha >= f32(1.0 / 255.0))
    # (T is 1 in front of the only splat, nothing is behind it; alpha stays below the cap)
    d0 = dL[0].reshape(-1, 16, tiles, 16).transpose(0, 2, 1, 3).reshape(n, 16, 16).astype(np.float64)
    G, alpha = np.where(on, G, 0).astype(np.float64), np.where(on, alpha, 0).astype(np.float64)
    v = G * d0 * ax(rgb[:, 0].astype(np.float64))
    dx, dy = X.astype(np.float64) - ax(mu[:, 0]), Y.astype(np.float64) - ax(mu[:, 1])
    gq = -0.5 * co[:, 3].astype(np.float64)
    total = lambda a: a.sum((1, 2))
    want_conic = np.stack([gq * total(v * dx * dx), 2 * gq * total(v * dx * dy), gq * total(v * dy * dy)], 1)
    gx, gy = gq * total(v * dx), gq * total(v * dy)
    a, b, cc = (co[:, k].astype(np.float64) for k in range(3))
    want_mean = -2 * np.stack([a * gx + b * gy, b * gx + cc * gy], 1)
    # (the place's gradient cancels from pixel to pixel where the contributions have one sign: measured by their magnitudes)
    mx, my = total(np.abs(v * dx)) * -gq, total(np.abs(v * dy)) * -gq
    of_mean = 2 * np.stack([a * mx + np.abs(b) * my, np.abs(b) * mx + cc * my], 1)
    norm = lambda got, want, of=None: float(np.linalg.norm(got - want) / np.linalg.norm(want if of is None else of))
    errors = (norm(gr["conic"], want_conic), norm(gr["mean2d"], want_mean, of_mean), norm(gr["opacities"], total(v)),
              norm(gr["rgb"][:, 0], total(alpha * d0)))
    if want_abs:
        a, b, cc = ax(a), ax(b), ax(cc)
        sizes = np.stack([total(np.abs(v * (a * dx + b * dy))), total(np.abs(v * (b * dx + cc * dy)))], 1)
        errors += (norm(gr["mean2d_abs"], co[:, 3:].astype(np.float64) * sizes),)
    return errors


@pytest.mark.parametrize("want_abs", [False, True])
@pytest.mark.parametrize("one_sign", [False, True])
@pytest.mark.parametrize("eigenvalues", [(0.3, 0.3), (0.35, 0.6), (1.0, 1.0), (2.0, 4.0), (0.3, 5.0)])
def test_gradients_of_small_splats_against_exact_sums(eigenvalues, one_sign, want_abs):
    """A contribution passes some ten roundings on its way (colour times loss gradient, transmittance, weight, place, place
    again, four levels of sums, the record), each off by at most 2^-24 and by 0.6 of that on average: 2^-24 * 0.6 * sqrt(10)
    = 1.1e-7 where they are independent.  Bound: twice that.  Moments formed about a sub-tile's centre and shifted to the
    splat leave 5e-7 at the low-pass floor."""
    from paper_2511_04283_amd import binding as B
    errors = gradient_errors(B, eigenvalues, one_sign, want_abs)
    assert max(errors) <= 2.3e-7, errors

"""GPU parity of fs_photo_loss (Sec. 4.3 E_photo, Sec. 4.5 loss) and the pruning score (Sec. 4.3, s_p)
against the fp64 oracle.  Floating point, no integer decisions: L1 / SSIM / E within 1e-5 relative
(fp32 window sums against fp64), gradient within 1e-3 relative with the 2e-3-of-max floor."""
import numpy as np
import pytest

import oracle
from oracle import Oracle
from paper_2511_04283_amd import scenes
from gpu_common import assert_grads_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2511_04283_amd import binding as B
    c = B.Context("cuda:0")
    yield c
    c.close()


def _run(ctx, x, y, lam, want_grad=True):
    import torch
    xt = torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(ctx.device)
    yt = torch.from_numpy(np.ascontiguousarray(y, np.float32)).to(ctx.device)
    out3, g = ctx.fs_photo_loss(xt, yt, lam, want_grad=want_grad)
    return out3.cpu().numpy(), (g.cpu().numpy() if g is not None else None)


def _check(ctx, x, y, lam, threads=3):
    x = np.ascontiguousarray(x, np.float32)
    y = np.ascontiguousarray(y, np.float32)
    out3, g = _run(ctx, x, y, lam)
    ref = oracle.photometric(x, y, lam, threads=threads)
    assert out3[0] == pytest.approx(ref["L1"], rel=1e-6)
    assert out3[1] == pytest.approx(ref["ssim"], rel=1e-5, abs=1e-6)
    assert out3[2] == pytest.approx(ref["E"], rel=1e-5, abs=1e-6)
    assert_grads_close({"dE": g}, {"dE": ref["grad"]})
    return out3, ref


@pytest.mark.parametrize("H,W,lam", [(16, 32, 0.2), (37, 53, 0.2), (5, 7, 0.5), (1, 1, 0.2), (130, 97, 1.0), (64, 64, 0.0)])
def test_random_images_ragged_sizes(ctx, H, W, lam):
    rng = np.random.default_rng(H * 1000 + W)
    x = rng.uniform(0, 1, (3, H, W))
    y = np.clip(x + rng.normal(0, 0.15, x.shape), 0, 1)
    out3, ref = _check(ctx, x, y, lam, threads=1)
    if lam == 0.0:
        assert out3[2] == pytest.approx(out3[0], rel=1e-12)


def test_identical_images_and_value_only_call(ctx):
    x = np.random.default_rng(1).uniform(0, 1, (3, 50, 70)).astype(np.float32)
    out3, g = _run(ctx, x, x, 0.2)
    assert out3[0] == 0.0 and out3[1] == pytest.approx(1.0, abs=1e-6) and abs(out3[2]) < 1e-6
    assert np.abs(g).max() < 1e-6
    out3b, gb = _run(ctx, x, 1 - x, 0.2, want_grad=False)
    assert gb is None and out3b[2] == pytest.approx(oracle.photometric(x, 1 - x, 0.2, want_grad=False)["E"], rel=1e-5)


def test_rendered_image_of_config2_against_its_target(ctx):
    """The loss on a real rendering (smooth regions, black background: the small-variance regime)."""
    from paper_2511_04283_amd import binding as B
    sc = scenes.make_scene(2, 20000)
    cam = sc.cameras[0]
    tgt = scenes.target_image(2, 0, cam)
    g = B.Gaussians.from_scene(sc, ctx.device)
    fcam = B.make_camera(cam)
    proj = ctx.fs_preprocess(g, fcam)
    bins = ctx.fs_bin_sort(proj, fcam)
    image, _, _ = ctx.fs_render_fwd(proj, bins, fcam)
    _check(ctx, image.cpu().numpy(), tgt, 0.2)


def test_full_size_config3_image(ctx):
    rng = np.random.default_rng(3)
    H, W = 1064, 1600
    yy, xx = np.mgrid[0:H, 0:W]
    base = 0.5 + 0.4 * np.sin(xx / 37.0) * np.cos(yy / 23.0)
    x = np.clip(np.stack([base, base[::-1], base[:, ::-1]]) + rng.normal(0, 0.05, (3, H, W)), 0, 1)
    y = np.clip(x + rng.normal(0, 0.1, x.shape) * (rng.uniform(size=(1, H, W)) < 0.3), 0, 1)
    _check(ctx, x, y, 0.2)


def test_prune_score_over_views_bit_exact(ctx):
    import torch
    rng = np.random.default_rng(5)
    K, n = 6, 70001
    counts = rng.integers(0, 4000, (K, n)).astype(np.int32)
    counts[:, ::13] = 0
    E = rng.uniform(0.02, 0.4, K)
    acc = torch.zeros(n, dtype=torch.float64, device=ctx.device)
    Et = torch.from_numpy(E).to(ctx.device)
    for j in range(K):
        ctx.fs_prune_score_accumulate(torch.from_numpy(counts[j]).to(ctx.device), Et[j:j + 1], acc)
    sp = ctx.fs_prune_score_normalize(acc).cpu().numpy()
    raw, ref = oracle.prune_score(counts, E)
    assert np.array_equal(acc.cpu().numpy(), raw)
    assert np.array_equal(sp, ref.astype(np.float32))
    assert sp.min() == 0.0 and sp.max() == 1.0
    # all sums equal: zeros
    acc.fill_(3.5)
    assert not ctx.fs_prune_score_normalize(acc).cpu().numpy().any()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 70001])
def test_view_end_is_the_three_separate_steps(ctx, n):
    """Bit for bit (the same additions), and the view's counts are zero afterwards."""
    import torch
    rng = np.random.default_rng(n)
    dev = ctx.device
    view = torch.from_numpy(rng.integers(0, 4000, n).astype(np.int32)).to(dev)
    E = torch.from_numpy(rng.uniform(0.02, 0.4, 1)).to(dev)
    acc = torch.from_numpy(rng.uniform(0, 100, n)).to(dev)
    counts = torch.from_numpy(rng.integers(0, 9000, n).astype(np.int32)).to(dev)
    acc_ref, counts_ref = acc.clone(), counts.clone()
    ctx.fs_prune_score_accumulate(view, E, acc_ref)
    ctx.fs_counts_add(counts_ref, view)
    ctx.fs_score_view_end(view, E, acc, counts)
    assert torch.equal(acc, acc_ref) and torch.equal(counts, counts_ref) and not view.any()


def test_vcp_pipeline_three_views(ctx, orc32):
    """Counts and E_photo of several views chained on the GPU exactly as the pruning score needs them."""
    import torch
    from paper_2511_04283_amd import binding as B
    sc = scenes.make_scene(4, 6000)
    g = B.Gaussians.from_scene(sc, ctx.device)
    acc = torch.zeros(sc.n, dtype=torch.float64, device=ctx.device)
    counts_ref, E_ref = [], []
    for v in (0, 3, 7):
        cam0 = sc.cameras[v]
        cam = scenes.Camera(333, 219, cam0.fx / 4, cam0.fy / 4, 333 / 2.0, 219 / 2.0, cam0.R, cam0.t)
        tgt = scenes.target_image(4, v, cam)
        fcam = B.make_camera(cam)
        tt = torch.from_numpy(tgt).to(ctx.device)
        proj = ctx.fs_preprocess(g, fcam)
        bins = ctx.fs_bin_sort(proj, fcam)
        image, fT, nc = ctx.fs_render_fwd(proj, bins, fcam)
        mask, _ = ctx.fs_error_mask(image, tt)
        cv = torch.zeros(sc.n, dtype=torch.int32, device=ctx.device)
        ctx.fs_score_accumulate(proj, bins, fcam, fT, nc, mask, cv)
        out3, _ = ctx.fs_photo_loss(image, tt, 0.2, want_grad=False)
        ctx.fs_prune_score_accumulate(cv, out3[2:3], acc)
        p_o, b_o, img_o, fT_o, nc_o = orc32.forward(sc, cam)
        m_o, _, _ = orc32.error_mask(img_o, tgt)
        counts_ref.append(orc32.score(p_o, b_o, cam, m_o, np.zeros(sc.n, np.int32)))
        E_ref.append(oracle.photometric(img_o, tgt, 0.2, want_grad=False)["E"])
        assert np.array_equal(cv.cpu().numpy(), counts_ref[-1])
        assert out3[2].item() == pytest.approx(E_ref[-1], rel=1e-5)
    sp = ctx.fs_prune_score_normalize(acc).cpu().numpy()
    _, ref = oracle.prune_score(np.stack(counts_ref), np.array(E_ref))
    assert np.abs(sp - ref).max() < 2e-5 and ref.max() == 1.0


@pytest.mark.parametrize("H,W", [(37, 31), (38, 32), (39, 33), (76, 64), (77, 65), (6, 200), (200, 6)])
def test_sizes_round_a_block_with_and_without_the_gradient(ctx, H, W):
    """Blocks are 38 x 32: one block exactly, one row or column fewer and more, two blocks, slivers.  The value-only call and
    the one with a gradient add the same numbers in the same order."""
    rng = np.random.default_rng(7 * H + W)
    x = rng.uniform(0, 1, (3, H, W))
    y = np.clip(x + rng.normal(0, 0.15, x.shape), 0, 1)
    out3, _ = _check(ctx, x, y, 0.2, threads=1)
    value_only, _ = _run(ctx, x, y, 0.2, want_grad=False)
    assert np.array_equal(value_only, out3)

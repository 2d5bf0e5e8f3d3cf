"""The order inside one tile (fs_bin_sort's per-tile ordering) at the list lengths where its variants begin and end, for
depths that spread evenly, that cluster with an outlier stretching their range, and that tie (ties go by index, and many
of them in one bucket take the sorting network): bit-exact against a stable sort of (depth bits, index)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depths", ["even", "clustered", "few_values", "equal"])
def test_order_of_one_list(depths):
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    c = B.Context("cuda:0")
    cam = B.make_camera(scenes.Camera(16, 16, 16.0, 16.0, 8.0, 8.0))
    for n in (1, 2, 64, 255, 257, 512, 513, 1000, 2048, 2049, 4096, 4097, 8192, 8193, 16384):
        rng = np.random.default_rng(n)
        if depths == "even":
            d = rng.uniform(0.2, 50.0, n)
        elif depths == "clustered":
            d = rng.normal(2.0, 0.003, n) + rng.integers(0, 3, n)
            d[n // 2] = 3.0e4
        elif depths == "few_values":
            d = rng.choice([1.0, 1.0000001, 2.5, 2.5000002, 7.0, 7.5, 8.0], n)
        else:
            d = np.full(n, 3.25)
        d = d.astype(np.float32)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(c.device)
        rect = np.tile(np.array([0, 0, 1, 1], np.int16), (n, 1))
        co = np.tile(np.array([0.1, 0.0, 0.1, 0.5], np.float32), (n, 1))
        proj = B.Projected(t(np.full((n, 2), 8.0, np.float32)), t(d), t(co), t(np.full((n, 3), 0.5, np.float32)), t(rect),
                           t(np.ones(n, np.int32)), t(np.zeros((n, 3), np.uint8)))
        bins = c.fs_bin_sort(proj, cam)
        order = np.lexsort((np.arange(n), d.view(np.uint32)))
        assert bins.num_pairs == n
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), order.astype(np.int32)), n
        assert np.array_equal(bins.copy_keys().cpu().numpy(), d.view(np.uint32)[order].astype(np.int64)), n
    c.close()


@pytest.mark.parametrize("n", [2049, 2055, 2056, 4088, 4097, 8193])
def test_every_list_is_long(n):
    """The launches for long lists are as wide as the pairs allow, which lists of one length reach: none may be left out,
    neither in a context's first ordering nor in the next one, which is enqueued ahead of its totals."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    tiles = 7
    c = B.Context("cuda:0")
    cam = B.make_camera(scenes.Camera(16 * tiles, 16, 16.0, 16.0, 8.0, 8.0))
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(c.device)
    for turn in range(2):
        rng = np.random.default_rng(10 * n + turn)
        tile = rng.permutation(np.repeat(np.arange(tiles), n)).astype(np.int16)
        d = rng.uniform(0.2, 50.0, n * tiles).astype(np.float32)
        rect = np.stack([tile, 0 * tile, tile + 1, 0 * tile + 1], 1)
        m = n * tiles
        proj = B.Projected(t(np.full((m, 2), 8.0, np.float32)), t(d), t(np.tile(np.array([0.1, 0.0, 0.1, 0.5], np.float32), (m, 1))),
                           t(np.full((m, 3), 0.5, np.float32)), t(rect), t(np.ones(m, np.int32)), t(np.zeros((m, 3), np.uint8)))
        bins = c.fs_bin_sort(proj, cam)
        order = np.lexsort((np.arange(m), d.view(np.uint32), tile))
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), order.astype(np.int32)), turn
    c.close()


@pytest.mark.parametrize("compact", [False, True])
@pytest.mark.parametrize("n, grid, most", [(1, (45, 29), 3), (63, (45, 29), 3), (64, (45, 29), 3), (65, (45, 29), 3), (16384, (45, 29), 3),
                                           (16385, (45, 29), 3), (262143, (45, 29), 3), (262209, (45, 29), 3),
                                           (64, (20, 30), 1), (64, (20, 30), 20), (129, (3, 1), 2), (2000, (128, 120), 40)])
def test_pairs_and_record_places(n, grid, most, compact):
    """The counting and placement kernels deal 64 Gaussians at a time out to their workgroups: one chunk, a last one that is not
    full, one for every workgroup and one more, one for every wavefront and a second round of one.  A chunk's pairs are walked
    128 at a time: none, fewer than 64, many, and on the largest grid of the per-tile ordering.  The order bit for bit,
    and every Gaussian's gradient records (one per tile of its rectangle) a place of their own."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    rng = np.random.default_rng(n)
    config = B.default_config()
    config.compact_box = 1 if compact else 0
    c = B.Context("cuda:0", config)
    tx, ty = grid
    cam = B.make_camera(scenes.Camera(16 * tx, 16 * ty, 500.0, 500.0, 8.0 * tx, 8.0 * ty))
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(c.device)
    x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
    w, h = np.minimum(rng.integers(0, most + 1, n), tx - x0), np.minimum(rng.integers(0, most, n), ty - y0)
    rect = np.stack([x0, y0, x0 + w, y0 + h], 1).astype(np.int16)
    area = w * h
    d = rng.uniform(0.2, 50.0, n).astype(np.float32)
    # (so wide that every tile of the rectangle meets the ellipse)
    co = np.tile(np.array([1e-5, 0.0, 1e-5, 0.5], np.float32), (n, 1))
    mean = np.stack([16.0 * x0 + 8.0, 16.0 * y0 + 8.0], 1).astype(np.float32)
    proj = B.Projected(t(mean), t(d), t(co), t(np.full((n, 3), 0.5, np.float32)), t(rect), t(area.astype(np.int32)),
                       t(np.zeros((n, 3), np.uint8)))
    for turn in range(2):   # (the second one's placement is enqueued ahead of the totals)
        bins = c.fs_bin_sort(proj, cam)
        assert bins.num_pairs == area.sum() and bins.struct.num_records == area.sum()
        gauss = np.repeat(np.arange(n), area)
        k = np.arange(area.sum()) - np.repeat(np.cumsum(area) - area, area)
        tile = (y0[gauss] + k // np.maximum(w[gauss], 1)) * tx + x0[gauss] + k % np.maximum(w[gauss], 1)
        order = np.lexsort((gauss, d.view(np.uint32)[gauss], tile))
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), gauss[order].astype(np.int32))
        first = bins._copy(bins.struct.record_offsets, n, torch.int32).cpu().numpy().astype(np.int64)
        places = np.repeat(first, area) + k
        assert np.array_equal(np.sort(places), np.arange(area.sum()))
        chunks = np.arange(n) // 64
        same = (chunks[1:] == chunks[:-1])
        assert np.array_equal((first[1:] - first[:-1])[same], area[:-1][same])   # (those of 64 Gaussians follow each other)
    c.close()

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

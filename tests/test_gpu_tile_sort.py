"""The order inside one tile (fs_bin_sort's per-tile ordering) at the list lengths where its variants begin and end, for
depths that spread evenly, that cluster with an outlier stretching their range, and that tie (ties go by index, and many
of them in one bucket take the sorting network): bit-exact against a stable sort of (depth bits, index)."""
import ctypes

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


def ordering_inputs(B, device, rect, depth, conic_opacity, mean, touched):
    import torch
    n = len(depth)
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a).astype(dt)).to(device)
    return B.Projected(t(mean, np.float32), t(depth, np.float32), t(conic_opacity, np.float32), t(np.full((n, 3), 0.5), np.float32),
                       t(rect, np.int16), t(touched, np.int32), t(np.zeros((n, 3)), np.uint8))


def pairs_met(o, rect, depth, mean, conic_opacity, tiles_x):
    """(tile, Gaussian) of every pair that the oracle's Compact Box emits for these rectangles."""
    from oracle import _p
    most = int(((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).sum())
    keys, gauss = np.zeros(max(most, 1), np.uint64), np.zeros(max(most, 1), np.uint32)
    rect = np.ascontiguousarray(rect, np.int32)
    met = int(o._f("orc_emit_pairs_cb")(ctypes.c_int64(len(depth)), _p(rect), _p(depth.view(np.uint32)), _p(mean), _p(conic_opacity),
                                        _p(o.cfg.array(np.float32)), ctypes.c_int(tiles_x), ctypes.c_int(16), _p(keys), _p(gauss)))
    return (keys[:met] >> np.uint64(32)).astype(np.int64), gauss[:met].astype(np.int64)


def check_lists(c, B, lengths, seed):
    """One-tile Gaussians on a row of tiles, so many on each: the order bit for bit."""
    from paper_2511_04283_amd import scenes
    rng = np.random.default_rng(seed)
    cam = B.make_camera(scenes.Camera(16 * len(lengths), 16, 16.0, 16.0, 8.0, 8.0))
    tile = rng.permutation(np.repeat(np.arange(len(lengths)), lengths))
    n = len(tile)
    d = rng.uniform(0.2, 50.0, n).astype(np.float32)
    proj = ordering_inputs(B, c.device, np.stack([tile, 0 * tile, tile + 1, 0 * tile + 1], 1), d, np.tile([0.1, 0.0, 0.1, 0.5], (n, 1)),
                           np.full((n, 2), 8.0), np.ones(n))
    bins = c.fs_bin_sort(proj, cam)
    order = np.lexsort((np.arange(n), d.view(np.uint32), tile))
    assert np.array_equal(bins.copy_gauss().cpu().numpy(), order.astype(np.int32)), lengths


@pytest.mark.parametrize("n", [2049, 2055, 2056, 4088, 4097, 8193])
def test_every_list_is_long(n):
    """The launches for long lists are as wide as the pairs allow, which lists of one length reach: none may be left out,
    neither in a context's first ordering nor in the next one, which is enqueued ahead of its totals."""
    from paper_2511_04283_amd import binding as B
    c = B.Context("cuda:0")
    for turn in range(2):
        check_lists(c, B, [n] * 7, 10 * n + turn)
    c.close()


# (shorter lists, the long one, empty tiles; the shortest length that the launch for the long one takes)
LONG_BEHIND_SHORT = [(2048, 2049, 0, 2049), (2048, 2049, 40, 2049), (2048, 2054, 40, 2049), (4088, 4097, 0, 4097), (4096, 4097, 0, 4097),
                     (4100, 8193, 0, 8193), (4100, 8193, 40, 8193), (8192, 8193, 40, 8193)]


@pytest.mark.parametrize("place", range(7))
@pytest.mark.parametrize("short, long, empty, least", LONG_BEHIND_SHORT)
def test_one_long_list_behind_shorter_ones(short, long, empty, least, place):
    """The tiles stand in order of buckets of lengths, not of lengths, so a launch for lists of `least` words and more may find
    shorter ones of the same bucket in front: it has to reach them all.  On a new context its width follows from the pairs to
    the word, and pairs / least would be too few workgroups for the last of the seven (which of them stands last in the
    bucket follows from their places).  With the empty tiles the launch has fewer workgroups than there are tiles."""
    from paper_2511_04283_amd import binding as B
    assert (6 * short + long) // least < 7
    lengths = [short] * 7 + [0] * empty
    lengths[place] = long
    c = B.Context("cuda:0")
    check_lists(c, B, lengths, long + 100 * place + empty)
    c.close()


@pytest.mark.parametrize("conics", ["square", "all_met", "some_missed"])
@pytest.mark.parametrize("n, grid, most", [(1, (45, 29), 3), (63, (45, 29), 3), (64, (45, 29), 3), (65, (45, 29), 3), (16384, (45, 29), 3),
                                           (16385, (45, 29), 3), (262143, (45, 29), 3), (262209, (45, 29), 3),
                                           (64, (20, 30), 1), (64, (20, 30), 20), (129, (3, 1), 2), (2000, (128, 120), 40)])
def test_pairs_and_record_places(n, grid, most, conics):
    """The counting and placement kernels deal 64 Gaussians at a time out to their workgroups: one chunk, a last one that is not
    full, one for every workgroup and one more, one for every wavefront and a second round of one.  A chunk's pairs are walked
    128 at a time: none, fewer than 64, many, and on the largest grid of the per-tile ordering.  The order bit for bit,
    and every Gaussian's gradient records (one per tile of its rectangle) a place of their own.  With the Compact Box, for
    ellipses that meet every tile of their rectangles and for ones that miss some: there the places of the missed tiles,
    which an earlier backward pass has left gradients in, add nothing."""
    import torch
    from oracle import Config, Oracle
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    rng = np.random.default_rng(n)
    config = B.default_config()
    config.compact_box = 0 if conics == "square" else 1
    c = B.Context("cuda:0", config)
    c.fs_set_record_mode(B.FS_RECORDS_DENSE)
    o = Oracle(np.float32, Config(compact_box=True))
    tx, ty = grid
    camera = scenes.Camera(16 * tx, 16 * ty, 500.0, 500.0, 8.0 * tx, 8.0 * ty)
    cam = B.make_camera(camera)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a).astype(np.float32)).to(c.device)
    g = B.Gaussians(t(np.tile([0, 0, 5.0], (n, 1))), t(np.full((n, 3), 0.1)), t(np.tile([1.0, 0, 0, 0], (n, 1))), t(np.full(n, 0.02)),
                    t(np.zeros((n, 1, 3))), 0)
    dL = torch.ones((3, camera.height, camera.width), device=c.device)
    for turn in range(2):   # (the second one's placement is enqueued ahead of the totals)
        x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
        w, h = np.minimum(rng.integers(0, most + 1, n), tx - x0), np.minimum(rng.integers(0, most, n), ty - y0)
        rect = np.stack([x0, y0, x0 + w, y0 + h], 1)
        area = w * h
        d = rng.uniform(0.2, 50.0, n).astype(np.float32)
        # (opacity 0.02: a pixel blends hundreds, so that the first turn leaves gradients in most records)
        co = np.tile(np.array([1e-6, 0.0, 1e-6, 0.02], np.float32), (n, 1))   # (so wide that every tile of the rectangle meets the ellipse)
        mean = np.stack([16.0 * x0 + 8.0, 16.0 * y0 + 8.0], 1).astype(np.float32)
        if conics == "some_missed" and turn == 1:   # an ellipse within its rectangle, round some point of it
            half = 8.0 * np.maximum(np.stack([w, h], 1), 1) * rng.uniform(0.3, 1.0, (n, 2))
            co[:, [0, 2]] = 2.0 * np.log(0.02 * 255.0) / half ** 2
            mean = (16.0 * rect[:, :2] + 16.0 * np.stack([w, h], 1) * rng.uniform(0.1, 0.9, (n, 2))).astype(np.float32)
        gauss = np.repeat(np.arange(n), area)
        k = np.arange(area.sum()) - np.repeat(np.cumsum(area) - area, area)
        tile = (y0[gauss] + k // np.maximum(w[gauss], 1)) * tx + x0[gauss] + k % np.maximum(w[gauss], 1)
        if conics != "square":   # the oracle's own hit test says which of them are pairs
            tile, gauss = pairs_met(o, rect, d, mean, co, tx)
            missed = area.sum() - len(gauss)
            assert turn == 1 or missed == 0
        touched = np.bincount(gauss, minlength=n)
        proj = ordering_inputs(B, c.device, rect, d, co, mean, touched)
        bins = c.fs_bin_sort(proj, cam)
        assert bins.num_pairs == len(gauss) and bins.struct.num_records == area.sum()
        order = np.lexsort((gauss, d.view(np.uint32)[gauss], tile))
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), gauss[order].astype(np.int32)), turn
        first = bins._copy(bins.struct.record_offsets, n, torch.int32).cpu().numpy().astype(np.int64)
        places = np.repeat(first, area) + k
        assert np.array_equal(np.sort(places), np.arange(area.sum()))
        chunks = np.arange(n) // 64
        same = (chunks[1:] == chunks[:-1])
        assert np.array_equal((first[1:] - first[:-1])[same], area[:-1][same])   # (those of 64 Gaussians follow each other)
        if conics == "square":
            continue
        final_T, n_contrib = c.fs_render_fwd(proj, bins, cam)[1:]
        dense = c.fs_render_bwd(g, cam, proj, bins, final_T, n_contrib, dL, want_2d=True)
        if turn == 0:
            left = (dense["rgb"] != 0).all(1).cpu().numpy()
            assert left.sum() >= 0.5 * (area > 0).sum()
            continue
        # (the sparse layout reads no place that nothing was written to; the terms are the same, so that sums of up to some
        # hundred of them in single precision are within 1e-5 in whatever order)
        c.fs_set_record_mode(B.FS_RECORDS_SPARSE)
        sparse = c.fs_render_bwd(g, cam, proj, bins, final_T, n_contrib, dL, want_2d=True)
        for name in ("mean2d", "conic", "rgb", "opacities"):
            assert (dense[name] - sparse[name]).abs().max() <= 1e-5 * sparse[name].abs().max(), name
    assert conics != "some_missed" or most < 2 or n < 63 or missed > 0
    c.close()

"""The placement in two steps (bands of 64 tiles, then tiles), taken from a million Gaussians on where the context's ordering before
had 2.85 M candidate tiles or there was none: the order bit for bit against a stable sort of (tile, depth bits, index) or the radix
path's, on a new context, ahead of the totals, and where what was enqueued ahead of them does not fit; at the sizes where the rule
begins and ends, with one tile too few, a last band of one tile, empty bands, one band that has nearly everything, and the highest
indices."""
import math

import numpy as np
import pytest

from test_gpu_tile_sort import pairs_met

pytestmark = pytest.mark.gpu

LEAST, MOST = 1000000, 1 << 26   # Gaussians
CANDIDATES = 2850000   # of the ordering before


def scattered(n, pairs, grid, crowd_bands, share, seed):
    """`pairs` pairs, in rows of neighbouring tiles; a share of the Gaussians starts on so many bands from the second on, the others anywhere."""
    import torch
    from paper_2511_04283_amd import binding as B
    dev = "cuda:0"
    tx, ty = grid
    gen = torch.Generator(device=dev).manual_seed(seed)
    rand = lambda *s: torch.rand(s, device=dev, generator=gen)
    at = torch.where(rand(n) < share, 64 + (rand(n) * 64 * crowd_bands).long(), (rand(n) * tx * ty).long().clamp_(max=tx * ty - 1))
    x0, y0 = at % tx, at // tx
    w = torch.minimum(pairs // n + (rand(n) < (pairs % n) / n).long(), tx - x0)
    rect = torch.stack([x0, y0, x0 + w, y0 + 1], 1).to(torch.int16)
    means = torch.stack([16.0 * x0 + 8.0, 16.0 * y0 + 8.0], 1)
    return B.Projected(means, 0.2 + 50.0 * rand(n), torch.tensor([1e-6, 0.0, 1e-6, 0.02], device=dev).repeat(n, 1), rand(n, 3),
                       rect, w.to(torch.int32), torch.zeros((n, 3), dtype=torch.uint8, device=dev))


@pytest.mark.parametrize("n, grid, crowd", [(LEAST - 1, (13, 5), 0), (LEAST, (13, 5), 0), (LEAST, (16, 4), 0), (LEAST + 65, (40, 32), 0),
                                            (LEAST, (128, 120), 0), (2 * LEAST, (40, 32), 90000), (MOST, (13, 5), 0), (MOST + 1, (13, 5), 0)])
@pytest.mark.parametrize("compact_box", [0, 1])
def test_order(n, grid, crowd, compact_box):
    """`crowd`: so many of the Gaussians stand on the 64 tiles of the second band, none on the third."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    if n > 3 * LEAST and compact_box:
        pytest.skip("the word's bits are the same")
    rng = np.random.default_rng(n + crowd)
    config = B.default_config()
    config.compact_box = compact_box
    c = B.Context("cuda:0", config)
    tx, ty = grid
    cam = B.make_camera(scenes.Camera(16 * tx, 16 * ty, 500.0, 500.0, 8.0 * tx, 8.0 * ty))
    # (the turns with few Gaussians are by bands on the new context and behind an ordering of many candidates; below the rule's least, the
    # last turn's pairs outgrow the buffers of the one before)
    for turn, visible in enumerate((20000, 30000, 200000 if tx * ty > 100 else 100000)):
        if n >= LEAST and turn:
            many = scattered(LEAST, 3200000, (128, 120), 0, 0.0, turn)
            assert c.fs_bin_sort(many, B.make_camera(scenes.Camera(2048, 1920, 500.0, 500.0, 1024.0, 960.0))).struct.num_records >= CANDIDATES
            del many
        if crowd:
            visible = min(visible, 100000)
        seen = np.sort(rng.choice(n, visible - 2, replace=False)) if n < MOST else np.sort(rng.integers(0, n, visible - 2))
        seen = np.unique(np.concatenate([seen, [0, n - 1]]))
        v = len(seen)
        x0, y0 = rng.integers(0, tx, v), rng.integers(0, ty, v)
        w, h = np.minimum(rng.integers(1, 4, v), tx - x0), np.minimum(rng.integers(1, 4, v), ty - y0)
        if crowd:
            in_crowd = rng.permutation(v) < crowd
            at = rng.integers(64, 128, v)
            other = np.where(rng.integers(0, 2, v) == 0, rng.integers(0, 64, v), rng.integers(192, tx * ty, v))
            at = np.where(in_crowd, at, other)
            x0, y0, w, h = at % tx, at // tx, np.ones(v, int), np.ones(v, int)
        d = rng.uniform(0.2, 50.0, v).astype(np.float32)
        d[rng.integers(0, v, v // 4)] = 7.0   # (ties go by index)
        area = w * h
        gauss = np.repeat(np.arange(v), area)
        k = np.arange(area.sum()) - np.repeat(np.cumsum(area) - area, area)
        tile = (y0[gauss] + k // w[gauss]) * tx + x0[gauss] + k % w[gauss]
        assert np.bincount(tile).max() <= 16384   # (the per-tile ordering's longest list)
        dev = c.device
        where = torch.from_numpy(seen).to(dev)
        put = lambda a, shape, dtype: torch.zeros((n, *shape), dtype=dtype, device=dev).index_copy_(
            0, where, torch.from_numpy(np.ascontiguousarray(a)).to(dtype).to(dev))
        rect = np.stack([x0, y0, x0 + w, y0 + h], 1)
        # (an ellipse so wide that every tile of its rectangle meets it)
        proj = B.Projected(put(np.stack([16.0 * x0 + 8.0, 16.0 * y0 + 8.0], 1), (2,), torch.float32), put(d, (), torch.float32),
                           put(np.tile([1e-6, 0.0, 1e-6, 0.02], (v, 1)), (4,), torch.float32), put(np.full((v, 3), 0.5), (3,), torch.float32),
                           put(rect, (4,), torch.int16), put(area, (), torch.int32), put(np.zeros((v, 3)), (3,), torch.uint8))
        bins = c.fs_bin_sort(proj, cam)
        assert bins.num_pairs == len(gauss)
        order = np.lexsort((gauss, d.view(np.uint32)[gauss], tile))
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), seen[gauss][order].astype(np.int32)), visible
        keys = tile[order].astype(np.int64) << 32 | d.view(np.uint32)[gauss][order].astype(np.int64)
        assert np.array_equal(bins.copy_keys().cpu().numpy(), keys), visible
        del proj, bins, put, where
    c.close()


def test_bands_of_very_different_lengths():
    """The second step's chunks of 4096 words go through the bands in one row: more chunks than workgroups, bands without a pair, a
    share of the first step's words beyond what the buffers hold.  Against the radix path's order."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    grid, n = (120, 68), 3 * LEAST
    config = B.default_config()
    tiled = B.Context("cuda:0", config)
    config.sort_mode = B.FS_SORT_RADIX
    radix = B.Context("cuda:0", config)
    cam = B.make_camera(scenes.Camera(16 * grid[0], 16 * grid[1], 500.0, 500.0, 8.0 * grid[0], 8.0 * grid[1]))
    longest = 0
    # (5 M: on a new context, then ahead of the totals; 8 M and 20 M outgrow the buffers of the one before)
    for pairs, bands, share in ((5, 6, 0.9), (5, 7, 1.0), (8, 9, 0.97), (20, 12, 0.5), (20, 14, 0.6), (4, 128, 0.0)):
        proj = scattered(n, pairs * 1000000, grid, bands, share, pairs + bands)
        got, want = tiled.fs_bin_sort(proj, cam), radix.fs_bin_sort(proj, cam)
        assert got.struct.pair_offsets is None and got.num_pairs == want.num_pairs   # (ordered per tile)
        for copy in ("copy_ranges", "copy_gauss", "copy_keys"):
            assert torch.equal(getattr(got, copy)(), getattr(want, copy)()), (pairs, bands, copy)
        longest = max(longest, got.num_pairs)
    assert longest > (4096 + 128) * 4096
    tiled.close()
    radix.close()


def test_chunks_at_their_edges():
    """Bands of 4096 words, of one more, of one and of none, and a last one of a single tile."""
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    grid, n = (13, 25), LEAST   # 325 tiles: five bands and five tiles
    lengths = [4096, 4097, 0, 1, 8192, 4095]
    rng = np.random.default_rng(3)
    tiles = np.concatenate([rng.integers(64 * b, min(64 * b + 64, 325), m) for b, m in enumerate(lengths)])
    v = len(tiles)
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(5)
    seen = torch.randperm(n, device=dev, generator=gen)[:v].sort().values
    put = lambda a, shape, dtype: torch.zeros((n, *shape), dtype=dtype, device=dev).index_copy_(0, seen, a.to(dtype))
    t = torch.from_numpy(rng.permutation(tiles)).to(dev)
    x0, y0 = t % grid[0], t // grid[0]
    one = torch.ones(v, device=dev)
    proj = B.Projected(put(torch.stack([16.0 * x0 + 8, 16.0 * y0 + 8], 1), (2,), torch.float32),
                       put(0.2 + 50.0 * torch.rand(v, device=dev, generator=gen), (), torch.float32),
                       put(torch.tensor([1e-2, 0.0, 1e-2, 0.5], device=dev).repeat(v, 1), (4,), torch.float32),
                       torch.zeros((n, 3), device=dev), put(torch.stack([x0, y0, x0 + 1, y0 + 1], 1), (4,), torch.int16),
                       put(one, (), torch.int32), torch.zeros((n, 3), dtype=torch.uint8, device=dev))
    config = B.default_config()
    tiled = B.Context(dev, config)
    config.sort_mode = B.FS_SORT_RADIX
    radix = B.Context(dev, config)
    cam = B.make_camera(scenes.Camera(16 * grid[0], 16 * grid[1], 500.0, 500.0, 8.0 * grid[0], 8.0 * grid[1]))
    got, want = tiled.fs_bin_sort(proj, cam), radix.fs_bin_sort(proj, cam)
    assert got.num_pairs == want.num_pairs == sum(lengths)
    for copy in ("copy_ranges", "copy_gauss", "copy_keys"):
        assert torch.equal(getattr(got, copy)(), getattr(want, copy)()), copy
    tiled.close()
    radix.close()


def test_missed_candidates():
    """With the Compact Box, ellipses that miss tiles of their rectangles: no word for those, and their gradient records, in which the
    turn before has left gradients, add nothing.  Against the oracle's pairs, the radix path's order, and the layout of records that
    reads no place that nothing was written to."""
    import torch
    from oracle import Config, Oracle
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    o = Oracle(np.float32, Config(compact_box=True))
    tx, ty, n, dev = 120, 68, LEAST + 65, "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(11)
    rand = lambda *s: torch.rand(s, device=dev, generator=gen)
    config = B.default_config()
    config.compact_box = 1
    tiled = B.Context(dev, config)
    tiled.fs_set_record_mode(B.FS_RECORDS_DENSE)
    config.sort_mode = B.FS_SORT_RADIX
    radix = B.Context(dev, config)
    cam = B.make_camera(scenes.Camera(16 * tx, 16 * ty, 500.0, 500.0, 8.0 * tx, 8.0 * ty))
    g = B.Gaussians(torch.tensor([0.0, 0.0, 5.0], device=dev).repeat(n, 1), torch.full((n, 3), 0.1, device=dev),
                    torch.tensor([1.0, 0.0, 0.0, 0.0], device=dev).repeat(n, 1), torch.full((n,), 0.02, device=dev),
                    torch.zeros((n, 1, 3), device=dev), 0)
    dL = torch.ones((3, 16 * ty, 16 * tx), device=dev)
    for turn in range(2):   # (the first one's placement is behind the totals, the second one's ahead of them)
        size = 1 + (rand(n, 2) * 3).long()
        first = (rand(n, 2) * torch.tensor([tx - 3, ty - 3], device=dev)).long()
        # (as wide as meets every tile; then within the rectangle, round some point of it)
        mean, conic = 16.0 * first + 8.0, torch.tensor([1e-6, 0.0, 1e-6, 0.02], device=dev).repeat(n, 1)
        if turn == 1:
            half = 8.0 * size * (0.3 + 0.7 * rand(n, 2))
            conic[:, [0, 2]] = 2.0 * math.log(0.02 * 255.0) / half ** 2
            mean = 16.0 * first + 16.0 * size * (0.1 + 0.8 * rand(n, 2))
        rect, depth = torch.cat([first, first + size], 1), 0.2 + 50.0 * rand(n)
        candidates = int(size.prod(1).sum())
        assert candidates >= CANDIDATES
        tile, gauss = pairs_met(o, *(a.cpu().numpy() for a in (rect, depth, mean, conic)), tx)
        proj = B.Projected(mean, depth, conic, rand(n, 3), rect.to(torch.int16),
                           torch.from_numpy(np.bincount(gauss, minlength=n)).to(dev, torch.int32), torch.zeros((n, 3), dtype=torch.uint8, device=dev))
        got, want = tiled.fs_bin_sort(proj, cam), radix.fs_bin_sort(proj, cam)
        assert got.num_pairs == len(gauss) and got.struct.num_records == candidates and got.struct.pair_offsets is None
        assert (got.num_pairs == candidates) == (turn == 0)
        ends = np.cumsum(np.bincount(tile, minlength=tx * ty))
        ranges = got.copy_ranges().cpu().numpy()
        assert np.array_equal(ranges[ranges[:, 1] > 0, 1], ends[ranges[:, 1] > 0])
        for copy in ("copy_ranges", "copy_gauss", "copy_keys"):
            assert torch.equal(getattr(got, copy)(), getattr(want, copy)()), (turn, copy)
        final_T, n_contrib = tiled.fs_render_fwd(proj, got, cam)[1:]
        dense = tiled.fs_render_bwd(g, cam, proj, got, final_T, n_contrib, dL, want_2d=True)
    assert got.num_pairs < 0.9 * candidates
    # (the terms are the same: sums of up to nine of them in single precision are within 1e-5 in whatever order)
    tiled.fs_set_record_mode(B.FS_RECORDS_SPARSE)
    sparse = tiled.fs_render_bwd(g, cam, proj, got, final_T, n_contrib, dL, want_2d=True)
    for name in ("mean2d", "conic", "rgb", "opacities"):
        assert sparse[name].abs().max() > 0
        assert (dense[name] - sparse[name]).abs().max() <= 1e-5 * sparse[name].abs().max(), name
    tiled.close()
    radix.close()

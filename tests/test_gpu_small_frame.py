"""The ordering of a small frame in one launch: order, keys, ranges and records bit for bit those of a stable sort of (tile, depth bits,
index), and those of the usual launches, which take the same rectangles in an image of more tiles."""
import numpy as np
import pytest

from test_gpu_tile_sort import ordering_inputs, pairs_met

pytestmark = pytest.mark.gpu


def context(compact_box):
    from paper_2511_04283_amd import binding as B
    config = B.default_config()
    config.compact_box = compact_box
    return B.Context("cuda:0", config)


def camera(tx, ty):
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd import scenes
    return B.make_camera(scenes.Camera(16 * tx, 16 * ty, 500.0, 500.0, 8.0 * tx, 8.0 * ty))


@pytest.mark.parametrize("conics", ["square", "all_met", "some_missed"])
@pytest.mark.parametrize("n, grid, most", [(1, (1, 1), 1), (63, (3, 1), 2), (256, (32, 32), 20), (257, (31, 33), 32), (4095, (20, 15), 6),
                                           (4096, (2, 2), 3), (4097, (7, 5), 4), (8192, (8, 8), 6), (10000, (20, 20), 3), (9999, (2, 1), 2), (3906, (1024, 1), 40)])
def test_order_in_one_launch(n, grid, most, conics):
    """Places of a thread's Gaussians that are whole or end within; tiles up to the most there may be; lists that the launch orders and
    ones that are left to the longer sorts; empty rectangles; buffers that are new, that fit and that are too small."""
    import torch
    from oracle import Config, Oracle
    from paper_2511_04283_amd import binding as B
    rng = np.random.default_rng(n)
    c, usual = context(conics != "square"), context(conics != "square")
    o = Oracle(np.float32, Config(compact_box=True))
    tx, ty = grid
    cam, more = camera(tx, ty), camera(tx, ty + (1024 + tx) // tx)
    for turn, share in enumerate((0.3, 0.2, 1.0)):
        x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
        w, h = np.minimum(rng.integers(0, most + 1, n), tx - x0), np.minimum(rng.integers(0, most + 1, n), ty - y0)
        w[rng.random(n) > share] = 0
        w[0], h[0] = max(w[0], 1), max(h[0], 1)
        rect = np.stack([x0, y0, x0 + w, y0 + h], 1)
        area = w * h
        d = rng.uniform(0.2, 50.0, n).astype(np.float32)
        d[rng.integers(0, n, n // 3)] = 7.0   # (ties go by index)
        co = np.tile(np.array([1e-6, 0.0, 1e-6, 0.02], np.float32), (n, 1))
        mean = np.stack([16.0 * x0 + 8.0, 16.0 * y0 + 8.0], 1).astype(np.float32)
        if conics == "some_missed":
            half = 8.0 * np.maximum(np.stack([w, h], 1), 1) * rng.uniform(0.3, 1.0, (n, 2))
            co[:, [0, 2]] = 2.0 * np.log(0.02 * 255.0) / half ** 2
            mean = (16.0 * rect[:, :2] + 16.0 * np.stack([w, h], 1) * rng.uniform(0.1, 0.9, (n, 2))).astype(np.float32)
        gauss = np.repeat(np.arange(n), area)
        k = np.arange(area.sum()) - np.repeat(np.cumsum(area) - area, area)
        tile = (y0[gauss] + k // np.maximum(w[gauss], 1)) * tx + x0[gauss] + k % np.maximum(w[gauss], 1)
        if conics != "square":
            tile, gauss = pairs_met(o, rect, d, mean, co, tx)
        proj = ordering_inputs(B, c.device, rect, d, co, mean, np.bincount(gauss, minlength=n))
        bins, want = c.fs_bin_sort(proj, cam), usual.fs_bin_sort(proj, more)
        assert bins.num_pairs == want.num_pairs == len(gauss) and bins.struct.num_records == area.sum()
        order = np.lexsort((gauss, d.view(np.uint32)[gauss], tile))
        assert np.array_equal(bins.copy_gauss().cpu().numpy(), gauss[order].astype(np.int32)), turn
        assert torch.equal(bins.copy_keys(), want.copy_keys()), turn
        ranges = bins.copy_ranges().reshape(-1, 2).cpu().numpy()
        end = np.cumsum(np.bincount(tile, minlength=tx * ty))
        len_ = ranges[:, 1] - ranges[:, 0]
        assert np.array_equal(len_, np.diff(end, prepend=0)) and np.array_equal(ranges[len_ > 0, 1], end[len_ > 0])
        assert np.array_equal(ranges, want.copy_ranges().reshape(-1, 2).cpu().numpy()[:tx * ty])
        # every tile once, longer lists first as far as their class says
        order = bins.copy_order().cpu().numpy()
        assert np.array_equal(np.sort(order), np.arange(tx * ty)) and (np.diff(len_[order]) < 8).all()
        first = bins._copy(bins.struct.record_offsets, n, torch.int32).cpu().numpy()
        assert np.array_equal(first, np.cumsum(area) - area)
        seen = area > 0
        got, ref = [b._copy(b.struct.splats, 16 * n, torch.int32).cpu().numpy().reshape(n, 16)[seen] for b in (bins, want)]
        assert np.array_equal(np.delete(got, 9, 1), np.delete(ref, 9, 1))   # (9: where the records are, and a flag)
        assert np.array_equal(got[:, 9] & 0x7fffffff, first[seen]) and np.array_equal(got[:, 9] >> 31, ref[:, 9] >> 31)
    c.close()
    usual.close()


def test_calls_are_told_apart_when_their_numbers_start_again():
    """A call knows its tiles' words by its number of 16 bits."""
    from paper_2511_04283_amd import binding as B
    rng = np.random.default_rng(3)
    c, cam = context(0), camera(3, 2)
    projs, orders = [], []
    for n in (40, 90):
        at = rng.integers(0, 6, n)
        x0, y0 = at % 3, at // 3
        d = rng.uniform(0.2, 50.0, n).astype(np.float32)
        projs.append(ordering_inputs(B, c.device, np.stack([x0, y0, x0 + 1, y0 + 1], 1), d, np.tile([0.1, 0.0, 0.1, 0.5], (n, 1)),
                                     np.full((n, 2), 8.0), np.ones(n)))
        orders.append(np.lexsort((np.arange(n), d.view(np.uint32), at)))
    for call in range(65545):
        if call < 5 or call > 65528:
            bins = c.fs_bin_sort(projs[call % 2], cam)
            assert np.array_equal(bins.copy_gauss().cpu().numpy(), orders[call % 2]), call
        else:
            c.fs_bin_sort(projs[call % 3 // 2], cam)
    c.close()

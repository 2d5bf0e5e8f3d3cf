"""What the host waits for by looking at pinned memory (fs_bin_sort's totals, fs_train_step's loss) comes out the same behind an
empty stream and behind a queue longer than the host looks for without a pause, in the first call of a context and in later ones.
(fs_train_step's loss never stands behind a queue of its caller's: the call waits for the totals first.  Its late and missing words
are tested on the CPU.)"""
import time

import numpy as np
import pytest

from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu
LOOKS_S = 0.020   # how long the host looks without a pause


@pytest.mark.parametrize("compact", [0, 1])
def test_totals_and_loss_behind_a_queue(compact):
    import torch
    from paper_2511_04283_amd import binding as B
    from paper_2511_04283_amd.trainer import TrainConfig, Trainer
    cfg = B.default_config()
    cfg.compact_box = compact
    sc = scenes.make_scene(2, 3000)
    cam0 = sc.cameras[0]
    cam = scenes.Camera(245, 137, cam0.fx / 4, cam0.fy / 4, 122.5, 68.5, cam0.R, cam0.t)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    target = t(np.random.default_rng(1).uniform(0, 1, (3, cam.height, cam.width)))
    big = torch.rand(8192, 8192, device="cuda:0")

    def busy():
        """Some 60 ms of work on the stream, none of which the host waits for."""
        nonlocal big
        for _ in range(8):
            big = (big @ big).remainder_(1.0)

    busy()
    torch.cuda.synchronize()
    results = []
    for queue in (False, True):
        ctx = B.Context("cuda:0", cfg)
        g, fcam = B.Gaussians.from_scene(sc, ctx.device), B.make_camera(cam)
        tr = Trainer(ctx, t(sc.means), t(sc.scales), t(sc.quats), t(sc.opacities), t(sc.sh), sc.sh_degree, TrainConfig())
        seen = []
        for _ in range(3):
            proj = ctx.fs_preprocess(g, fcam)
            torch.cuda.synchronize()
            if queue:
                busy()
            start = time.perf_counter()
            bins = ctx.fs_bin_sort(proj, fcam)
            assert not queue or time.perf_counter() - start > LOOKS_S
            seen.append((bins.num_pairs, bins.copy_gauss().cpu()))
            if queue:
                busy()
            start = time.perf_counter()
            loss = tr.step(cam, target)
            assert not queue or time.perf_counter() - start > LOOKS_S
            seen.append((loss, tr.p["means"].cpu()))
        assert len({n for n, _ in seen[0::2]}) == 1
        results.append(seen)
        ctx.close()
    for (a, x), (b, y) in zip(*results):
        assert a == b and torch.equal(x, y)

"""What the host waits for by looking at pinned memory (fs_bin_sort's totals, fs_train_step's loss) comes out the same behind an
empty stream and behind a queue longer than the host looks for (then the stream's own wait takes over), in the first call of a
context and in later ones."""
import numpy as np
import pytest

from paper_2511_04283_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("compact", [0, 1])
@pytest.mark.parametrize("busy", [False, True])
def test_totals_and_loss_behind_a_queue(busy, compact):
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
    big = torch.rand(8192, 8192, device="cuda:0") if busy else None
    results = []
    for queue in (False, busy):
        ctx = B.Context("cuda:0", cfg)
        g, fcam = B.Gaussians.from_scene(sc, ctx.device), B.make_camera(cam)
        tr = Trainer(ctx, t(sc.means), t(sc.scales), t(sc.quats), t(sc.opacities), t(sc.sh), sc.sh_degree, TrainConfig())
        seen = []
        for _ in range(3):
            proj = ctx.fs_preprocess(g, fcam)
            if queue:
                for _ in range(8):   # some 60 ms, three times what the host looks for
                    big = (big @ big).remainder_(1.0)
            bins = ctx.fs_bin_sort(proj, fcam)
            seen.append((bins.num_pairs, bins.copy_gauss().cpu()))
            if queue:
                for _ in range(8):
                    big = (big @ big).remainder_(1.0)
            seen.append((tr.step(cam, target), tr.p["means"].cpu()))
        assert len({n for n, _ in seen[0::2]}) == 1
        results.append(seen)
        ctx.close()
    for (a, x), (b, y) in zip(*results):
        assert a == b and torch.equal(x, y)

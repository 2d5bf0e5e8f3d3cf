"""Trainer.step's order of calls, on a context that only writes down what is asked of it."""
import numpy as np
import torch

from paper_2511_04283_amd import scenes
from paper_2511_04283_amd.trainer import GROUPS, TrainConfig, Trainer


class Stream:
    def __init__(self, calls):
        self.calls = calls

    def synchronize(self):
        self.calls.append("wait")


class Ctx:
    def __init__(self):
        self.calls = []
        self.stream = Stream(self.calls)

    def fs_adam_interval(self, iteration):
        return 1

    def fs_train_step(self, *args, **kw):
        self.calls.append("fs_train_step")
        return 0.1, 0.2, 0.3


def trainer(ctx):
    tr = Trainer.__new__(Trainer)
    tr.ctx, tr.cfg, tr.sh_degree = ctx, TrainConfig(), 0
    tr.p = {k: torch.zeros(1) for k in GROUPS}
    tr.m = tr.v = tr.acc = tr.p
    tr.grad_accum = tr.abs_accum = tr.denom = torch.zeros(1)
    tr.iteration = tr.pending = tr.updates = 0
    return tr


def test_a_step_returns_when_its_update_is_done():
    """fs_train_step returns once the loss is known; a caller of Trainer.step may read the parameters on another stream."""
    ctx = Ctx()
    tr = trainer(ctx)
    cam = scenes.Camera(32, 16, 16.0, 16.0, 16.0, 8.0, np.eye(3), np.zeros(3))
    assert tr.step(cam, None) == 0.3
    assert ctx.calls == ["fs_train_step", "wait"]
    assert (tr.iteration, tr.pending, tr.updates) == (1, 0, 1)

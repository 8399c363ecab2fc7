"""Calls that leave the launch shape unused."""

import numpy as np
import pytest
import torch

from _common import room_workload
from paper_2509_14442_amd import api

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PERSISTENT, GRID = api.make_launch((8, 8), 2, True), api.make_launch((8, 8), 4)


def _scene(w, dtype="f32"):
    field = api.Field.from_temperature(torch.from_numpy(w.T32).to(DEV), dtype)
    return api.Scene(w.scene, field, torch.from_numpy(w.pattern32).to(DEV))


def _seeds(scenes, seed):
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(rng.standard_normal((s.n_rays, 2)).astype(np.float32)).to(DEV) for s in scenes]


def test_unused_persistent_flag_enqueues_nothing():
    """A small call writes the same workspace bytes whether persistent blocks were asked for or
    not: no queue is reset that no kernel reads."""
    sc = _scene(room_workload((30, 24, 20), 40, 32, seed=6, ckpt=3, pat=256))
    seeds = _seeds([sc], 2)
    written = []
    for launch in (GRID, PERSISTENT):
        tr = api.Tracer([sc], launch)
        assert tr.forms() == ("ahead", "pipe")
        for run in (tr.forward, lambda: tr.adjoint(dL_duv=seeds)):
            tr.workspace.fill_(0xA5)
            run()
            written.append((tr.workspace != 0xA5).nonzero().max().item())
    assert written[:2] == written[2:]

"""Parity of the kernels that only larger calls reach: persistent forwards and adjoints of both
tracers, the coherent adjoint's chunk forms, and its cache of cell totals under tiles whose
rays sit in many cells. Every test asserts the form its call takes.

Bars: forwards bitwise; gradients against the FP64 oracle rel-L2 < 1e-3 and per-voxel 1e-3 for
all but 0.5 % of the voxels, as every adjoint test; two launches of one kernel 1e-5 (the cells'
partial sums in another order)."""

import numpy as np
import pytest
import torch

import bos_inputs as bi
import oracle
from _common import grad_errors, room_workload, stored_delta
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


def _listed(w, ids):
    s = _scene(w)
    return api.Scene(w.scene, s.field, s.pattern, torch.from_numpy(ids.astype(np.int32)).to(DEV))


def _forward(scenes, launch, form):
    tr = api.Tracer(scenes, launch)
    assert tr.forms()[0] == form
    print([(s.dims, s.desc.width, s.desc.height) for s in scenes], form, flush=True)
    for t in tr.ckpt + tr.uv + tr.duv:
        t.zero_()
    return tr.forward()


def _gradient(w, scene, seeds):
    """The oracle's gradient for seeds on the GPU."""
    F = oracle.grid_field(stored_delta(w.T32), w.scene.box_lo, w.scene.box_hi)
    return oracle.adjoint(F, w.scene, seeds.cpu().numpy().astype(np.float64))


def _near(g, ref):
    l2, frac = grad_errors(g.cpu().numpy(), ref)
    print(f"  rel-L2 {l2:.2e}, voxels off {frac:.1e}", flush=True)
    assert l2 < 1e-3 and frac <= 5e-3


def _rel(a, b):
    return float((a - b).norm() / b.norm())


def _same_rays(a, i, b, j):
    for x, y in ((a.uv, b.uv), (a.duv, b.duv), (a.n_steps, b.n_steps), (a.status, b.status), (a.ckpt, b.ckpt)):
        assert torch.equal(x[i].view(torch.uint8), y[j].view(torch.uint8))  # bits: NaN for missing rays


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "bf16-xpair"])
@pytest.mark.parametrize("tracer", [0, 1])
def test_forward_forms_agree_bitwise(tracer, dtype):
    """One set of scenes through the grid and the persistent kernel, and each small one alone, with
    its gathers issued ahead (FP16 codes: in a small grid): the same bits, checkpoints included."""
    large = room_workload((60, 52, 44), 580, 500, seed=3, ckpt=3, pat=256)
    small = [room_workload((41, 64, 33), 77, 61, seed=4, ckpt=3, pat=256),
             room_workload((24, 20, 18), 13, 130, seed=5, ckpt=3, max_steps=40, pat=256)]
    for w in [large] + small:
        w.scene = w.scene.replace(tracer=tracer)
    scenes = [_scene(w, dtype) for w in [large] + small]
    grid, pers = _forward(scenes, GRID, "grid"), _forward(scenes, PERSISTENT, "persistent")
    for i in range(3):
        _same_rays(grid, i, pers, i)
    for i in (1, 2):
        _same_rays(grid, i, _forward([scenes[i]], None, "grid" if dtype == "f16" and not tracer else "ahead"), 0)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "f32-xpair", "f16-xpair", "bf16-xpair"])
@pytest.mark.parametrize("height", [512, 517])
def test_forward_without_checkpoints_agrees_bitwise(dtype, height):
    """4096 and 4160 tiles: beyond 16 per compute unit a call without checkpoints is compiled for 8
    wavefronts per SIMD, one with them for 6 (FP32 for 8)."""
    w = room_workload((31, 28, 36), 512, height, seed=6, ckpt=3, pat=256)
    kept = _scene(w, dtype)
    a = _forward([kept], GRID, "grid")
    b = api.Tracer([kept], GRID, checkpoints=False).forward()
    assert b.ckpt == [None] and b.forms()[0] == "grid"
    for x, y in ((a.uv, b.uv), (a.duv, b.duv), (a.n_steps, b.n_steps), (a.status, b.status)):
        assert torch.equal(x[0].view(torch.uint8), y[0].view(torch.uint8))


@pytest.mark.parametrize("ckpt", [1, 3, 4, 6, 8, 16, 40])
def test_adjoint_coherent_grid_and_persistent(ckpt):
    """1444 tiles: 6 per compute unit, so strides from 8 on take chunks of 4."""
    w = room_workload((20, 24, 16), 304, 304, seed=7, ckpt=ckpt, pat=256)
    _adjoint_pair(w)


@pytest.mark.parametrize("ckpt", [1, 6, 8, 32, 48, 256])
def test_adjoint_coherent_parts_in_chunks_of_3(ckpt):
    """3364 tiles: 14 per compute unit, one round in chunks of 3 and two in chunks of 4. Strides
    over 24 take several parts."""
    w = room_workload((20, 24, 16), 464, 464, seed=8, ckpt=ckpt, pat=256)
    _adjoint_pair(w)


def test_adjoint_quasilinear_grid_and_persistent():
    w = room_workload((20, 24, 16), 304, 304, seed=9, pat=256)
    w.scene = w.scene.replace(tracer=1)
    _adjoint_pair(w)


def _adjoint_pair(w):
    sc = _scene(w)
    seeds = _seeds([sc], 3)
    out = []
    for launch, form in ((GRID, "grid"), (PERSISTENT, "persistent")):
        tr = api.Tracer([sc], launch)
        assert tr.forms()[1] == form
        print(w.scene.dims, w.scene.width, "ckpt", w.scene.ckpt_stride, form, flush=True)
        out.append(tr.forward().adjoint(dL_duv=seeds)[0])
    assert _rel(out[1], out[0]) < 1e-5
    _near(out[0], _gradient(w, sc, seeds[0]))


_SPARSE = {}


def _sparse(tracer):
    """A 24 x 24 camera on a 240 x 240 x 180 room: rays 3-10 cells apart. With the oracle's gradient."""
    if tracer not in _SPARSE:
        w = room_workload((240, 240, 180), 24, 24, seed=7, max_steps=800, pat=256)
        w.scene = w.scene.replace(tracer=tracer)
        sc = _scene(w)
        seeds = _seeds([sc], 8)[0]
        _SPARSE[tracer] = (w, sc, seeds, _gradient(w, sc, seeds))
    return _SPARSE[tracer]


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("tracer,ckpt", [(0, 1), (0, 3), (0, 4), (0, 6), (0, 8), (0, 16), (0, 64), (1, 3)])
def test_coherent_adjoint_with_every_lane_in_its_own_cell(tracer, ckpt, persistent):
    """The sparse camera beside a large one of many rays per cell: the call takes the coherent
    kernels, where one wavefront reduction then follows another for dozens of cells, and the
    32-slot cache of cell totals fills and writes slots out within a chunk."""
    w, sparse, seeds, ref = _sparse(tracer)
    dense = room_workload((20, 24, 16), 304, 304, seed=7, ckpt=ckpt, pat=256)
    dense.scene = dense.scene.replace(tracer=tracer)
    scenes = [_scene(dense), api.Scene(w.scene, sparse.field, sparse.pattern, ckpt_stride=ckpt)]
    tr = api.Tracer(scenes, PERSISTENT if persistent else GRID)
    assert tr.forms()[1] == ("persistent" if persistent else "grid")
    print("tracer", tracer, "ckpt", ckpt, tr.forms(), flush=True)
    _near(tr.forward().adjoint(dL_duv=[_seeds(scenes[:1], 3)[0], seeds])[1], ref)


def _lists(w):
    """Pixel lists of more than 512 tiles: a region, the same in random order, random pixels of the
    whole image, and a list that turns from one into the other, with a ragged last tile."""
    W, H = w.scene.width, w.scene.height
    region = (np.arange(H // 2 - 100, H // 2 + 100)[:, None] * W + np.arange(W // 2 - 85, W // 2 + 85)[None]).ravel()
    spread = np.sort(np.random.default_rng(1).choice(W * H, 34000, replace=False))
    return {"region": region, "shuffled": np.random.default_rng(2).permutation(region), "random": spread,
            "both": np.concatenate([region[:17003], spread[::2]])}


@pytest.mark.parametrize("name", ["region", "shuffled", "random", "both"])
def test_pixel_list_forward_equals_the_image_bitwise(name):
    """A wavefront of a list issues its gathers ahead or not as its pixels lie: the image's bits."""
    w = room_workload((112, 108, 90), 400, 360, seed=3, ckpt=3, pat=256)
    ids = _lists(w)[name]
    tr, image = _forward([_listed(w, ids)], None, "ahead"), _forward([_scene(w)], GRID, "ahead")
    at = torch.from_numpy(ids).to(DEV).long()
    for x, y in ((tr.uv, image.uv), (tr.duv, image.duv), (tr.n_steps, image.n_steps), (tr.status, image.status)):
        assert torch.equal(x[0].view(torch.uint8), y[0][at].view(torch.uint8))


@pytest.mark.parametrize("name,ckpt", [("region", k) for k in (1, 3, 4, 6, 8, 40)] +
                         [("both", k) for k in (1, 3, 4, 6, 8)] + [("shuffled", 3), ("random", 3)])
def test_pixel_list_adjoint(name, ckpt):
    """Lists between two tiles per compute unit and one residency: tiles of few cells go coherent,
    the others by queue, within one launch. 1600 x 1200 pixels: the region's tiles lie in 1 or 2 cells."""
    w = room_workload((20, 24, 16), 1600, 1200, seed=4, ckpt=ckpt, pat=256)
    ids = _lists(w)[name]
    sc = _listed(w, ids)
    seeds = _seeds([sc], 3)
    tr = api.Tracer([sc])
    assert tr.forms()[1] == "queue"
    print(name, "ckpt", ckpt, len(ids), flush=True)
    F = oracle.grid_field(stored_delta(w.T32), w.scene.box_lo, w.scene.box_hi)
    _near(tr.forward().adjoint(dL_duv=seeds)[0], oracle.adjoint(F, w.scene, seeds[0].cpu().numpy().astype(np.float64), ids.astype(np.int32)))


def test_noalloc_adjoint_orders_its_tiles_in_the_scratch():
    """Persistent coherent adjoints: queues, tile costs and order in the static scratch, the second
    call on what the first left there. Bar 1e-12: the FP64 additions in another order."""
    for side, dims, ckpt in ((304, (20, 24, 16), 3), (296, (16, 16, 16), 8)):
        sc = _scene(room_workload(dims, side, side, seed=side, ckpt=ckpt, pat=256))
        tr = api.Tracer([sc], PERSISTENT)
        assert tr.forms()[1] == "persistent"
        seeds = _seeds([sc], 5)
        print(side, dims, ckpt, flush=True)
        a = tr.forward().adjoint(dL_duv=seeds)[0]
        b = tr.adjoint(dL_duv=seeds, noalloc=True)[0]
        assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max())


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


@pytest.mark.parametrize("tracer", [0, 1])
def test_queued_batch_of_views_along_every_axis(tracer):
    """Cameras along +y, +x and -z in one queued call: each scene's voxel table lies along its own
    view."""
    views = [{}, dict(cam_pos=(-1.5, 2.0, 1.5), cam_fwd=(1.0, 0.0, 0.0), cam_right=(0.0, -1.0, 0.0), cam_up=(0.0, 0.0, 1.0),
                      wall_origin=(4.0, 2.0, 1.5), wall_normal=(-1.0, 0.0, 0.0), wall_u=(0.0, -1.0, 0.0), wall_v=(0.0, 0.0, 1.0)),
             dict(cam_pos=(2.0, 2.0, 4.5), cam_fwd=(0.0, 0.0, -1.0), cam_right=(1.0, 0.0, 0.0), cam_up=(0.0, 1.0, 0.0),
                  wall_origin=(2.0, 2.0, 0.0), wall_normal=(0.0, 0.0, 1.0), wall_u=(1.0, 0.0, 0.0), wall_v=(0.0, 1.0, 0.0))]
    ws = []
    for i, view in enumerate(views):
        w = room_workload((60, 68, 56), 120, 112, seed=20 + i, ckpt=3, pat=256)
        w.scene = w.scene.replace(tracer=tracer, **view)
        ws.append(w)
    scenes = [_scene(w) for w in ws]
    seeds = _seeds(scenes, 4)
    tr = api.Tracer(scenes)
    assert tr.forms()[1] == "queue"
    for w, sc, d, g in zip(ws, scenes, seeds, tr.forward().adjoint(dL_duv=seeds)):
        print("view", w.scene.cam_fwd, "tracer", tracer, flush=True)
        _near(g, _gradient(w, sc, d))

"""Parity of the adjoint's forms at the sizes where the launcher changes between them: few
rays per cell or few wavefronts (sums queued per lane), and many wavefronts of coherent rays
(sums reduced per cell), each at every chunk form, both tracers, with ragged tiles, apron
cells on every face, rays that miss the box, pixel lists and batches.

Bars as for every adjoint test: rel-L2 < 1e-3 and per-voxel 1e-3 for all but 0.5 % of the
voxels (the FP32 sweep against the FP64 oracle on the same seeds)."""

import numpy as np
import pytest
import torch

import bos_inputs as bi
import oracle
from _common import grad_errors, room_workload, stored_delta, unit_box_workload
from paper_2509_14442_amd import api

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


WORKLOADS = {
    # 1.9 rays per cell, ragged tiles; every ray meets the box's edge cells on entry and exit
    "unit-box": lambda: unit_box_workload(61, 47),
    # 1 wavefront
    "one-tile": lambda: room_workload((20, 24, 16), 8, 8, seed=5, pat=256),
    # a random pixel list, every lane in a cell of its own
    "pixel-list": lambda: _with_ids(room_workload((64, 64, 48), 200, 150, seed=6, pat=256), 700),
    # 1369 tiles of about 150 rays per cell: the coherent form
    "coherent": lambda: room_workload((20, 24, 16), 296, 296, seed=7, pat=256),
    # 1444 tiles of about 3 rays per cell: the queue form beyond one residency
    "many-sparse": lambda: room_workload((224, 200, 180), 300, 300, seed=8, max_steps=1024, pat=256),
}


def _with_ids(w, count):
    w.pixel_ids = bi.pixel_subset(w.scene.width * w.scene.height, count, 15)
    return w


def _check(w, name, dtype="f32", ckpt=3, launch=None, **replace):
    w.scene = w.scene.replace(ckpt_stride=ckpt, **replace)
    print(f"{name} {dtype} ckpt {ckpt} {replace}", flush=True)
    field = api.Field.from_temperature(torch.from_numpy(w.T32).to(DEV), dtype)
    ids = None if w.pixel_ids is None else torch.from_numpy(w.pixel_ids).to(DEV)
    tr = api.Tracer([api.Scene(w.scene, field, torch.from_numpy(w.pattern32).to(DEV), ids)], launch)
    tr.forward().render()
    seeds = np.random.default_rng(3).standard_normal((tr.scenes[0].n_rays, 2)).astype(np.float32)
    g = tr.adjoint(dL_duv=[torch.from_numpy(seeds).to(DEV)])[0].cpu().numpy()
    F = oracle.grid_field(stored_delta(w.T32, dtype, field.scale, field.offset), w.scene.box_lo, w.scene.box_hi)
    out = oracle.trace(F, w.scene, w.pixel_ids)
    assert np.array_equal(tr.n_steps[0].cpu().numpy(), out["n_steps"])
    assert np.array_equal(tr.status[0].cpu().numpy() & 15, out["status"])
    l2, frac = grad_errors(g, oracle.adjoint(F, w.scene, seeds.astype(np.float64), w.pixel_ids))
    print(f"  rel-L2 {l2:.2e}, voxels off {frac:.1e}")
    assert l2 < 1e-3 and frac <= 5e-3


@pytest.mark.parametrize("ckpt", [1, 3, 4, 6, 8, 16, 24])
@pytest.mark.parametrize("name", ["unit-box", "coherent"])
def test_every_chunk_form(name, ckpt):
    _check(WORKLOADS[name](), name, ckpt=ckpt)


@pytest.mark.parametrize("ckpt", [32, 40, 256])
@pytest.mark.parametrize("persistent", [False, True])
def test_strides_of_several_parts(ckpt, persistent):
    """Segments longer than the 24 steps whose chunk starts the coherent form keeps at once."""
    _check(WORKLOADS["coherent"](), "coherent", ckpt=ckpt, launch=api.make_launch((8, 8), 4, persistent))


@pytest.mark.parametrize("name", ["one-tile", "pixel-list", "many-sparse"])
@pytest.mark.parametrize("ckpt", [3, 16])
def test_sparse_rays(name, ckpt):
    _check(WORKLOADS[name](), name, ckpt=ckpt)


@pytest.mark.parametrize("ckpt", [1, 4, 6, 8])
def test_sparse_rays_one_wavefront_per_tile(ckpt):
    """600 tiles: beyond the form of four wavefronts per tile, each chunk length of the other."""
    w = room_workload((96, 88, 80), 160, 240, seed=9, max_steps=1024, pat=256)
    _check(w, "sparse", ckpt=ckpt)


@pytest.mark.parametrize("name", list(WORKLOADS))
def test_quasilinear(name):
    _check(WORKLOADS[name](), name, tracer=1)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32-xpair", "f16-xpair", "bf16-xpair"])
@pytest.mark.parametrize("name,tracer", [("unit-box", 0), ("unit-box", 1), ("coherent", 0)])
def test_storage_formats(name, tracer, dtype):
    _check(WORKLOADS[name](), name, dtype, tracer=tracer)


@pytest.mark.parametrize("tracer", [0, 1])
def test_samples_per_pixel_and_launch_shapes(tracer):
    for launch in (api.make_launch((16, 4), 4), api.make_launch((8, 8), 2, True), api.make_launch((64, 1), 1)):
        _check(unit_box_workload(40, 33), "spp", launch=launch, tracer=tracer, spp=3, seed=4)


@pytest.mark.parametrize("tracer", [0, 1])
def test_batch_of_sparse_scenes_equals_single_launches(tracer):
    """Scenes of uneven sizes in one call against each alone (FP64 sums in another order)."""
    pat = torch.from_numpy(bi.blurred_noise(12, (256, 256)).astype(np.float32)).to(DEV)
    scenes = []
    for i, (dims, w, h) in enumerate([((30, 22, 26), 40, 24), ((64, 60, 40), 17, 61), ((18, 18, 18), 9, 9)]):
        sc = bi.scene_room(dims, w, h, 512, 3, pat=256).replace(tracer=tracer)
        T = bi.temperature_grid(bi.plumes_room(20 + i, sc.box_lo, sc.box_hi), sc.box_lo, sc.box_hi, sc.dims)
        scenes.append(api.Scene(sc, api.Field.from_temperature(torch.from_numpy(T.astype(np.float32)).to(DEV)), pat))
    rng = np.random.default_rng(4)
    seeds = [torch.from_numpy(rng.standard_normal((s.n_rays, 2)).astype(np.float32)).to(DEV) for s in scenes]
    grads = api.Tracer(scenes).forward().adjoint(dL_duv=seeds)
    for s, d, g in zip(scenes, seeds, grads):
        alone = api.Tracer([s]).forward().adjoint(dL_duv=[d])[0]
        assert float((g - alone).norm() / alone.norm()) < 1e-5

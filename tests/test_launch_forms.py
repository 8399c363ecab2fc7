"""The rule that chooses a call's kernel forms, on the host: rbos_launch_forms validates and
decides as the launching calls do, without a GPU. 256 compute units throughout."""

import ctypes as C
import math

import pytest

import paper_2509_14442_amd._lib as L

CUS = 256


def room(dims=(128, 128, 128), width=512, height=512, stride=3, tracer=0, pixels=0, axis=1, dtype=0):
    """A 4 x 4 x 3 m room seen from 1.5 m in front of a face, 40 degrees wide, along `axis`."""
    s = L.rbos_scene()
    s.nx, s.ny, s.nz = dims
    s.box_lo, s.box_hi = L.D3(0, 0, 0), L.D3(4, 4, 3)
    s.dtype, s.enc_scale, s.enc_offset, s.field = dtype, 1.0, 0.0, 0x1000
    fwd, right, up = [(1, 0, 0), (0, 1, 0), (0, 0, 1)], [(0, 1, 0), (1, 0, 0), (1, 0, 0)], [(0, 0, 1), (0, 0, 1), (0, 1, 0)]
    pos = [2.0, 2.0, 1.5]
    pos[axis] = -1.5
    s.cam_pos, s.cam_fwd = L.D3(*pos), L.D3(*fwd[axis])
    s.cam_right, s.cam_up, s.cam_fov_x_deg = L.D3(*right[axis]), L.D3(*up[axis]), 40.0
    s.width, s.height, s.spp = width, height, 1
    s.n_pixels = pixels or width * height
    s.pixel_ids = 0x2000 if pixels else None
    s.wall_origin, s.wall_normal = L.D3(2, 4, 1.5), L.D3(0, -1, 0)
    s.wall_u, s.wall_v = L.D3(1, 0, 0), L.D3(0, 0, 1)
    voxel = min(4 / dims[0], 4 / dims[1], 3 / dims[2])
    s.step, s.max_steps, s.ckpt_stride, s.tracer = 0.5 * voxel, 16 * math.ceil(7.1 / voxel / 8), stride, tracer
    return s


def forms(*scenes, launch=None, cus=CUS):
    arr = (L.rbos_scene * len(scenes))(*scenes)
    f, a = C.c_int32(-1), C.c_int32(-1)
    L.check(L.load().rbos_launch_forms(arr, len(scenes), C.byref(launch) if launch else None, cus, C.byref(f), C.byref(a)))
    return L.FORMS[f.value], L.FORMS[a.value]


def launch(persistent=0, wpb=4):
    return L.rbos_launch(8, 8, wpb, persistent, 0)


def test_validates_as_the_launching_calls_do():
    lib = L.load()
    f, a = C.c_int32(-1), C.c_int32(-1)
    s = room()
    assert lib.rbos_launch_forms(C.byref(s), 1, None, CUS, None, C.byref(a)) == -1
    assert lib.rbos_launch_forms(C.byref(s), 1, None, 0, C.byref(f), C.byref(a)) == -3
    assert lib.rbos_launch_forms(C.byref(s), 1, C.byref(launch(wpb=3)), CUS, C.byref(f), C.byref(a)) == -3
    s.nx = 1
    assert lib.rbos_launch_forms(C.byref(s), 1, None, CUS, C.byref(f), C.byref(a)) == -2
    assert (f.value, a.value) == (-1, -1) and lib.rbos_last_error()


@pytest.mark.parametrize("tracer", [0, 1])
def test_few_wavefronts_leave_the_launch_shape_unused(tracer):
    small, large = room((64, 64, 48), 96, 80, tracer=tracer), room((128, 128, 128), 1024, 1024, tracer=tracer)
    for shape in (None, launch(), launch(1), launch(1, 2)):
        assert forms(small, launch=shape) == ("ahead", "queue" if tracer else "pipe")
    assert forms(large) == forms(large, launch=launch()) == ("grid", "grid")
    assert forms(large, launch=launch(1)) == ("persistent", "persistent")


@pytest.mark.parametrize("tracer", [0, 1])
@pytest.mark.parametrize("stride", [1, 3, 4, 6, 8, 16])
def test_pixel_lists_are_queued_up_to_one_residency(tracer, stride):
    """Nothing is known on the host of a list but its length: 512 x 512 pixels of a 2048 x 2048
    camera may be a region of it, whose rows hold 22 rays per cell."""
    per_cu = 4 if tracer or stride in (3, 4, 6) else 3  # one-wavefront blocks, by registers and LDS
    for width in (300, 512, 2048, 8192):
        def adjoint(tiles):
            return forms(room(width=width, height=width, stride=stride, tracer=tracer, pixels=64 * tiles))[1]
        assert adjoint(CUS) == ("queue" if tracer else "pipe")
        assert adjoint(CUS + 1) == adjoint(per_cu * CUS) == "queue"
        assert adjoint(per_cu * CUS + 1) == adjoint(4096) == "grid"


def test_a_list_among_images_keeps_the_call_coherent_beyond_one_residency():
    image = room((224, 200, 180), 300, 300)  # 3 rays per cell
    assert forms(image)[1] == forms(image, image)[1] == "queue"
    assert forms(image, room(pixels=64))[1] == "grid"


@pytest.mark.parametrize("stride", [1, 3, 4, 6, 8, 16])
def test_many_rays_per_cell_go_coherent_within_one_residency(stride):
    """700 tiles, beyond the four-wavefront form: about 145, 67 and 16 rays per cell."""
    def adjoint(n):
        return forms(room((n, n, n), 211, 211, stride=stride))[1]
    assert adjoint(24) == ("queue" if stride == 6 else "grid")
    assert adjoint(35) == ("queue" if stride in (3, 6, 8) else "grid")
    assert adjoint(72) == "queue"


def test_long_strides_leave_the_queue_form_by_their_walk():
    """The queue forms walk half a segment to every 8-step chunk: the more rays share a cell, the
    shorter the strides they are taken for."""
    def first_coherent(n, side):
        return next((k for k in (16, 32, 64, 128, 256) if forms(room((n, n, n), side, side, stride=k))[1] == "grid"), None)
    assert first_coherent(32, 160) == 32  # 46 rays per cell, 400 tiles
    assert first_coherent(96, 176) == 256  # 6, 484
    assert first_coherent(192, 160) is None  # 1.3, 400
    assert first_coherent(224, 290) == 128  # 3.1, 1369: two residencies
    assert first_coherent(300, 360) == 64  # 2.7, 2025: three
    assert first_coherent(32, 96) is None  # 144: four wavefronts per tile
    assert forms(room((192, 192, 192), 176, 176, stride=16))[1] == "pipe"
    assert forms(room((192, 192, 192), 176, 176, stride=64))[1] == "queue"
    short = room((96, 96, 96), 176, 176, stride=256)
    short.max_steps = 60  # one segment, cut short
    assert forms(short)[1] == "queue"


def test_second_round_of_four_wavefront_blocks():
    """Between one tile per compute unit and two: for small fields, or few rays per cell and a short
    round."""
    def adjoint(n, side, dtype=0, scenes=1, **kw):
        return forms(*[room((n, n, n), side, side, dtype=dtype, **kw)] * scenes)[1]
    assert adjoint(64, 128) == "pipe"  # 256 tiles
    assert adjoint(96, 136) == "pipe"  # 289 tiles, 3.5 rays per cell
    assert adjoint(96, 150) == adjoint(96, 176) == adjoint(64, 136) == adjoint(64, 176) == "queue"
    assert adjoint(80, 136) == "queue" and adjoint(80, 136, stride=16) == adjoint(80, 136, dtype=1) == "pipe"  # 5
    assert adjoint(64, 136, stride=16) == adjoint(64, 136, dtype=1) == adjoint(64, 136, dtype=3) == "queue"  # 8
    assert adjoint(128, 160) == "pipe" and adjoint(128, 176) == "queue"  # 400 tiles, 2.8; 484, 3.4
    assert adjoint(192, 176) == adjoint(160, 176) == "pipe"  # 484, 1.6 and 2.2
    assert adjoint(50, 176) == adjoint(32, 176) == "pipe"
    assert adjoint(51, 176) == adjoint(51, 176, dtype=3) == "queue"
    assert adjoint(48, 120) == "pipe" and adjoint(48, 120, scenes=2) == "queue"  # 225 tiles; 450 on two fields
    assert adjoint(32, 184) == "queue"  # 529 tiles
    assert adjoint(50, 2048, pixels=64 * 512) == "pipe" and adjoint(50, 2048, pixels=64 * 513) == "queue"
    assert adjoint(51, 2048, pixels=64 * 257) == "queue"


@pytest.mark.parametrize("dtype,least", [(0, 80), (3, 145), (2, 145), (5, 145), (1, None), (4, None)])
def test_gathers_ahead_by_field_size_and_type(dtype, least):
    """Nonlinear forwards: gathers ahead up to two tiles per compute unit, from `least` voxels per axis
    on up to nine; FP16 codes never. Quasi-linear ones up to 16, BF16 up to 4 and, from 67^3 on, 2."""
    def forward(n, side, **kw):
        return forms(room((n, n, n), side, side, dtype=dtype, **kw))[0]
    for n in (24, 64, 79, 80, 144, 145, 224):
        few = "grid" if least is None else "ahead"
        assert forward(n, 64) == forward(n, 176) == few
        assert forward(n, 184) == forward(n, 384) == (few if least is not None and n >= least else "grid")
        assert forward(n, 392) == "grid"
    for n, last in ((24, 512), (66, 512), (67, 512), (224, 512)) if dtype != 2 else ((24, 256), (66, 256), (67, 176), (224, 176)):
        assert forward(n, 64, tracer=1) == forward(n, last, tracer=1) == "ahead"
        assert forward(n, last + 8, tracer=1) == "grid"

"""Masked volumes of 2^23 voxels and more, well above where the mask's cells begin, MI355X
only: inside the mask every output equals the unmasked call's bit for bit, outside
every output is 0 (flags: the outside bit).  The workspace starts as NaNs, so that
nothing a pass left out can reach an output.  Voxels on both sides of cell and tile
edges, runs with gaps of one to four cells between them, axes whose unsplit piece
is longer than the 64 cells a wave looks at together, gradient tiles of 8 and of 4
rows, and replays of a captured batch, whose cells are made anew each time from
where the outputs of the replay before lie."""

import ctypes

import pytest
import torch

import paper_2508_07476_amd as st
from paper_2508_07476_amd._binding import load_library

from test_gpu_parity import DEV, _log

pytestmark = pytest.mark.gpu


def _volume(shape, dtype):
    gen = torch.Generator(device=DEV).manual_seed(shape[0])
    base = torch.rand(shape, generator=gen, device=DEV)
    return base if dtype == "f32" else (base * 60000).round().to(torch.int32).to(torch.uint16)


def _mask(shape):
    """Single voxels at corners and edges, a block, and along each axis runs that
    start in the middle of a cell with 1 to 4 empty cells after them."""
    nz, ny, nx = shape
    m = torch.zeros(shape, dtype=torch.uint8, device=DEV)
    for z, y, x in ((0, 0, 0), (nz - 1, ny - 1, nx - 1), (15, 7, 63), (16, 8, 64), (nz // 2, ny - 1, 0)):
        m[z, y, x] = 1
    m[nz // 3:nz // 3 + 9, 20:45, 50:101] = 1
    for axis, n in enumerate(shape):
        at, gap = 3, 1
        while at < n:
            i = [nz - 3, ny - 5, nx - 7]
            i[axis] = slice(at, min(at + 6, n))
            m[tuple(i)] = 1
            at += 8 * (gap + 1)
            gap = gap % 4 + 1
    return m


def _check(got, whole, m, label):
    for k in whole:
        outside = torch.full_like(whole[k], st.ST_FLAG_OUTSIDE_MASK if k == "flags" else 0)
        assert torch.equal(got[k], torch.where(m != 0, whole[k], outside)), (label, k)


def _axis(shape):
    nz, ny, nx = shape
    return dict(axis_center=(nz / 2, ny / 3, nx / 2 + 0.5), axis_direction=(1.0, 0.1, -0.2))


def _nan_workspace(shape):
    return torch.full((st.st_workspace_bytes(shape) // 4,), float("nan"), device=DEV).view(torch.uint8)


CASES = [
    ((130, 250, 260), "u16", 1.0, 1.0),
    ((70, 420, 300), "f32", 1.5, 4.0),
    ((600, 130, 111), "u16", 2.0, 8.0),
    ((274, 1100, 320), "u16", 0.5, 1.0),   # y pieces of 550: cells of two looks
    ((1100, 274, 320), "u16", 0.5, 1.0),   # z pieces of 550
]


@pytest.mark.parametrize("shape,dtype,sigma,rho", CASES)
def test_masked_equals_unmasked_inside(shape, dtype, sigma, rho):
    _log("case: masked runs", shape, dtype, sigma, rho)
    assert shape[0] * shape[1] * shape[2] >= 1 << 23
    vol, m = _volume(shape, dtype), _mask(shape)
    if max(shape) > 1000:  # beyond the first look of a piece only, and on both sides of its end
        long = shape.index(max(shape))
        i = [slice(100, 104), slice(100, 104), slice(100, 104)]
        for a, b in ((505, 519), (530, 534), (1090, 1100)):
            i[long] = slice(a, b)
            m[tuple(i)] = 1
            i[2] = slice(i[2].start + 64, i[2].stop + 64)
    kw = dict(outputs=st.ALL_OUTPUTS, **_axis(shape))
    whole = st.st_compute(vol, sigma, rho, **kw)
    got = st.st_compute(vol, sigma, rho, mask=m, workspace=_nan_workspace(shape), **kw)
    torch.cuda.synchronize()
    _check(got, whole, m, str(shape))


class _LaunchShape(ctypes.Structure):
    _fields_ = [("grad_min_blocks", ctypes.c_int64), ("strided_min_waves", ctypes.c_int64),
                ("grad_rows", ctypes.c_int), ("xfinal_lanes", ctypes.c_int), ("rest", ctypes.c_int64 * 4)]


@pytest.mark.parametrize("sigma", [1.0, 1.5])
def test_gradient_tiles_of_four_rows(sigma):
    """The launch shape that the batch autotuner may take at these radii, given to
    the library's own pass sequence: two tiles then share a row of cells."""
    shape, rho = (130, 250, 260), 2.0
    _log("case: masked, 4-row tiles", shape, sigma)
    vol, m, ax = _volume(shape, "u16"), _mask(shape), _axis(shape)
    whole = st.st_compute(vol, sigma, rho, outputs=st.ALL_OUTPUTS, **ax)
    out = {k: torch.full_like(v, 7) for k, v in whole.items()}
    ws = _nan_workspace(shape)
    lib = load_library()
    prepare = lib._ZN2st4host12prepare_pathERNS0_8PathArgsEPKviPKhllldddPKdS8_PfS9_S9_S9_S9_Ph
    enqueue = lib._ZN2st4host12enqueue_pathERKNS0_8PathArgsEPcP12ihipStream_tRKNS0_11LaunchShapeEbPPKc
    P, D, L = ctypes.c_void_p, ctypes.c_double, ctypes.c_int64
    prepare.argtypes = [P, P, ctypes.c_int, P, L, L, L, D, D, D, P, P, P, P, P, P, P, P]
    enqueue.argtypes = [P, P, P, P, ctypes.c_bool, P]
    prepare.restype = enqueue.restype = ctypes.c_int
    args = ctypes.create_string_buffer(4096)
    center, direction = (D * 3)(*ax["axis_center"]), (D * 3)(*ax["axis_direction"])
    assert prepare(args, vol.data_ptr(), st.ST_DTYPE_U16, m.data_ptr(), *shape, sigma, rho, 4.0, center, direction,
                   *(out[k].data_ptr() for k in ("e3", "evals", "fa", "ha", "ia", "flags"))) == 0
    launch = _LaunchShape(1024, 16384, 4, 0)
    stage = ctypes.c_char_p()
    assert enqueue(args, ws.data_ptr(), torch.cuda.current_stream().cuda_stream, ctypes.byref(launch), False,
                   ctypes.byref(stage)) == 0, stage.value
    torch.cuda.synchronize()
    _check(out, whole, m, f"4 rows, sigma {sigma}")


def test_replayed_batch_makes_its_cells_anew():
    shape = (130, 250, 260)
    _log("case: masked batch replays", shape)
    vols, m = [_volume(shape, "u16"), _volume((131,) + shape[1:], "u16")[:130].contiguous()], _mask(shape)
    ax = _axis(shape)
    whole = [st.st_compute(v, 1.0, 2.0, outputs=st.ALL_OUTPUTS, **ax) for v in vols]
    batch = st.Batch([{"volume": v, "mask": m, "rho": 2.0, "origin": (0.0, 0.0, 0.0)} for v in vols], sigma=1.0,
                     outputs=st.ALL_OUTPUTS, lanes=1, **ax)
    assert batch.plan()["kernels"] == 12  # the cells' two kernels are in the graph of each
    for _ in range(3):
        batch.launch()
        torch.cuda.synchronize()
        for got, want in zip(batch.results, whole):
            _check(got, want, m, "replay")
            for v in got.values():
                v.fill_(7)
    m.copy_(_mask(shape).flip(0))  # the cells follow the mask as it is at the launch
    batch.launch()
    torch.cuda.synchronize()
    for got, want in zip(batch.results, whole):
        _check(got, want, m, "another mask")
    batch.close()

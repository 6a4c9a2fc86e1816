"""The surrogate's layers at the edges of their tiles (MI355X only), against the
FP64 oracle with the tolerances derived beside the other inference tests: 16 x
32 voxel tiles one short, full and one over, a single plane, and more planes
than one block takes."""

import pytest
import torch

import paper_2508_07476_amd as st
from oracle import surrogate as S

from test_gpu_surrogate import DEV, _check, _inputs, _log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 15, 31), (2, 16, 32), (3, 17, 33), (70, 16, 33)])
def test_layers_at_tile_edges(shape):
    _log("case: surrogate layers at tile edges", shape)
    vol, _, blob, center, direction, _ = _inputs(shape, "f32", False, 21)
    g = st.st_surrogate_infer(vol.to(DEV), torch.from_numpy(blob).to(DEV), axis_center=center,
                              axis_direction=direction, outputs=st.SURROGATE_OUTPUTS)
    torch.cuda.synchronize()
    _check({k: v.double().cpu().numpy() for k, v in g.items()}, S.forward(vol.numpy(), blob), None, center, direction,
           label=str(shape))


@pytest.mark.parametrize("slab_bytes", [None, 70 * 130 * 140 * 64])
def test_masked_network_equals_unmasked_inside(slab_bytes, monkeypatch):
    """With a mask only the tiles near it are computed: inside it every output
    equals the unmasked run's bit for bit, outside every output is 0.  Single
    voxels at corners and tile edges, a slab of planes, an empty z range; whole
    and in z slabs."""
    shape = (70, 130, 140)
    _log("case: masked network", shape, "slab bytes", slab_bytes)
    if slab_bytes is not None:
        monkeypatch.setenv("ST_SURROGATE_SLAB_BYTES", str(slab_bytes))
    vol, _, blob, center, direction, _ = _inputs(shape, "f32", False, 22)
    mask = torch.zeros(shape, dtype=torch.uint8)
    for z, y, x in ((0, 0, 0), (69, 129, 139), (5, 15, 31), (5, 16, 32), (9, 64, 63), (33, 48, 96)):
        mask[z, y, x] = 1
    mask[20:24, 70:100, 30:75] = 1
    kw = dict(axis_center=center, axis_direction=direction, outputs=st.SURROGATE_OUTPUTS)
    w = torch.from_numpy(blob).to(DEV)
    whole = st.st_surrogate_infer(vol.to(DEV), w, **kw)
    out = {k: torch.full_like(v, 7.0) for k, v in whole.items()}
    got = st.st_surrogate_infer(vol.to(DEV), w, mask=mask.to(DEV), out=out, **kw)
    torch.cuda.synchronize()
    for k in whole:
        assert torch.equal(got[k], torch.where(mask.to(DEV) != 0, whole[k], torch.zeros_like(whole[k]))), k

"""The surrogate on masked volumes of 2^23 voxels, in both of the chunk lengths that the
kernels choose by how much work a mask leaves, MI355X only: inside the mask every output equals the unmasked run's bit for
bit, outside every output is 0.  Single voxels at corners and tile edges, a slab of
planes, an empty z range; whole and in z slabs."""

import pytest
import torch

import paper_2508_07476_amd as st

from test_gpu_surrogate import DEV, _inputs, _log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tissue", ["few", "many", "none"])
@pytest.mark.parametrize("slab_bytes", [None, 2 * 50 * 250 * 261 * 64])
def test_masked_network_equals_unmasked_inside(slab_bytes, tissue, monkeypatch):
    shape = (130, 250, 261)
    assert shape[0] * shape[1] * shape[2] >= 1 << 23
    _log("case: masked network", shape, "slab bytes", slab_bytes, tissue)
    if slab_bytes is not None:
        monkeypatch.setenv("ST_SURROGATE_SLAB_BYTES", str(slab_bytes))
    _, _, blob, center, direction, _ = _inputs((6, 6, 6), "f32", False, 22)
    gen = torch.Generator(device=DEV).manual_seed(4)
    vol = torch.rand(shape, generator=gen, device=DEV) * 65535.0
    mask = torch.zeros(shape, dtype=torch.uint8, device=DEV)
    if tissue == "many":  # a voxel in every column of 16 x 32, at different depths
        mask[:, 7::16, 5::32] = (torch.arange(130, device=DEV) % 37 == 11).to(torch.uint8).view(-1, 1, 1)
    for z, y, x in () if tissue == "none" else ((0, 0, 0), (129, 249, 260), (5, 15, 31), (5, 16, 32), (9, 64, 63), (63, 48, 96), (41, 200, 130)):
        mask[z, y, x] = 1
    if tissue == "few":
        mask[20:24, 70:100, 30:75] = 1
    kw = dict(axis_center=center, axis_direction=direction, outputs=st.SURROGATE_OUTPUTS)
    w = torch.from_numpy(blob).to(DEV)
    whole = st.st_surrogate_infer(vol, w, **kw)
    out = {k: torch.full_like(v, 7.0) for k, v in whole.items()}
    got = st.st_surrogate_infer(vol, w, mask=mask, out=out, **kw)
    torch.cuda.synchronize()
    for k in whole:
        assert torch.equal(got[k], torch.where(mask != 0, whole[k], torch.zeros_like(whole[k]))), k

"""Large masked volumes compute only what the mask needs (MI355X only): inside the
mask every output equals the unmasked call's bit for bit, outside every output is
0 (flags: the outside bit).  The workspace starts as NaNs, so that nothing a pass
left out can reach an output.  Masks with single voxels at corners and on both
sides of cell and tile edges, a block, long empty stretches; widths on and off
the cells' 64; each gradient tile form; integration radii 4, 16 and 32; the mask
8-byte aligned and not."""

import pytest
import torch

import paper_2508_07476_amd as st

from test_gpu_parity import DEV, _log

pytestmark = pytest.mark.gpu

CASES = [
    ((130, 180, 192), "u16", 1.0, 1.0),
    ((70, 300, 205), "f32", 1.5, 4.0),
    ((600, 66, 111), "u16", 2.0, 8.0),
]


@pytest.mark.parametrize("shape,dtype,sigma,rho", CASES)
@pytest.mark.parametrize("shift", [0, 1])
def test_masked_equals_unmasked_inside(shape, dtype, sigma, rho, shift):
    _log("case: masked path", shape, dtype, sigma, rho, "mask shift", shift)
    nz, ny, nx = shape
    n = nz * ny * nx
    assert n >= 1 << 22
    gen = torch.Generator().manual_seed(nz)
    base = torch.rand(shape, generator=gen)
    vol = ((base * 60000).round().to(torch.int32).to(torch.uint16) if dtype == "u16" else base).to(DEV)
    mask = torch.zeros(shape, dtype=torch.uint8)
    for z, y, x in ((0, 0, 0), (nz - 1, ny - 1, nx - 1), (15, 7, 63), (16, 8, 64), (nz // 2, ny - 1, 0)):
        mask[z, y, x] = 1
    mask[nz // 3:nz // 3 + 9, 20:45, 50:101] = 1
    mask[nz - 30:nz - 25, ny // 2:, :9] = 1
    buf = torch.empty(n + shift, dtype=torch.uint8, device=DEV)
    m = buf[shift:].view(shape)
    m.copy_(mask)
    kw = dict(axis_center=(nz / 2, ny / 3, nx / 2 + 0.5), axis_direction=(1.0, 0.1, -0.2), outputs=st.ALL_OUTPUTS)
    whole = st.st_compute(vol, sigma, rho, **kw)
    ws = torch.full((st.st_workspace_bytes(shape) // 4,), float("nan"), device=DEV).view(torch.uint8)
    got = st.st_compute(vol, sigma, rho, mask=m, workspace=ws, **kw)
    torch.cuda.synchronize()
    for k in whole:
        outside = torch.full_like(whole[k], st.ST_FLAG_OUTSIDE_MASK if k == "flags" else 0)
        assert torch.equal(got[k], torch.where(m != 0, whole[k], outside)), k

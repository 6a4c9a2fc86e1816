"""st_angles at the edges of its two access forms (MI355X only) against the FP64
oracle's frame: voxel counts on both sides of a multiple of four, one wave's and
one block's voxels, and buffers that do not start on 16 bytes.  The kernel's
frame is float64 and its angles float32 (relative error of a few 1e-7 of terms
below pi / 2, and the arguments' rounding divided by the projection, here at
least 0.1): 2e-5 rad.  Mask and axis bits are compared exactly."""

import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2508_07476_amd as st

from _parity import wrap_pi

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 2e-5


def _place(a, shift):
    """The array on the GPU, its first element `shift` elements into an allocation."""
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    buf = torch.empty(t.numel() + shift, dtype=t.dtype, device=DEV)
    out = buf[shift:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (2, 16, 32), (1, 1, 1027), (5, 3, 68)])
@pytest.mark.parametrize("shift", [0, 1])
def test_angles_at_access_edges(shape, shift):
    print("case: angles", shape, "shift", shift, file=sys.stderr, flush=True)
    rng = np.random.default_rng(7)
    e3 = rng.normal(size=(3,) + shape)
    e3 /= np.linalg.norm(e3, axis=0, keepdims=True)
    e3 = e3.astype(np.float32)
    mask = (rng.random(shape) < 0.8).astype(np.uint8)
    center, direction = tuple(float(n // 2) for n in shape), (1.0, 0.2, -0.1)
    out = {k: _place(np.zeros(shape, np.float32), shift) for k in ("ha", "ia")}
    out["flags"] = _place(np.zeros(shape, np.uint8), shift)
    g = st.st_angles(_place(e3, shift), center, direction, mask=_place(mask, shift), outputs=("ha", "ia", "flags"), out=out)
    torch.cuda.synchronize()
    ha, ia, flags = (g[k].cpu().numpy() for k in ("ha", "ia", "flags"))
    frame = oracle.cylindrical_frame(shape, center, direction)
    ho, io, on = oracle.helix_intrusion(e3.astype(np.float64), frame)
    e_r, e_t, a, r = frame
    inside = mask != 0
    assert np.array_equal(flags, np.where(inside, np.where(on, st.ST_FLAG_ON_AXIS, 0), st.ST_FLAG_OUTSIDE_MASK))
    assert np.all(ha[~inside] == 0) and np.all(ia[~inside] == 0)
    f_r, f_t = (e3 * e_r).sum(0), (e3 * e_t).sum(0)
    f_a = (e3 * a.reshape(3, 1, 1, 1)).sum(0)
    for got, want, proj in ((ha, ho, np.hypot(f_t, f_a)), (ia, io, np.hypot(f_t, f_r))):
        sel = inside & (r >= 1) & (proj >= 0.1)
        d = wrap_pi(got[sel] - want[sel])
        assert d.size == 0 or d.max() <= TOL, d.max()

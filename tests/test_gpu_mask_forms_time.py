"""What a mask leaves out is left out of the time (MI355X only).  The times are
compared within one process and one volume, and the bounds lie half way between
what the pass takes with and without the work in question."""

import os

import numpy as np
import pytest
import torch

import paper_2508_07476_amd as st

from test_gpu_parity import DEV, _log

pytestmark = pytest.mark.gpu


def _pass_times(vol, mask, sigma, rho, outputs, n=20):
    """Microseconds of each pass, the least of three means over n calls."""
    ws = torch.empty(st.st_workspace_bytes(vol.shape), dtype=torch.uint8, device=DEV)
    out = st.st_compute(vol, sigma, rho, mask=mask, outputs=outputs, workspace=ws)
    best = {}
    for _ in range(3):
        torch.cuda.synchronize()
        st.profile_reset()
        st.profile_enable(True)
        for _ in range(n):
            st.st_compute(vol, sigma, rho, mask=mask, outputs=outputs, out=out, workspace=ws)
        torch.cuda.synchronize()
        got = st.profile_read()
        st.profile_enable(False)
        for k, (ms, calls) in got.items():
            best[k] = min(best.get(k, float("inf")), 1e3 * ms / calls)
    return best


@pytest.mark.parametrize("shape", [(160, 256, 512), (100, 300, 200)])
def test_final_pass_skips_voxel_positions_without_tissue(shape):
    """Tissue in every 64th plane along x: a wave's lanes hold it at one of their
    four voxels, and the eigen-decomposition, half of the pass, runs for that one
    only.  Both segment widths (64 and 16 lanes)."""
    _log("case: final pass, planes along x", shape)
    vol = torch.rand(shape, device=DEV)
    full = torch.ones(shape, dtype=torch.uint8, device=DEV)
    planes = torch.zeros_like(full)
    planes[:, :, ::64] = 1
    t_full = _pass_times(vol, full, 1.0, 1.0, ("fa",))["integrate_x_eigen"]
    t_planes = _pass_times(vol, planes, 1.0, 1.0, ("fa",))["integrate_x_eigen"]
    _log(f"final pass: full mask {t_full:.1f} us, planes {t_planes:.1f} us")
    assert t_planes < 0.8 * t_full


def _surrogate_time(vol, mask, weights, n=12):
    """Microseconds a call, the least of five means over n calls in a row."""
    kw = dict(axis_center=(60.0, 20.0, 70.0), axis_direction=(1.0, 0.0, 0.1), outputs=st.SURROGATE_OUTPUTS, mask=mask)
    out = st.st_surrogate_infer(vol, weights, **kw)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(5):
        a.record()
        for _ in range(n):
            st.st_surrogate_infer(vol, weights, out=out, **kw)
        b.record()
        torch.cuda.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / n)
    return best


@pytest.mark.parametrize("shape,tissue,most", [((128, 128, 128), "all", 1.14), ((316, 48, 143), "ring", 0.75)])
def test_surrogate_layers_split_by_the_work(shape, tissue, most):
    """Neither a full mask pays for chunks that suit an empty one, nor a ring in a
    long plane, which fills a fifth of it, for chunks that suit a full one."""
    _log("case: surrogate, masked", shape, tissue)
    nz, ny, nx = shape
    vol = (torch.rand(shape, device=DEV) * 60000).round().to(torch.int32).to(torch.uint16)
    weights = torch.from_numpy(np.load(os.path.join(os.path.dirname(st.__file__), "surrogate_weights.npy"))).to(DEV)
    y = (torch.arange(ny, device=DEV) - (ny - 1) / 2).view(1, ny, 1)
    x = (torch.arange(nx, device=DEV) - (nx - 1) / 2).view(1, 1, nx)
    r = torch.sqrt(y * y + x * x) / min(ny, nx)
    mask = (torch.ones(shape, dtype=torch.uint8, device=DEV) if tissue == "all"
            else ((r >= 0.1875) & (r <= 0.4375)).expand(shape).to(torch.uint8).contiguous())
    t_none, t_mask = _surrogate_time(vol, None, weights), _surrogate_time(vol, mask, weights)
    _log(f"surrogate: no mask {t_none:.1f} us, {tissue} {t_mask:.1f} us")
    assert t_mask < most * t_none

"""What a mask leaves out is left out of the time (MI355X only).  The times are
compared within one process and one volume, and the bounds lie half way between
what the pass takes with and without the work in question."""

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

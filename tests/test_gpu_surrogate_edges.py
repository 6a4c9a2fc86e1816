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

"""The training kernels at the edges of their tiles (MI355X only), against the
FP64 oracle with the tolerances derived beside the other gradient tests: one
y tile more or less than full (11, 17, 25 rows against tiles of 8), rows one
short of an MFMA step (31), and more planes than weight-gradient blocks, with a
short last chunk (26 patches of 11 planes over 128 chunks of 3)."""

import pytest

from test_gpu_surrogate_train import _case, _compare, _gpu, _log, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npatch,P,dtype", [(1, 11, "f32"), (26, 11, "u16"), (2, 17, "u16"), (1, 25, "f32"),
                                            (1, 31, "u16")])
def test_gradient_at_tile_edges(npatch, P, dtype):
    _log("case: surrogate gradient at tile edges", npatch, P, dtype)
    case = _case(100 + npatch + P, npatch, P, dtype)
    g, s = _gpu(*case)
    _compare(g, s, _oracle(*case, npatch, P))

"""The path at the edges of its passes' blocks and pieces (MI355X only) against
the FP64 oracle, with the path's tolerances: integration axes one short of, equal
to and one past the register window (9 samples at rho radius 4) and whole
multiples of it, rows on both sides of 64 columns, and small volumes whose axes
are cut into many pieces.  Gradient radii 1 to 8 with odd and even numbers of
planes (which are filtered in pairs), from fewer than a window's slots to one
past a multiple of them."""

import pytest
import torch

from test_gpu_parity import _log, _run_both

from _parity import assert_parity, compare, summary

pytestmark = pytest.mark.gpu

CASES = [
    ((8, 9, 63), "u16", 0.5, 1.0),
    ((10, 18, 65), "f32", 0.5, 1.0),
    ((19, 27, 1), "u16", 0.5, 1.0),
    ((28, 36, 130), "f32", 1.0, 1.0),
    ((61, 40, 70), "u16", 1.0, 3.0),    # pieces of both axes
    ((25, 24, 200), "f32", 1.75, 4.0),  # 4-row gradient tiles, a 33-sample window
]

PAIRS = [
    ((4, 9, 65), "u16", 0.25, 1.0),    # radius 1: four slots
    ((7, 8, 64), "f32", 0.5, 1.0),
    ((9, 7, 63), "u16", 0.75, 1.0),
    ((10, 17, 66), "f32", 1.0, 1.0),
    ((12, 15, 128), "u16", 1.25, 1.0),
    ((15, 16, 129), "f32", 1.5, 1.0),
    ((16, 5, 67), "u16", 1.75, 1.0),
    ((19, 11, 80), "u16", 2.0, 1.0),   # radius 8: eighteen slots, and one plane more
    ((2, 12, 70), "f32", 2.0, 1.0),
]


@pytest.mark.parametrize("shape,dtype,sigma,rho", CASES + PAIRS)
def test_pass_edges(shape, dtype, sigma, rho):
    _log("case: pass edges", shape, dtype, sigma, rho)
    gen = torch.Generator().manual_seed(shape[0] * 1000 + shape[2])
    base = torch.rand(shape, generator=gen, dtype=torch.float64)
    vol = (base * 60000).round().to(torch.int32).to(torch.uint16) if dtype == "u16" else base.to(torch.float32)
    mask = (torch.rand(shape, generator=gen) > 0.25).to(torch.uint8)
    center, direction = tuple((n - 1) / 2 + 0.25 for n in shape), (1.0, 0.2, -0.3)
    g, o = _run_both(vol, sigma, rho, mask, center, direction)
    stats = compare(g, o, shape, center, direction, mask=mask.numpy())
    _log(summary(stats))
    assert_parity(stats, str(shape))

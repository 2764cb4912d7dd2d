"""GPU parity of the 64 x 64 NS kernel whose waves share a tile's K slices
(the planner's choice for launches of few tiles) against the fp64 oracle.

Sides around its tile (64), its wave quadrant (32) and its K slice (32, one in
four per wave): units of one partial tile, one tile exactly, a tile and a
row of chunks, fewer slices than waves, a slice cut by K, and K just past a
round of the four waves; transposed and untransposed, iterated as printed and
on the Gram matrix, read in place and packed, with the NT apply, Nesterov and
per-iteration coefficients.  Bars: the bf16 parity bars of the other GPU tests
(operands rounded to bf16 after every product).
"""

import pytest

from tests.gpu_harness import Case, announce, run_case

pytestmark = pytest.mark.gpu

TOL = 2e-2


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2510_16981_amd import muonbp as mb
    mb.load_library()


CASES = {
    "one partial tile": dict(mats=[(8, 24, 1, 1)]),
    "one tile": dict(mats=[(64, 64, 1, 1)]),
    "a tile and a chunk": dict(mats=[(72, 136, 1, 1), (136, 72, 1, 1)]),
    "quadrant edges": dict(mats=[(32, 96, 1, 1), (40, 104, 1, 1), (96, 40, 1, 1)]),
    "slices around four waves": dict(mats=[(64, 120, 1, 1), (64, 128, 1, 1), (64, 136, 1, 1), (64, 264, 1, 1)]),
    "gram-space, in place and transposed": dict(mats=[(128, 512, 1, 2), (512, 128, 1, 1), (200, 1000, 1, 1)], rank=64),
    "blocks and whole": dict(mats=[(256, 384, 2, 2)], period=2, rank=64),
    # Rank 128: these coefficients multiply small singular values by 3.4 and
    # then 2 a step, bf16 rounding with them, and a rank-16 signal's worst tile
    # is 2.5% from fp64 on any of the bf16 kernels (128 x 128 tiles: 2.55%).
    "nesterov, coefficients, fp32 weights": dict(mats=[(136, 328, 1, 1), (328, 136, 1, 1)], nesterov=1, param="f32",
                                                 state="f32", rank=128, coeffs=[(3.4445, -4.7750, 2.0315), (2.0, -1.5, 0.5)]),
    "NT apply": dict(mats=[(72, 200, 1, 1), (200, 72, 1, 1)], apply_mode=1),
    "one iteration": dict(mats=[(104, 264, 1, 1)], ns_steps=1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_wave_k_kernel(name):
    from paper_2510_16981_amd import muonbp as mb
    case = Case(**{**dict(period=1, steps=2, rank=16, seed=5), **CASES[name]})
    opts = mb.options_default(ns_steps=case.ns_steps, apply_mode=case.apply_mode)
    info = mb.describe_plan(case.mats, case.period == 1, opts)
    assert list(info.gemm_tile_rows) == [64] * 3 and list(info.gemm_tile_cols) == [64] * 3
    announce(f"{name}: {case}")
    w = run_case(case).worst()
    announce(f"worst errors {w}")
    assert w["u"] <= TOL and w["u_unit"] <= TOL and w["u_tile"] <= TOL, w
    assert w["m"] <= TOL and w["x"] <= TOL, w
    assert w["m_ulp"] <= 1.0 and w["x_ulp"] <= 1.0, w

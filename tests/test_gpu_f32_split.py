"""GPU parity of the fp32 NS kernels that split their operands into three
bf16 parts, against the fp64 oracle and against the fp32 MFMA kernels
(tile_policy = 1).

The three tile shapes the planner picks from (32 x 32 with the K slices shared
by the waves, 64 x 64, 128 x 128), at sides around their tiles, wave sub-tiles
and 32-column slices, K of every remainder by 4, fewer slices than waves and
fewer than the pipeline's three, transposed and untransposed units.

Bars: with fp32 products and sums U was 0.4e-6 to 1.4e-6 from fp64 (sides from
33 to 4096, K to 40000); 3e-6 is twice the worst of them, and a 64 x 64 tile
of a few small entries may be three times that.  The split kernels measure
0.2e-6 to 0.7e-6.
"""

import numpy as np
import pytest

from tests.gpu_harness import Case, announce, rel, run_case

pytestmark = pytest.mark.gpu

TOL, TOL_TILE = 3e-6, 1e-5


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2510_16981_amd import muonbp as mb
    mb.load_library()


def _many(r, c, n):
    return [(r, c, 1, 1)] * n


# name: (matrices, tile rows of Gram, polynomial, apply)
CASES = {
    "single row and column": ([(1, 7, 1, 1), (5, 1, 1, 1)], [32, 32, 32]),
    "32: edges": ([(31, 33, 1, 1), (32, 64, 1, 1), (33, 95, 1, 1), (65, 34, 1, 1)], [32, 32, 32]),
    "32: K remainders": ([(24, 129, 1, 1), (24, 130, 1, 1), (24, 131, 1, 1), (132, 24, 1, 1)], [32, 32, 32]),
    "64: edges": (_many(513, 577, 2) + _many(578, 514, 2), [64, 64, 64]),
    "128: edges": (_many(1281, 1153, 5) + _many(1150, 1282, 3), [128, 64, 128]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_kernels(name):
    from paper_2510_16981_amd import muonbp as mb
    mats, rows = CASES[name]
    f32 = dict(param="f32", state="f32", ns="f32")
    info = mb.describe_plan(mats, True, mb.options_default(param_dtype=mb.F32, state_dtype=mb.F32, ns_dtype=mb.F32))
    announce(f"{name}: tiles {list(info.gemm_tile_rows)}")
    assert list(info.gemm_tile_rows) == rows
    case = dict(mats=mats, period=1, steps=1, rank=16, seed=3, **f32)
    new, old = run_case(Case(**case), keep_updates=True), run_case(Case(tile_policy=1, **case), keep_updates=True)
    w = new.worst()
    announce(f"worst errors {w}, fp32 MFMA {old.worst()}")
    assert w["u"] <= TOL and w["u_unit"] <= TOL and w["u_tile"] <= TOL_TILE, w
    assert w["m_ulp"] <= 1.0 and w["x_ulp"] <= 1.0, w
    for a, b in zip(new.updates[0], old.updates[0]):
        assert rel(np.asarray(a, np.float64), np.asarray(b, np.float64)) <= 2 * TOL


def test_non_finite_input_spreads():
    """An Inf or NaN in a unit's input leaves no finite entry in its U, and
    does not touch another unit."""
    import torch
    from paper_2510_16981_amd import muonbp as mb
    for bad in (float("inf"), float("nan")):
        opt = mb.MuonBP([(48, 80, 1, 1), (48, 80, 1, 1)], 1, 0.02, 0.02, 0.95,
                        options=mb.options_default(param_dtype=mb.F32, state_dtype=mb.F32, ns_dtype=mb.F32))
        g = [torch.randn(48, 80, device="cuda") for _ in range(2)]
        g[0][7, 11] = bad
        opt.step([torch.zeros(48, 80, device="cuda") for _ in range(2)], g, 0)
        u = [opt.get_update(k) for k in range(2)]
        assert not torch.isfinite(u[0]).any() and torch.isfinite(u[1]).all()
        opt.close()


def test_columns_past_the_tile_index_of_narrow_tiles():
    """2200000 columns are more 32-wide tiles than a tile index holds: beside
    30000 small units (whose launches prefer those tiles) every column of U is
    still written."""
    import torch
    from oracle import muonbp_oracle as O
    from paper_2510_16981_amd import muonbp as mb
    mats = [(1, 2200000, 1, 1), (8, 240000, 1, 30000)]
    opt = mb.MuonBP(mats, 0, 0.02, 0.02, 0.95,
                    options=mb.options_default(param_dtype=mb.F32, state_dtype=mb.F32, ns_dtype=mb.F32))
    gen = torch.Generator().manual_seed(5)
    g = [torch.randn(r, c, generator=gen) for r, c, _, _ in mats]
    announce("1 x 2200000 beside 30000 units of 8 x 8, fp32 block step")
    opt.step([torch.zeros(r, c, device="cuda") for r, c, _, _ in mats], [x.cuda() for x in g], 0)
    u = [opt.get_update(k).double().cpu().numpy() for k in range(2)]
    opt.close()
    y = [x.double().numpy() for x in g]
    ref = O.orthogonalize_via_ns(y[0])
    assert rel(u[0], ref) <= TOL and rel(u[0][:, 2097152:], ref[:, 2097152:]) <= TOL
    for c in (0, 8 * 12345, 240000 - 8):
        assert rel(u[1][:, c:c + 8], O.orthogonalize_via_ns(y[1][:, c:c + 8])) <= TOL

"""Steps with the plan of the smallest tables and workspace, which a context
takes where its device_memory_limit leaves no room for the preferred one, and
the allocation-free step where the static array does not.

bf16: limits one byte below the preferred plan's bulk (device_bytes), so that
only the other plan fits; odd sides then run the register K loop with the Z^T
pair, and units of a mixed plan iterate as printed.  fp32: the two differ in
their tile lists only, so the smallest limit that is accepted is the other
plan's.  Compared with the fp64 oracle at the parity bars; the allocation-free
step bit for bit with such a context.
"""

import ctypes

import pytest

from tests.gpu_harness import Case, announce, run_case

pytestmark = pytest.mark.gpu

# The parity bars (relative Frobenius, of units and of 64 x 64 tiles): 2e-2 for
# bf16; fp32 as for the fp32 kernels elsewhere (the worst seen with fp32 products
# is 1.4e-6).
BARS = {"bf16": (2e-2, 2e-2), "f32": (3e-6, 1e-5)}


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2510_16981_amd import muonbp as mb
    mb.load_library()


def _options(dtype, **kw):
    from paper_2510_16981_amd import muonbp as mb
    d = mb.F32 if dtype == "f32" else mb.BF16
    return mb.options_default(param_dtype=d, state_dtype=d, ns_dtype=d, **kw)


def _smallest_limit(mats, dtype, start):
    """The smallest limit accepted, in steps of 1 KB (less than the tile lists
    of the two plans differ by)."""
    from paper_2510_16981_amd import muonbp as mb
    lib = mb.load_library()
    for limit in range(start, start + (1 << 20), 1024):
        ctx = ctypes.c_void_p()
        o = _options(dtype, device_memory_limit=limit)
        st = lib.muonbp_create(mb._mats(mats), len(mats), 2, 0.013, 0.02, 0.95, 0.1, ctypes.byref(o), None,
                               ctypes.byref(ctx))
        if st == 0:
            lib.muonbp_destroy(ctx)
            return limit
        assert st == 4
    raise AssertionError("no limit accepted")


CASES = {
    "odd sides": ("bf16", [(333, 420, 3, 2), (230, 200, 1, 1)]),
    "mixed plan": ("bf16", [(512, 512, 1, 1), (512, 2048, 1, 2), (640, 320, 1, 1)]),
    "odd beside wide": ("bf16", [(501, 640, 1, 1), (256, 1024, 1, 4)]),
    "fp32": ("f32", [(200, 300, 1, 1), (300, 200, 2, 1), (33, 500, 1, 2), (129, 129, 1, 1)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_context_under_a_limit(name):
    from paper_2510_16981_amd import muonbp as mb
    dtype, mats = CASES[name]
    bulk = mb.describe_plan(mats, True, _options(dtype)).device_bytes
    limit = bulk - 1 if dtype == "bf16" else _smallest_limit(mats, dtype, bulk)
    announce(f"{name}: limit {limit}, preferred bulk {bulk}")
    w = run_case(Case(mats=mats, period=2, steps=3, param=dtype, state=dtype, ns=dtype, rank=16, seed=11,
                      device_memory_limit=limit)).worst()
    announce(f"worst errors {w}")
    unit, tile = BARS[dtype]
    assert w["u"] <= unit and w["u_unit"] <= unit and w["u_tile"] <= tile, w
    assert w["m_ulp"] <= 1.0 and w["x_ulp"] <= 1.0, w


def test_static_step_with_the_smaller_plan():
    """18 pairs of 512 x 512 and 512 x 640: the preferred plan's workspace alone is
    larger than the static array, the other plan's scratch is not."""
    import torch
    from oracle import muonbp_oracle as O
    from paper_2510_16981_amd import muonbp as mb
    from tests.gpu_harness import rel
    mats = [(512, 512, 1, 1), (512, 640, 1, 1)] * 18
    info = mb.describe_plan(mats, True)
    assert info.static_scratch_bytes <= mb.STATIC_SCRATCH_BYTES < info.workspace_bytes
    announce("static step, 18 x (512 x 512, 512 x 640)")
    gen = torch.Generator().manual_seed(3)
    g = [torch.randn(r, c, generator=gen).to(torch.bfloat16) for r, c, _, _ in mats]
    gd = [x.cuda() for x in g]
    ps = [torch.zeros_like(x) for x in gd]
    pc = [torch.zeros_like(x) for x in gd]
    mom = torch.zeros(sum(x.numel() for x in g), dtype=torch.bfloat16, device="cuda")
    mb.step_static(mats, ps, gd, mom, 0, 1, 0.02, 0.02, 0.95, 0.1)
    ctx = mb.MuonBP(mats, 1, 0.02, 0.02, 0.95, 0.1,
                    options=mb.options_default(device_memory_limit=info.device_bytes - 1))
    ctx.step(pc, gd, 0)
    torch.cuda.synchronize()
    for k, x in enumerate(ps):
        assert torch.equal(x, pc[k])
    for k in (0, 1, 34, 35):
        u = ctx.get_update(k).double().cpu().numpy()
        assert rel(u, O.orthogonalize_via_ns(g[k].double().numpy())) <= BARS["bf16"][0]
    ctx.close()

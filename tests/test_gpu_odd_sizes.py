"""GPU parity of bf16 units whose sides are not multiples of 8 on the DMA
kernels, which read the last 8-element chunk of a row whole, into zeros that
the pack and the epilogues write behind every row; and of the elementwise
kernels on windows of any alignment.

Every remainder of both sides by 8, transposed and untransposed, blocks that
start anywhere in their matrix, iterated as printed and on the Gram matrix,
each tile family the planner takes there, the NT apply and the K split; against
the oracle at the bf16 parity bar, and element by element for M and X.
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
    "one row, one column": dict(mats=[(1, 9, 1, 1), (11, 1, 1, 1), (3, 5, 1, 1)]),
    "remainders of both sides": dict(mats=[(120 + r, 209 - r, 1, 1) for r in range(1, 8)] +
                                     [(210 + r, 131 - r, 1, 1) for r in range(1, 8)], rank=64),
    "gram-space": dict(mats=[(129, 333, 1, 1), (271, 205, 1, 1), (397, 1003, 1, 1)], rank=64),
    "blocks at any offset": dict(mats=[(202, 381, 2, 3), (303, 130, 3, 2)], period=2, steps=4, rank=64),
    "beside aligned units": dict(mats=[(128, 512, 1, 1), (127, 513, 1, 1), (512, 128, 1, 1)], rank=64),
    "large tiles": dict(mats=[(1021, 1343, 1, 1)] * 6 + [(1343, 1021, 1, 1)] * 6, steps=1, rank=128),
    "NT apply": dict(mats=[(77, 203, 1, 1), (203, 77, 1, 1)], apply_mode=1, rank=64),
    "K split": dict(mats=[(301, 411, 1, 1), (411, 301, 1, 1)], k_split=3, rank=64),
    "the planner's K split": dict(mats=[(129, 6149, 1, 1), (6151, 70, 1, 1), (200, 8201, 1, 1)], rank=64, steps=1),
    "nesterov, fp32 weights": dict(mats=[(301, 411, 1, 1), (411, 301, 1, 1)], nesterov=1, param="f32", rank=64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_odd_sizes(name):
    from paper_2510_16981_amd import muonbp as mb
    case = Case(**{**dict(period=1, steps=2, rank=16, seed=7), **CASES[name]})
    opts = mb.options_default(apply_mode=case.apply_mode, k_split=case.k_split)
    info = mb.describe_plan(case.mats, case.period == 1, opts)
    announce(f"{name}: tiles {list(info.gemm_tile_rows)} x {list(info.gemm_tile_cols)}, split "
             f"{list(info.gemm_split)}, gram units {info.gram_units}: {case}")
    assert info.apply_nn == (0 if case.apply_mode else 1)  # only the DMA kernels read Z row-major
    if name == "large tiles":
        assert min(info.gemm_tile_rows) >= 128
    if name == "the planner's K split":
        assert info.gemm_split[0] == 3
    w = run_case(case).worst()
    announce(f"worst errors {w}")
    assert w["u"] <= TOL and w["u_unit"] <= TOL and w["u_tile"] <= TOL, w
    assert w["m"] <= TOL and w["x"] <= TOL, w
    assert w["m_ulp"] <= 1.0 and w["x_ulp"] <= 1.0, w


@pytest.mark.parametrize("mats", [[(77, 203, 1, 1), (205, 75, 1, 1)], [(1021, 1343, 1, 1)] * 6])
def test_padding_is_rewritten(mats):
    """A step on NaN leaves NaN behind the rows of some operands; a later step
    must not read it: after the momentum is reset, the context gives the bits
    of a new one."""
    import torch
    from paper_2510_16981_amd import muonbp as mb

    def grads(seed, bad):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        g = [torch.randn(r, c, generator=gen, device="cuda").bfloat16() for r, c, _, _ in mats]
        if bad:
            for x in g:
                x[0, 0] = float("nan")
        return g

    def make():
        return mb.MuonBP(mats, 1, 0.02, 0.02, 0.95), [torch.zeros(r, c, device="cuda").bfloat16() for r, c, _, _ in mats]

    used, p = make()
    used.step(p, grads(1, True), 0)
    for k, (r, c, _, _) in enumerate(mats):
        used.set_momentum(k, torch.zeros(r, c, device="cuda").bfloat16())
        p[k].zero_()
    fresh, q = make()
    used.step(p, grads(2, False), 1)
    fresh.step(q, grads(2, False), 1)
    for k in range(len(mats)):
        assert torch.isfinite(p[k]).all() and torch.equal(p[k], q[k])
        assert torch.equal(used.get_update(k), fresh.get_update(k))
    used.close()
    fresh.close()


def test_unaligned_tensors():
    """Weights and gradients that start at any element (views one to seven
    elements into a buffer) give the bits of aligned ones."""
    import torch
    from paper_2510_16981_amd import muonbp as mb
    mats = [(64, 72, 1, 1), (33, 47, 1, 1)]
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = [torch.randn(r, c, generator=gen, device="cuda").bfloat16() for r, c, _, _ in mats]
    x = [torch.randn(r, c, generator=gen, device="cuda").bfloat16() for r, c, _, _ in mats]

    def run(shift):
        opt = mb.MuonBP(mats, 1, 0.02, 0.02, 0.95, 0.1)
        ps, gs = [], []
        for k, (r, c, _, _) in enumerate(mats):
            for src, dst, s in ((x[k], ps, shift), (g[k], gs, (2 * shift) % 8)):
                buf = torch.full((r * c + 16,), 7.0, device="cuda").bfloat16()
                view = buf[s:s + r * c].view(r, c)
                view.copy_(src)
                dst.append((view, buf, s))
        for t in range(2):
            opt.step([p[0] for p in ps], [q[0] for q in gs], t)
        m = [opt.get_momentum(k) for k in range(len(mats))]
        opt.close()
        for view, buf, s in ps + gs:  # nothing written outside the views
            assert (buf[:s] == 7).all() and (buf[s + view.numel():] == 7).all()
        return [p[0].clone() for p in ps], m

    want = run(0)
    for shift in range(1, 8):
        got = run(shift)
        for a, b in zip(want[0] + want[1], got[0] + got[1]):
            assert torch.equal(a, b)

"""The zones' node transforms fused with the transfers around them, against the
same solve step by step (timed solves run every step as its own kernel): the
same sums in the same order, every multiply-add written out, so the potentials
and local values are equal bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,p,iso,precision", [
    (16, 2, 3, False, "fp64"),  # s = 4, no level between leaf and top
    (64, 2, 8, True, "fp64"),   # s = 16
    (32, 3, 4, True, "fp64"),   # s = 4
    (64, 3, 7, False, "fp64"),  # s = 8, odd
    (128, 3, 5, False, "fp64"),
    (16, 3, 6, False, "fp64"),  # s = 2: the mesh transfers stay alone
    (64, 4, 5, False, "fp32"),   # FP32 leaf level: the coarse levels fused
    (64, 4, 4, True, "fp32"),
])
def test_fused_levels_match_the_separate_steps(N, L, p, iso, precision):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    dt = torch.float64 if precision == "fp64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(901 + N + p)
    r = torch.randn((N, N, N), generator=g, device="cuda", dtype=dt)
    r -= r.mean()
    phi, ref = torch.empty_like(r), torch.empty_like(r)
    with Plan(N, L, p, "X" if iso else "S1", precision=precision, isolated=iso) as pl:
        pl.solve(r, phi)
        loc = [pl.locals(l).double().clone() for l in range(2, L + 1)]
        pl.set_profile("serial")
        pl.solve(r, ref)
        steps = [pl.locals(l).double().clone() for l in range(2, L + 1)]
        torch.cuda.synchronize()
    assert torch.equal(phi, ref)
    for a, b in zip(loc, steps):
        assert torch.equal(a, b)

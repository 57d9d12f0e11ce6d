"""The zones' node transforms fused with the transfers around them, against the
same solve step by step (timed solves run every step as its own kernel).  Both
are FP64 with the same sums in the same order; compilers may contract a product
and a sum differently, so some 10^2 roundings of 2^-53 per value, amplified by
the gridlets' alternating weights by up to 10^3 at p = 8: 1e-11 of the largest
potential.  With an FP32 leaf level the masses and local values are rounded to
FP32 and may then differ in their last bit: 2^-23 times the same 10^2 at most of
p = 5."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,p,iso,precision,tol", [
    (16, 2, 3, False, "fp64", 1e-11),  # s = 4, no level between leaf and top
    (64, 2, 8, True, "fp64", 1e-11),   # s = 16
    (32, 3, 4, True, "fp64", 1e-11),   # s = 4
    (64, 3, 7, False, "fp64", 1e-11),  # s = 8, odd
    (128, 3, 5, False, "fp64", 1e-11),
    (16, 3, 6, False, "fp64", 1e-11),  # s = 2: the mesh transfers stay alone
    (64, 4, 5, False, "fp32", 1e-5),   # FP32 leaf level: the coarse levels fused
    (64, 4, 4, True, "fp32", 1e-5),
])
def test_fused_levels_match_the_separate_steps(N, L, p, iso, precision, tol):
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
    e = float((phi - ref).abs().max() / ref.abs().max())
    print("fused zones", (N, L, p, iso, precision), "%.3e" % e)
    assert e < tol
    for a, b in zip(loc, steps):  # read back in FP32
        assert float((a - b).abs().max() / b.abs().max()) < max(tol, 2e-7)

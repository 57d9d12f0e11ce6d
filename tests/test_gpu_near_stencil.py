"""The FFT near zone's stencil at every way its launch cuts the box (blocks of 2 x
2 pencils in segments of 2 or more planes or whole, blocks of 2 x 4), periodic and
isolated, potential (even kernel) and accelerations (odd kernels), against the
FP64 near zone with the same tree.

What differs is the FP32 near zone: 2^-24 per pass of a transform of (2s)^3
values, log2 (2s)^3 = 15 of them forward and back at s = 16, 30 x 6e-8 = 1.8e-6
of the largest value if they all added up; a wrong wrap, edge or plane shows at
order one.  Repeated solves are equal bit for bit (every sum has one order)."""
import pytest

from gpu_util import rel_max

pytestmark = pytest.mark.gpu

TOL = 2e-6


@pytest.mark.parametrize("N,L,iso,accel", [
    (16, 2, False, True),    # 4 leaves per axis, segments of 2 planes
    (32, 3, True, True),     # 8, segments of 2
    (128, 3, False, True),   # 8, whole, s = 16
    (128, 3, True, False),
    (128, 5, False, False),  # 32, segments of 16, s = 4
    (128, 4, True, True),    # 16, whole, s = 8
    (64, 3, True, True),     # 8, segments of 2, s = 8
    (256, 5, False, False),  # 32, s = 8, whole
    (256, 4, True, False),   # 16, s = 16, blocks of 2 x 4
])
def test_stencil_matches_the_fp64_near_zone(N, L, iso, accel):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    g = torch.Generator(device="cuda").manual_seed(701 + N + L)
    r = torch.randn((N, N, N), generator=g, device="cuda")
    r -= r.mean()
    out = {}
    for near in ("fft", "direct"):
        phi = torch.empty_like(r)
        acc = torch.empty((3, N, N, N), device="cuda") if accel else None
        with Plan(N, L, 4, "X" if iso else "S1", near=near, m2l="spectral", isolated=iso,
                  accel="expansion" if accel else "fd4", fp64_levels=30) as pl:
            pl.solve(r, phi, acc)
            if near == "fft":
                first = phi.clone(), None if acc is None else acc.clone()
                for _ in range(3):
                    pl.solve(r, phi, acc)
                assert torch.equal(first[0], phi) and (acc is None or torch.equal(first[1], acc))
            torch.cuda.synchronize()
        out[near] = [phi] + ([acc] if accel else [])
    for a, b in zip(out["fft"], out["direct"]):
        e = rel_max(a.double().cpu().numpy(), b.double().cpu().numpy())
        print("near stencil", (N, L, iso), "%.3e" % e)
        assert e < TOL

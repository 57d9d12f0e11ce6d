"""The default interaction zones by per-node FP64 transforms: gridlets that the
spectral option does not serve, periodic and isolated, on the 4^3, 8^3 and 16^3
levels, against the reference FMM; and the fallback of the levels whose spectra
are too large.

With every level in FP64 what is left is the FP32 result: the near part rounded
once on its way to the mesh and once more when the far field is added, with the
FP64 far field rounded in between: 3 x 2^-24 < 2.5e-7 of max |phi|."""
import numpy as np
import pytest

from oracle import fmm as ofmm
from paper_2011_07099_amd import fields

from gpu_util import f32, rel_max

pytestmark = pytest.mark.gpu

TOL = 2.5e-7


@pytest.mark.parametrize("N,L,p,iso", [
    (16, 2, 10, False),
    (16, 2, 7, True),
    (32, 3, 9, False),
    (32, 3, 5, True),
    (32, 3, 2, False),   # the largest gridlet that keeps the block-Toeplitz products
    (64, 4, 3, False),   # the smallest that does not
    (64, 4, 3, True),
])
def test_default_zones_match_the_reference(N, L, p, iso):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    green = "X" if iso else "S1"
    rho = f32(fields.lognormal(N, 1.5, 1.0, seed=601 + N + p))
    r = torch.from_numpy(rho.astype(np.float32)).cuda()
    phi = torch.empty_like(r)
    with Plan(N, L, p, green, isolated=iso, fp64_levels=30) as pl:
        pl.solve(r, phi)
        torch.cuda.synchronize()
    e = rel_max(phi.cpu().numpy().astype(np.float64), ofmm.fmm(rho, L, p, green, periodic=not iso))
    print("default zones", (N, L, p, iso), "%.3e" % e)
    assert e < TOL


def test_levels_over_the_memory_bound_fall_back():
    """64^3 nodes at p = 6 need 8.5 GB of spectra: that level by block-Toeplitz
    products in FP32 (each offset's 216 terms: at most 216 x 2^-24 = 1.3e-5 of
    their absolute sum, about 3 times the potential with one-cell leaves), the
    coarser ones by transforms; the spectral option takes all of it."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N, L, p = 64, 6, 6
    r = torch.from_numpy(f32(fields.lognormal(N, 1.5, 1.0, seed=613)).astype(np.float32)).cuda()
    out = []
    with Plan(N, L, p, "S1") as pl:
        for m2l in ("gemm", "spectral", "gemm"):
            pl.set_m2l(m2l)
            phi = torch.empty_like(r)
            pl.solve(r, phi)
            out.append(phi)
        torch.cuda.synchronize()
    scale = out[1].abs().max()
    assert (out[0] - out[1]).abs().max() < 4e-5 * scale
    assert torch.equal(out[0], out[2])

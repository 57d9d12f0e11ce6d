"""The spectral zone stencil on the levels it cuts into tiles with a halo (32^3
nodes, and isolated levels from 8^3 on), against the block-Toeplitz sums with
every level in FP64.  Both are FP64, so their FP32 read-backs differ by at most
one FP32 rounding of the largest value (2^-23 = 1.2e-7); a wrong halo, wrap or
tile origin would show at order one."""
import numpy as np
import pytest

from paper_2011_07099_amd import fields

from gpu_util import f32, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,p,iso", [
    (64, 5, 4, False),   # 32^3 leaf level: 4 x 4 x 2 tiles, wrapped halo
    (64, 5, 4, True),    # the same with empty nodes outside the box
    (64, 4, 4, True),    # isolated 16^3 level: 2 x 2 x 1 tiles
    (32, 3, 6, True),    # isolated 8^3 level: one tile with its halo
])
def test_tiled_zone_levels_match_the_fp64_gemm(N, L, p, iso):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    rho = torch.from_numpy(f32(fields.lognormal(N, 2.0, 1.0, seed=401 + N + p)).astype(np.float32)).cuda()
    phi = torch.empty_like(rho)
    loc = {}
    for m2l in ("spectral", "gemm"):
        with Plan(N, L, p, "X" if iso else "S1", fp64_levels=30, isolated=iso, m2l=m2l) as pl:
            pl.solve(rho, phi)
            loc[m2l] = [pl.locals(l).cpu().numpy().astype(np.float64) for l in range(2, L + 1)]
            torch.cuda.synchronize()
    for l, (a, b) in enumerate(zip(loc["spectral"], loc["gemm"]), start=2):
        e = rel_max(a, b)
        print("tiled zones", (N, L, p, iso), "level", l, "%.3e" % e)
        assert e < 2e-7

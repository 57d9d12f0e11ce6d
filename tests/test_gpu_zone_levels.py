"""The zone sums of every kind of level (4^3; 8^3 in one tile, wrapped or with a
halo; 16^3 whole or tiled; 32^3 tiled) against the oracle's locals, by the default
zones and by the spectral option, with every level and array in FP64.

Locals are read back in FP32: one rounding, 2^-24 of the largest, and the
oracle's own far below it; 2e-7 allowed.  The FP64 potential keeps what the FP32
read-back hides: the sums of a zone cancel up to 10^3 fold and L2P extrapolates up to
some 10 fold, so roundings of 2^-53 in the 30 passes of a solve come to 30 x 10^4 x
1.1e-16 = 3e-11 of the largest value at most."""
import numpy as np
import pytest

from oracle import fmm as ofmm
from paper_2011_07099_amd import fields

from gpu_util import rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,p,iso", [
    (32, 3, 4, False),
    (32, 3, 8, True),
    (32, 3, 6, True),
    (64, 3, 6, False),
    (64, 4, 4, True),    # isolated 16^3 level: 2 x 2 x 1 tiles
    (64, 4, 8, False),   # periodic 16^3 level, whole
    (64, 5, 4, False),   # 32^3 level: 4 x 4 x 2 tiles, wrapped halo
    (64, 5, 4, True),    # the same with empty nodes outside the box
    (64, 5, 3, False),   # a gridlet that the option does not serve
])
def test_zone_levels_match_the_oracle(N, L, p, iso):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    green = "X" if iso else "S1"
    rho = fields.lognormal(N, 2.0, 1.0, seed=961 + N + p)
    ref, st = ofmm.fmm(rho, L, p, green, stages=True, periodic=not iso)
    r = torch.from_numpy(rho).cuda()
    for m2l in ("gemm",) + (("spectral",) if p in (4, 6, 8) else ()):
        phi = torch.empty_like(r)
        with Plan(N, L, p, green, precision="fp64", isolated=iso, m2l=m2l) as pl:
            pl.solve(r, phi)
            loc = [pl.locals(l).cpu().numpy().astype(np.float64) for l in range(2, L + 1)]
            torch.cuda.synchronize()
        e = [rel_max(a, st["Phi"][l].ravel()) for l, a in enumerate(loc, start=2)]
        ep = rel_max(phi.cpu().numpy(), ref)
        print("zone levels", (N, L, p, iso, m2l), " ".join("%.3e" % x for x in e), "potential %.3e" % ep)
        assert max(e) < 2e-7 and ep < 3e-11

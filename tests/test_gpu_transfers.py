"""P2M, M2M, L2L and L2P by columns (leaves of 8 and 16 cells, every p), and the
differenced accelerations by vectors.

With every level in FP64 what is left against the reference FMM is the FP32
result: three FP32 roundings of values up to the largest |phi|, 3 x 2^-24 <
2.5e-7.  With FP32 gridlets of p <= 3 a value also passes some 20 rounded sums
whose weights add up to (5/4)^3 at most: 1e-5."""
import numpy as np
import pytest

from oracle import fmm as ofmm
from paper_2011_07099_amd import fields

from gpu_util import f32, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,p,levels,tol", [
    (32, 2, 10, 30, 2.5e-7),  # s = 8, columns over more than one wave's lanes
    (64, 2, 9, 30, 2.5e-7),   # s = 16, the columns of a pass over three waves
    (64, 3, 7, 30, 2.5e-7),   # s = 8, odd
    (128, 3, 3, 30, 2.5e-7),  # s = 16, eight tasks to a wave idle
    (32, 2, 1, 30, 2.5e-7),
    (64, 3, 3, 1, 1e-5),      # FP32 leaf gridlets, FP64 parents
    (128, 3, 2, 1, 1e-5),
])
def test_transfers_match_the_reference(N, L, p, levels, tol):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    rho = f32(fields.lognormal(N, 1.5, 1.0, seed=801 + N + p))
    r = torch.from_numpy(rho.astype(np.float32)).cuda()
    phi = torch.empty_like(r)
    acc = torch.empty((3, N, N, N), dtype=torch.float32, device="cuda")
    with Plan(N, L, p, "S1", fp64_levels=levels) as pl:
        pl.solve(r, phi, acc)
        # the same through buffers that are only 4-byte aligned
        odd = [torch.empty(n * N ** 3 + 1, dtype=torch.float32, device="cuda")[1:] for n in (1, 1, 3)]
        odd[0].copy_(r.flatten())
        pl.solve(*odd)
        torch.cuda.synchronize()
    assert torch.equal(odd[1], phi.flatten()) and torch.equal(odd[2], acc.flatten())
    got = phi.cpu().numpy().astype(np.float64)
    e = rel_max(got, ofmm.fmm(rho, L, p, "S1"))
    print("transfers", (N, L, p, levels), "%.3e" % e)
    assert e < tol
    # differences of the potential just read back: four FP32 products and sums of
    # values up to 8 |phi| on the way to N / 12 times them, 8 roundings of 2^-24
    g = np.stack([sum(w * np.roll(got, -k, ax) for k, w in ((-2, 1.0), (-1, -8.0), (1, 8.0), (2, -1.0)))
                  for ax in range(3)]) * (-N / 12)
    d = np.abs(acc.cpu().numpy() - g).max()
    assert d < 8 * 2.0 ** -24 * 18 * np.abs(got).max() * N / 12

"""The near zone of FP32 plans by FP64 transforms (leaf edges 4, 8, 16), with
every tree level in FP64, against the reference FMM.

The near sums are FP64, so what is left is the FP32 result: the near part is
rounded once on its way to the mesh and once more when the far field is added,
two roundings of 2^-24 of values up to about the largest |phi|, with the FP64
far field rounded in between: 3 x 6e-8 < 2.5e-7 of max |phi|.  Accelerations
(expansion) carry the same two roundings per component."""
import numpy as np
import pytest

from oracle import fmm as ofmm
from paper_2011_07099_amd import fields

from gpu_util import f32, rel_max

pytestmark = pytest.mark.gpu

TOL = 2.5e-7


@pytest.mark.parametrize("N,L,p,iso", [
    (16, 2, 3, False),   # s = 4, four leaves per axis: every neighbour wraps
    (32, 3, 4, True),    # s = 4 isolated, z segments of two planes
    (64, 3, 5, False),   # s = 8, an odd gridlet
    (32, 2, 4, True),    # s = 8 isolated
    (64, 2, 6, False),   # s = 16
])
def test_near_zone_in_fp64_matches_the_reference(N, L, p, iso):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    green = "X" if iso else "S1"
    rho = f32(fields.lognormal(N, 1.5, 1.0, seed=501 + N + p))
    r = torch.from_numpy(rho.astype(np.float32)).cuda()
    phi, acc = torch.empty_like(r), torch.empty((3, N, N, N), dtype=torch.float32, device="cuda")
    with Plan(N, L, p, green, isolated=iso, accel="expansion", fp64_levels=30) as pl:
        pl.solve(r, phi, acc)
        # the same through buffers that are only 4-byte aligned
        big = [torch.empty(n * N ** 3 + 1, dtype=torch.float32, device="cuda") for n in (1, 1, 3)]
        odd = [b[1:] for b in big]
        odd[0].copy_(r.flatten())
        pl.solve(*odd)
        torch.cuda.synchronize()
    assert torch.equal(odd[1], phi.flatten()) and torch.equal(odd[2], acc.flatten())
    ref, ref_phi = ofmm.fmm_accel(rho, L, p, green, periodic=not iso)
    e = rel_max(phi.cpu().numpy().astype(np.float64), ref_phi)
    ea = rel_max(acc.cpu().numpy().astype(np.float64), ref)
    print("FP64 near zone", (N, L, p, iso), "potential %.3e accelerations %.3e" % (e, ea))
    assert e < TOL and ea < TOL


def test_options_switch_the_near_zone_back_and_forth():
    """Direct, transforms in FP32, split and back: the last solve is the first's, bit for bit."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N = 32
    r = torch.from_numpy(f32(fields.lognormal(N, 1.5, 1.0, seed=511)).astype(np.float32)).cuda()
    outs = []
    with Plan(N, 2, 4, "S1") as pl:
        for near, prec in (("direct", "fp32"), ("fft", "fp32"), ("fft", "fp64"), ("direct", "bf16x3"),
                           ("direct", "fp32")):
            pl.set_near(near)
            pl.set_precision(prec)
            phi = torch.empty_like(r)
            pl.solve(r, phi)
            outs.append(phi)
        torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[-1])
    scale = outs[0].abs().max()
    for o, tol in zip(outs[1:4], (2e-6, 1e-6, 1e-4)):
        assert (o - outs[0]).abs().max() < tol * scale

"""The exact periodic convolution (pfmm_plan_direct) by FP64 transforms against
the oracle's FFT convolution with the same G, for even and odd powers of two
(both orders of the two-stage passes), one and many lines a workgroup.  Sums are
FP64, so the error is the one rounding to FP32: 2^-24 = 6e-8 of the largest
value, 1e-7 allowed."""
import numpy as np
import pytest

from oracle import conv
from paper_2011_07099_amd import fields

from gpu_util import f32, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,green", [(8, 2, "S1"), (16, 2, "K"), (32, 3, "X"), (64, 3, "S1"),
                                       (128, 3, "K"), (256, 4, "S1")])
def test_direct_matches_the_oracle(N, L, green):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    rho = f32(fields.lognormal(N, 1.5, 1.0, seed=601 + N))
    r = torch.from_numpy(rho.astype(np.float32)).cuda()
    phi = torch.empty_like(r)
    big = torch.empty(2 * N ** 3 + 2, dtype=torch.float32, device="cuda")
    odd_r, odd_phi = big[1:N ** 3 + 1], big[N ** 3 + 2:]
    odd_r.copy_(r.flatten())
    with Plan(N, L, 2, green) as pl:
        pl.direct(r, phi)
        pl.direct(odd_r, odd_phi)   # 4-byte aligned
        torch.cuda.synchronize()
    assert torch.equal(odd_phi, phi.flatten())
    e = rel_max(phi.cpu().numpy().astype(np.float64), conv.pm(rho, green))
    print("direct periodic convolution N=%d G_%s: %.3e" % (N, green, e))
    assert e < 1e-7


def test_direct_on_two_streams_and_after_a_new_g():
    """Calls on alternating streams share the plan's spectrum and wait for each
    other; a change of a1 changes the convolution."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N = 64
    rhos = [torch.from_numpy(fields.lognormal(N, 1.5, 1.0, seed=611 + i).astype(np.float32)).cuda()
            for i in range(6)]
    ref = [torch.empty_like(r) for r in rhos]
    out = [torch.full_like(r, float("nan")) for r in rhos]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    with Plan(N, 3, 2, "S", a1=-0.125) as pl:
        for r, o in zip(rhos, ref):
            pl.direct(r, o)
            torch.cuda.synchronize()
        for i, (r, o) in enumerate(zip(rhos, out)):
            pl.set_stream(streams[i % 2])
            pl.direct(r, o)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ref, out))
        pl.set_a1(-0.2)
        pl.direct(rhos[0], out[0])
        torch.cuda.synchronize()
    rho = rhos[0].cpu().numpy().astype(np.float64)
    assert rel_max(out[0].cpu().numpy().astype(np.float64), conv.pm(rho, "S", a=(-0.2, 0.0))) < 1e-7

"""Options leave solves that are still running alone: precision and near-zone
route are the host's choice for the next solve (nothing runs, nothing waits),
and the acceleration kernels are made without touching what a solve reads."""
import numpy as np
import pytest

from paper_2011_07099_amd import fields

pytestmark = pytest.mark.gpu


def density(N, seed):
    import torch
    return torch.from_numpy(fields.lognormal(N, 1.5, 1.0, seed=seed).astype(np.float32)).cuda()


def busy(plan, rho, out, stream, n=200):
    """Some 100 ms of work on the stream: n solves with expansion accelerations."""
    import torch
    with torch.cuda.stream(stream):
        for _ in range(n):
            plan.solve(rho, *out)


def test_precision_and_near_zone_options_wait_for_nothing():
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    s = torch.cuda.Stream()
    N = 128
    rho = density(N, 921)
    out = torch.empty_like(rho), torch.empty((3, N, N, N), device="cuda")
    with Plan(N, 3, 8, "S1", stream=s, accel="expansion") as work, Plan(64, 3, 8, "S1", stream=s) as pl:
        pl.set_near("fft")                 # its buffers, on first use
        pl.set_near("direct")
        busy(work, rho, out, s)
        assert not s.query()               # the stream is busy
        for name, value in (("set_precision", "bf16x3"), ("set_near", "fft"), ("set_precision", "fp64"),
                            ("set_precision", "fp32"), ("set_near", "direct")):
            getattr(pl, name)(value)
            assert not s.query(), (name, value)
        torch.cuda.synchronize()


@pytest.mark.parametrize("then", [("set_precision", "bf16x3"), ("set_near", "fft"), ("set_accel", "expansion")])
def test_options_do_not_disturb_a_running_solve(then):
    """Solves queued on one stream, the plan moved to another and the option set
    there: every queued solve gives what it gives alone, bit for bit."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    s, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    N, n = 128, 40
    rho = density(N, 922)
    ref = torch.empty_like(rho)
    outs = [torch.full_like(rho, float("nan")) for _ in range(n)]
    with Plan(N, 4, 4, "S1", stream=s) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, ref)
            torch.cuda.synchronize()
            for o in outs:
                pl.solve(rho, o)
        pl.set_stream(s2)
        getattr(pl, then[0])(then[1])
        torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for o in outs)

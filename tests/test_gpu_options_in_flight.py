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
        small = density(64, 925)
        pl.solve(small, torch.empty_like(small))
        pl.set_near("fft")                 # its buffers, on first use
        pl.set_near("direct")
        torch.cuda.synchronize()
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


@pytest.mark.parametrize("change", ["a1", "gstar"])
def test_a_new_g_waits_for_a_running_convolution(change):
    """direct() queued behind other work on one stream, then a new G set on
    another: the queued convolution has the old G, the next one the new."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    s, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    N = 64
    rho, big = density(N, 923), density(128, 924)
    acc = torch.empty_like(big), torch.empty((3, 128, 128, 128), device="cuda")
    ref, new, out, after = (torch.empty_like(rho) for _ in range(4))

    def set_g(pl):
        if change == "a1":
            pl.set_a1(-0.2)
        else:
            n = pl.gstar_params()
            pl.set_gstar(1e-2 * np.random.default_rng(5).standard_normal(n).astype(np.float32))
    with Plan(N, 4, 2, "S", a1=-0.125) as pl:
        pl.direct(rho, ref)
        set_g(pl)
        pl.direct(rho, new)
        torch.cuda.synchronize()
    assert not torch.equal(ref, new)
    with Plan(128, 3, 8, "S1", stream=s, accel="expansion") as work, \
            Plan(N, 4, 2, "S", a1=-0.125, stream=s2) as pl:
        pl.direct(rho, out)                # its tables
        if change == "gstar":
            pl.set_gstar(None)             # its buffers
        torch.cuda.synchronize()
        busy(work, big, acc, s)
        pl.set_stream(s)
        pl.direct(rho, out)
        assert not s.query()
        pl.set_stream(s2)
        set_g(pl)
        pl.direct(rho, after)
        torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(after, new)

"""Solves captured into a HIP graph stay replayable when the plan's options then
select other routes: the buffers that a captured solve uses live as long as the
plan, and its kernels follow a change of G like every other table.

Replays are compared with the eager solve of the same options, bit for bit (same
kernels, same operands).  Between the option and the replay the test allocates
and fills what the plan would have given back, so that a freed buffer would not
hold its old values."""
import numpy as np
import pytest

from paper_2011_07099_amd import fields

pytestmark = pytest.mark.gpu


def density(N, seed):
    import torch
    return torch.from_numpy(fields.lognormal(N, 1.5, 1.0, seed=seed).astype(np.float32)).cuda()


def captured(pl, rho, phi, acc, stream):
    """A graph of one solve on the plan's stream."""
    import torch
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        pl.solve(rho, phi, acc)
    torch.cuda.synchronize()
    return g


def replays(g, out, ref, nbytes):
    """Replay with eager work between; every replay equals `ref` bit for bit."""
    import torch
    for _ in range(3):
        junk = torch.full((nbytes // 4,), float("nan"), device="cuda")
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref))
        del junk
        torch.cuda.empty_cache()


@pytest.mark.parametrize("N,L,p,accel,first,then", [
    (64, 3, 4, False, {}, [("set_near", "fft")]),
    (64, 2, 4, True, {}, [("set_near", "fft")]),
    (64, 3, 8, False, {}, [("set_precision", "bf16x3"), ("set_near", "fft"), ("set_precision", "fp32")]),
    (32, 3, 4, False, {"near": "fft", "precision": "fp64"}, [("set_precision", "fp32")]),
    (64, 3, 4, False, {"near": "fft"}, [("set_near", "direct"), ("set_precision", "fp64")]),
])
def test_a_captured_solve_outlives_the_near_zone_options(N, L, p, accel, first, then):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    s = torch.cuda.Stream()
    rho, rho2 = density(N, 901), density(N, 902)
    phi, ref = torch.empty_like(rho), torch.empty_like(rho)
    acc = torch.empty((3, N, N, N), device="cuda") if accel else None
    racc = torch.empty_like(acc) if accel else None
    other = torch.empty_like(rho)
    kw = dict(first, accel="expansion") if accel else first
    with Plan(N, L, p, "S1", stream=s, **kw) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, ref, racc)
        g = captured(pl, rho, phi, acc, s)
        for name, value in then:
            getattr(pl, name)(value)
        with torch.cuda.stream(s):
            pl.solve(rho2, other)          # the new route, eager
        torch.cuda.synchronize()
        replays(g, [phi] + ([acc] if accel else []), [ref] + ([racc] if accel else []), 160 * N ** 3)


def test_a_captured_solve_outlives_the_spectral_option():
    """One-cell leaves at 64^3, p = 6: the default zones have spectra up to 32^3
    nodes, the spectral option makes its own for all levels (8.5 GB)."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N, L, p = 64, 6, 6
    s = torch.cuda.Stream()
    rho = density(N, 903)
    phi, ref, other = (torch.empty_like(rho) for _ in range(3))
    with Plan(N, L, p, "S1", stream=s) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, ref)
        g = captured(pl, rho, phi, None, s)
        pl.set_m2l("spectral")
        with torch.cuda.stream(s):
            pl.solve(rho, other)
        torch.cuda.synchronize()
        replays(g, [phi], [ref], 3 << 29)


@pytest.mark.parametrize("then", [("set_near", "fft"), ("set_m2l", "spectral")])
def test_a_captured_solve_follows_g_after_the_options(then):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N, L, p = 32, 3, 4
    s = torch.cuda.Stream()
    rho = density(N, 904)
    phi, ref = torch.empty_like(rho), torch.empty_like(rho)
    with Plan(N, L, p, "S", stream=s, a1=-0.2) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, ref)
        torch.cuda.synchronize()
    with Plan(N, L, p, "S", stream=s, a1=-0.1) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, phi)
        g = captured(pl, rho, phi, None, s)
        getattr(pl, then[0])(then[1])
        pl.set_a1(-0.2)
        replays(g, [phi], [ref], 1 << 24)


def test_a_captured_solve_in_fp32_columns_follows_g_after_the_option():
    """FP32 columns of the 16^3 leaf level: captured with the option on, then the
    option off and a new G; the replay has every kernel of the new G."""
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    N, L, p = 64, 4, 4
    s = torch.cuda.Stream()
    rho = density(N, 905)
    phi, ref = torch.empty_like(rho), torch.empty_like(rho)
    kw = dict(m2l="spectral", zones_fp32=True, stream=s)
    with Plan(N, L, p, "S", a1=-0.2, **kw) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, ref)
        torch.cuda.synchronize()
    with Plan(N, L, p, "S", a1=-0.1, **kw) as pl:
        with torch.cuda.stream(s):
            pl.solve(rho, phi)
        g = captured(pl, rho, phi, None, s)
        pl.set_zones_fp32(False)
        pl.set_a1(-0.2)
        replays(g, [phi], [ref], 1 << 24)

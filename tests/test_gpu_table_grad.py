"""Table gradients at every block edge the kernels are compiled for, by
directional differences of the device loss.

The loss is exactly quadratic in the tables' relative corrections, so the
central difference along any direction equals gradient . direction up to the
rounding of two losses: each sums FP32 potentials (2^-24 relative) that a
correction of 3 % leaves far from the target, so 1e-4 relative is allowed.
With G_* the target moves too and the loss is a ratio of quadratics: a step of
1e-3 leaves a relative error of its square times the curvature, 1e-3 allowed."""
import numpy as np
import pytest

from paper_2011_07099_amd import fields

pytestmark = pytest.mark.gpu


def _density(N, seed):
    import torch
    return torch.from_numpy(fields.lognormal(N, 1.5, 1.0, seed=seed).astype(np.float32)).cuda()


@pytest.mark.parametrize("N,L,p", [(16, 3, 1), (16, 3, 2), (32, 3, 3), (32, 3, 5), (32, 2, 6), (32, 3, 7),
                                   (32, 3, 8), (16, 2, 9), (32, 3, 10)])
def test_zone_table_gradient(N, L, p):
    import torch
    from paper_2011_07099_amd.pfmm import Plan
    rho = _density(N, 701 + p)
    target = torch.empty_like(rho)
    rng = np.random.default_rng(702 + p)
    with Plan(N, L, p, "S1") as pl:
        pl.direct(rho, target)
        pl.table_train_begin(1e-6)
        n = pl.table_params()
        base, step = (0.03 * rng.standard_normal((2, n))).astype(np.float32)
        loss = []
        for sign in (1.0, -1.0):
            pl.set_table(base + np.float32(sign) * step)
            loss.append(pl.loss(rho, target))
        pl.set_table(base)
        pl.train_accumulate(rho, target)
        g = pl.table_grad().astype(np.float64)
    fd, got = 0.5 * (loss[0] - loss[1]), float(g @ step.astype(np.float64))
    print("zone table gradient", (N, L, p), "difference %.6e gradient %.6e" % (fd, got))
    assert abs(got - fd) < 1e-4 * max(abs(fd), 0.1 * loss[0])


@pytest.mark.parametrize("N,L,p", [(8, 3, 1), (16, 3, 2), (32, 3, 4), (32, 2, 4), (64, 2, 8)])
def test_near_table_gradient_in_gstar(N, L, p):
    """Leaf edges 1, 2, 4, 8 and 16 (the last as 8^3 sub-blocks)."""
    from paper_2011_07099_amd.pfmm import Plan
    rho = _density(N, 711 + N + L)
    rng = np.random.default_rng(712 + N + L)
    with Plan(N, L, p, "S1") as pl:
        n = pl.gstar_params()
        base, step = 0.02 * rng.standard_normal(n), 1e-3 * rng.standard_normal(n)
        loss = []
        for sign in (1.0, -1.0):
            pl.set_gstar(base + sign * step)
            loss.append(pl.gstar_loss(rho))
        pl.set_gstar(base)
        pl.gstar_accumulate(rho)
        g = pl.gstar_grad().astype(np.float64)
    fd, got = 0.5 * (loss[0] - loss[1]), float(g @ step)
    print("G_* gradient", (N, L, p), "loss %.3e difference %.6e gradient %.6e" % (loss[0], fd, got))
    assert abs(got - fd) < 1e-3 * max(abs(fd), 0.05 * loss[0])

"""The rest-state-with-velocity map's vector-Jacobian product against a central
difference of the map, within what rounding and truncation can move the difference
by (the sum that the products form may cancel, so it is no measure of either)."""
import numpy as np
import pytest

from paper_2009_14555_amd import problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", range(8))
def test_vjp_against_central_difference(seed):
    import torch

    from paper_2009_14555_amd import adjoint as A
    from paper_2009_14555_amd import solver as S

    n = 24
    pb, W = P.plate_impact(n, noise=1e-3, seed=2)
    L = P.layout(pb)
    W[L.u(0)] = 0.0
    g = S.Grid(pb)
    g.set_primitive(W)
    rest = g.state.clone()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rand = lambda shape: torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda")  # noqa: E731
    vel = [(400.0 * rand((n, n))).requires_grad_(True) for _ in range(2)]
    Ur = rest.clone().requires_grad_(True)
    out = A.with_velocity(g, Ur, *vel)
    w = rand(out.shape)
    (out * w).sum().backward()
    dU = rand(rest.shape) * rest.abs().amax(dim=(1, 2), keepdim=True) * 1e-3
    dv = [rand((n, n)) for _ in range(2)]
    h = 1e-4
    with torch.no_grad():
        fp, fm = (A.with_velocity(g, rest + s * dU, *[v + s * d for v, d in zip(vel, dv)]) for s in (h, -h))
        lhs = ((fp - fm) / (2 * h) * w).sum()
        rhs = (Ur.grad * dU).sum() + sum((v.grad * d).sum() for v, d in zip(vel, dv))
        # each value carries up to five roundings of its own magnitude (its inputs'
        # displacement, the density, the product or square, the sum) on either side
        mag = torch.maximum(fp.abs(), fm.abs())
        mag[L.E] = mag[L.E] + 0.5 * (rest[L.m(0)] + rest[L.m(1)]) * sum(v * v for v in vel) + rest[L.E].abs()
        rounding = 5 * 2.0**-53 * (w.abs() * mag).sum() / h
        # the map is a cubic of its inputs: the difference's third-order term
        dr = (dU[L.m(0)] + dU[L.m(1)]).abs()
        truncation = h**2 * (w[L.E].abs() * 0.5 * dr * sum(d * d for d in dv)).sum()
    assert abs(float(lhs - rhs)) <= float(rounding + truncation)
    assert float(rounding + truncation) <= 1e-6 * float((Ur.grad * dU).abs().sum())

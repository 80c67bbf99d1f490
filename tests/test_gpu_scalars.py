"""The stages' reciprocal, quotient, root and exponential against extended
precision: rounded as the IEEE operations (and no further off than the library's
exponential) that they stand in place of; and the pressure of unreacted explosive at
rest, which the two-gas split has to find between two nearly equal roots."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2009_14555_amd import problems as P
from tests.parity_util import to_np

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
FN = {"frcp": 0, "quot": 1, "fsqrt": 2, "times_inverse": 3, "exp_curve": 4, "lib_exp": 5}
LD = np.longdouble


@pytest.fixture(scope="module")
def gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = C.CDLL(os.path.join(HERE, "libdimp_scalars.so"))

    def run(fn, a, b):
        a, b = (torch.tensor(np.ascontiguousarray(v, dtype=np.float64), device="cuda") for v in (a, b))
        out = torch.empty_like(a)
        torch.cuda.synchronize()
        assert lib.scalar_run(FN[fn], a.numel(), *(C.c_void_p(t.data_ptr()) for t in (a, b, out))) == 0
        return out.cpu().numpy()

    return run


def ulps(got, want):
    """errors in units of the last place of want (extended precision)"""
    return np.abs(got.astype(LD) - want) / np.exp2(np.floor(np.log2(np.abs(want))) - 52)


def points(n, seed):
    rng = np.random.default_rng(seed)
    return rng.uniform(-60.0, 0.0, n), np.exp2(rng.uniform(-40, 40, n))


@pytest.mark.parametrize("fn", ["frcp", "quot", "fsqrt", "times_inverse"])
def test_rounded_as_the_ieee_operation(gpu, fn):
    """half an ulp, and what a correction of relative size 2^-50 or less can add"""
    a, b = points(1 << 20, 1)
    want = {"frcp": 1 / b.astype(LD), "quot": a.astype(LD) / b.astype(LD), "fsqrt": np.sqrt(b.astype(LD)),
            "times_inverse": a.astype(LD) / b.astype(LD)}[fn]
    assert ulps(gpu(fn, a, b), want).max() <= 0.5 + 2.0**-7


def test_exponential_no_further_off_than_the_librarys(gpu):
    a, b = points(1 << 22, 2)
    want = np.exp(a.astype(LD))
    mine, lib = ulps(gpu("exp_curve", a, b), want), ulps(gpu("lib_exp", a, b), want)
    print("max %.4f %.4f rms %.4f %.4f" % (mine.max(), lib.max(), np.sqrt((mine**2).mean()), np.sqrt((lib**2).mean())))
    # the maxima of a sample scatter by some 0.01 ulp
    assert mine.max() <= lib.max() + 0.02 and (mine**2).mean() <= 1.01 * (lib**2).mean()


def test_special_values(gpu):
    x = np.array([0.0, -0.0, np.inf, np.nan, -1.0, 1e-290, 1e300, 4.0])
    r = gpu("fsqrt", x, x)
    with np.errstate(invalid="ignore"):
        np.testing.assert_array_equal(r, np.sqrt(x))
    assert np.array_equal(gpu("exp_curve", np.array([0.0, -800.0, np.nan, 800.0]), np.ones(4)),
                          np.array([1.0, 0.0, np.nan, np.inf]), equal_nan=True)


def pressure_of(E, py, rho, lam, solid, r, p0):
    """p of the mixture cell from rho e in extended precision: the split at a
    trial p is explicit (equal temperatures), rho e(p) is monotone"""
    a, b = r.reactant, r.product
    ga, gb = LD(a.gamma) - 1, LD(b.gamma) - 1
    pa, pb = (-LD(m.gamma) * LD(m.pinf) for m in (a, b))
    ps, x = 1 - py, rho[1] / LD(solid.rho0)
    gs, pref = LD(solid.Gamma0), LD(solid.K0) * x * x * (x - 1)
    es = rho[1] * LD(solid.K0) / (2 * LD(solid.rho0)) * (x - 1) ** 2

    def f(p):
        al, be = (p - pa) / (ga * LD(a.cv)), (p - pb) / (gb * LD(b.cv))
        s = lam * be / (lam * be + (1 - lam) * al)
        mix = s * (p - pa) / ga + (1 - s) * (p - pb) / gb - rho[0] * (1 - lam) * LD(r.Q)
        return py * mix + ps * ((p - pref) / gs + es) - E

    p = p0
    for _ in range(60):
        h = p * LD(1e-7)
        p = p - f(p) * (2 * h) / (f(p + h) - f(p - h))
    return p


def test_pressure_between_two_nearly_equal_roots(gpu):
    """progress 1 - 1e-11 at 1e5 Pa: the error allowed is twice what one rounding
    of the progress and one of the energy move the pressure by"""
    from paper_2009_14555_amd import solver as S

    n = 4096
    solid = P.solid_c2()
    pb = P.Problem(ndim=1, n=(n, 1, 1), dx=(1.0 / n, 1, 1), materials=[P.placeholder_for_reactive(), solid],
                   reactive=P.generic_explosive(0))
    L = P.layout(pb)
    rng = np.random.default_rng(4)
    W = P.blank_prim(pb)
    W[L.phi(0)] = 1.0 - P.PHI_PURE
    W[L.rho(0)] = 1600.0 * (1 + 0.01 * rng.uniform(-1, 1, n))
    W[L.rho(1)] = solid.rho0
    W[L.lam] = 1.0 - 1e-11 * rng.uniform(1.0, 2.0, n)
    W[L.p] = 1e5 * (1 + 0.1 * rng.uniform(-1, 1, n))
    g = S.Grid(pb)
    g.set_primitive(W)
    U = to_np(g.state).astype(LD)
    p = to_np(g.primitive())[L.p].astype(LD)
    py, E = U[0], U[L.E]
    m = [U[L.m(0)], U[L.m(1)]]
    rho = [m[0] / py, m[1] / (1 - py)]
    lam = U[L.lam] / m[0]
    args = (py, rho, lam, solid, pb.reactive, W[L.p].astype(LD))
    ref = pressure_of(E, *args)
    du = LD(2.0) ** -53
    dlam = np.abs(pressure_of(E, py, rho, lam - 8 * du, *args[3:]) - ref) / 8
    dE = np.abs(pressure_of(E * (1 + 8 * du), *args) - ref) / 8
    assert np.all(np.abs(p - ref) <= 2 * (dlam + dE)), float((np.abs(p - ref) / (dlam + dE)).max())

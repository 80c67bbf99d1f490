"""The fluxes recorded at a refined patch's boundary are the ones the sweep
applied: a cell's update is U - nu (F_right - F_left) with the recorded pair,
to the rounding of that expression, for the general and the calibrated
arithmetic (see tests/flux_units.hip)."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2009_14555_amd import problems as P
from tests.parity_util import to_np

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("d", [0, 1])
@pytest.mark.parametrize("limiter", [P.LIM_MINMOD, P.LIM_VANALBADA])
def test_recorded_fluxes_are_the_sweeps(limiter, d):
    """at rest at 1e9 Pa, so that the momentum update is a small difference of
    large fluxes: one rounding of a flux is 1e8 times the bound, which is one
    rounding each of the difference, of its product with nu and of the sum"""
    import torch

    from paper_2009_14555_amd import dimp as D
    from paper_2009_14555_amd import solver as S

    lib = C.CDLL(os.path.join(HERE, "libdimp_fluxunits.so"))
    n = (70, 66)
    pb = P.Problem(ndim=2, n=(n[0], n[1], 1), dx=(1 / n[0], 1 / n[1], 1), bc=(P.BC_PERIODIC,) * 3,
                   materials=[P.water_sg(), P.solid_c2()], thinc=1, limiter=limiter)
    L = P.layout(pb)
    rng = np.random.default_rng(3)
    y, x = np.meshgrid((np.arange(n[1]) + 0.5) / n[1], (np.arange(n[0]) + 0.5) / n[0], indexing="ij")
    W = np.zeros((L.nfields, n[1], n[0]))
    W[0] = np.clip(0.5 + (np.hypot(x - 0.5, y - 0.5) - 0.25) * 30, 1e-6, 1 - 1e-6)  # a solid disc in water
    W[1] = 1000.0 * (1 + 1e-3 * rng.uniform(-1, 1, x.shape))
    W[2] = 2700.0 * (1 + 1e-3 * rng.uniform(-1, 1, x.shape))
    W[L.p] = 1e9 * (1 + 1e-9 * rng.uniform(-1, 1, x.shape))
    for q, (i, j) in enumerate(P.vbar_components(2)):
        W[L.V(q)] = float(i == j)
    g = S.Grid(pb)
    g.set_primitive(W)
    U = g.state.clone()
    mats = (D.dimp_material * 2)(*[D.material(m) for m in pb.materials])
    opt = D.options(pb)
    dt = 0.3 * pb.dx[0] / 8500.0
    nt = n[1 - d] - 2
    for pos in (5, 18, 34, 35, 52, 59):  # both sides of the interface, the ends of a 58-cell segment
        Un, flux = torch.empty_like(U), torch.empty((L.nfields, 2, nt), dtype=torch.float64, device=U.device)
        rc = lib.flux_unit(mats, C.byref(opt), (C.c_int64 * 2)(*n), (C.c_double * 2)(*pb.dx[:2]),
                           int(limiter == P.LIM_VANALBADA), d, C.c_double(dt), C.c_int64(pos), C.c_int64(1),
                           C.c_int64(nt), C.c_void_p(U.data_ptr()), C.c_void_p(Un.data_ptr()),
                           C.c_void_p(flux.data_ptr()))
        assert rc == 0
        u0, u1, F = to_np(U), to_np(Un), to_np(flux)
        c = (slice(None), slice(1, 1 + nt), pos) if d == 0 else (slice(None), pos, slice(1, 1 + nt))
        u0, u1 = u0[c].astype(np.longdouble), u1[c].astype(np.longdouble)
        nu = np.longdouble(dt) / np.longdouble(pb.dx[d])
        inc = nu * (F[:, 1].astype(np.longdouble) - F[:, 0].astype(np.longdouble))
        cons = list(range(L.nphi, L.V(0)))  # the fields a patch's boundary corrects
        # nu itself is rounded up to twice (dt times the inverse width)
        bound = 2.0**-53 * (4 * np.abs(inc) + np.maximum(np.abs(u0), np.abs(u1)))
        off = np.abs(u1 - (u0 - inc)) - bound
        assert np.all(off[cons] <= 0), (pos, d, [(f, float((np.abs(u1 - (u0 - inc)) / bound)[f].max())) for f in cons])


@pytest.mark.parametrize("integrator", ["split", "rk3"])
def test_refined_interface_conserves_with_van_albada(integrator):
    """a solid disc moving in water, THINC on, its interface crossing the patch's
    boundary: the composite grid keeps partial masses, momentum and energy to
    round-off (the bound of the other refinement tests)"""
    from oracle import amr as A
    from paper_2009_14555_amd import solver as S
    from tests.test_oracle_amr import prolong_prim

    n, box = (40, 36), (8, 7, 24, 27)
    pbc = P.Problem(ndim=2, n=(n[0], n[1], 1), dx=(1 / n[0], 1 / n[1], 1), bc=(P.BC_PERIODIC,) * 3,
                    materials=[P.water_sg(), P.solid_c2()], thinc=1, limiter=P.LIM_VANALBADA, cfl=0.4)
    L = P.layout(pbc)
    x, y = P.cell_centres(pbc)
    W = P.blank_prim(pbc)
    W[L.phi(0)] = np.clip(0.5 + (np.hypot(x - 0.5, y - 0.5) - 0.22) * n[0], 1e-6, 1 - 1e-6)
    W[L.rho(0)] = 1000.0 * (1 + 0.01 * np.sin(2 * np.pi * (x + y)))
    W[L.rho(1)] = 2700.0
    W[L.u(0)], W[L.u(1)] = 60.0, 20.0 * np.cos(2 * np.pi * x)
    W[L.p] = 1e8 * (1 + 0.5 * np.exp(-60.0 * ((x - 0.4) ** 2 + (y - 0.5) ** 2)))
    pbf = A.fine_problem(pbc, box)
    gc, gf = S.Grid(pbc), S.Grid(pbf)
    gc.set_primitive(W)
    gf.set_primitive(prolong_prim(pbc, W, pbf, box)[0])
    gc.set_integrator(integrator)
    gf.set_integrator(integrator)
    h = S.Hierarchy(gc, gf, box)
    cons = list(range(L.nphi, L.V(0)))
    inner = A.interior_mask(box)
    i0, j0, i1, j1 = box

    def totals():
        Uc, Uf = to_np(gc.state), to_np(gf.state)
        out = Uc[cons].sum(axis=(1, 2)) - Uc[cons, j0:j1, i0:i1].sum(axis=(1, 2))
        return out + Uf[cons][:, inner].sum(axis=1) / 4

    m0 = totals()
    for _ in range(12):
        h.advance(h.dt(pbc.cfl))
    drift = np.abs(totals() - m0) / np.maximum(np.abs(m0), 1.0)
    h.close()
    assert np.all(np.isfinite(drift)) and np.all(drift < 1e-12), drift

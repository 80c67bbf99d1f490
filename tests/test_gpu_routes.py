"""The instances and launch shapes that a step chooses by its materials and its
size, at the edges of each rule: material profiles and the general instance
against the oracle, the runs of blocks, the slots of the wave-speed reduction,
and the adjoint's general instance against the oracle's dual numbers."""
import dataclasses

import numpy as np
import pytest

from paper_2009_14555_amd import problems as P
from tests.parity_util import TOL, assert_parity, to_np
from tests.test_gpu_adjoint import directions

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_14555_amd import solver

    return solver


SOLID_AB = dataclasses.replace(P.solid_c2(yield_stress=0.05e9), abar=1.3, bbar=2.5)
IG_HALF = dataclasses.replace(P.lx17(0), ig=dict(P.lx17(0).ig, x=6.5, y=2.5, d=1.5))
# name: materials, reactive mixture (the Johnson-Cook instances have their own
# tests, which start from a plastic strain above its rounding)
MATERIALS = {
    "gas_solid": ([P.water_sg(), P.solid_c2(yield_stress=0.05e9)], None),
    "solid_gas": ([P.solid_c2(yield_stress=0.05e9), P.water_sg()], None),
    "gas_solid_exponents": ([P.water_sg(), SOLID_AB], None),
    "gas_gas": ([P.water_sg(), P.air()], None),
    "mix_solid": ([P.placeholder_for_reactive(), P.solid_c2()], P.generic_explosive(0)),
    "solid_mix": ([P.solid_c2(), P.placeholder_for_reactive()], P.generic_explosive(1)),
    "mix_solid_power": ([P.placeholder_for_reactive(), P.solid_c2()], P.generic_explosive(0, n=1.5)),
    "jwl_solid": ([P.placeholder_for_reactive(), P.solid_c2()], P.lx17(0)),
    "jwl_solid_exponents": ([P.placeholder_for_reactive(), P.solid_c2()], IG_HALF),
}
# x rows of 58 + 1 and 58 - 1 cells and one that is not a multiple of the tile's
# four columns; in 3-D eight columns and one more, and 58 + 2 and 58 + 1 cells
# along the tile's axis
GRIDS = {"1d": (117,), "2d": (59, 61), "2d_narrow": (57, 9), "3d_y": (9, 60, 6), "3d_z": (8, 6, 59)}


@pytest.mark.parametrize("limiter", [P.LIM_MINMOD, P.LIM_VANALBADA])
@pytest.mark.parametrize("grid", list(GRIDS))
@pytest.mark.parametrize("mats", list(MATERIALS))
def test_instances_match_oracle(S, mats, grid, limiter):
    from oracle import pyoracle as O

    n = GRIDS[grid]
    d = len(n)
    m, rx = MATERIALS[mats]
    kw = {} if rx is None else {"reactive": rx}
    pb = P.Problem(ndim=d, n=tuple(n) + (1,) * (3 - d), dx=tuple(1.0 / k for k in n) + (1.0,) * (3 - d),
                   bc=(P.BC_PERIODIC,) * 3, materials=m, thinc=1, limiter=limiter, **kw)
    L = P.layout(pb)
    W = P.random_smooth_state(pb, seed=11, solid_strain=1e-3)
    if mats.startswith("jwl"):  # a state on the curves of the explosive
        W[L.rho(0)] *= 1.905
        W[L.p] *= 50.0
    o, g = O.Oracle(pb), S.Grid(pb)
    g.set_primitive(W)
    U = o.prim_to_cons(W)
    for k in range(3):
        dt = o.dt_cfl(U)
        U = o.step(U, dt, k)
        g.advance(dt)
        np.testing.assert_allclose(g.max_wavespeed(), o.max_wavespeed(U), rtol=TOL)
    assert_parity(to_np(g.state), U, TOL, f"{mats} {grid}", L)


@pytest.mark.parametrize("d", [0, 1])
@pytest.mark.parametrize("blocks", [1, 255, 256, 257, 1023, 1024, 1040, 16383, 16384, 16500])
def test_every_block_of_a_sweep_runs_once(S, blocks, d):
    """lines along the sweep axis that hold the same cells leave with the same
    bits, whichever block took them (four lines a block)"""
    import torch

    n = (58, 4 * blocks) if d == 0 else (4 * blocks, 58)
    pb = P.Problem(ndim=2, n=n + (1,), dx=(1 / 58, 1 / 58, 1), materials=[P.water_sg(), P.solid_c2()], thinc=1)
    g = S.Grid(pb)
    row = P.random_smooth_state(P.Problem(ndim=1, n=(58, 1, 1), dx=(1 / 58, 1, 1),
                                          materials=pb.materials, thinc=1), seed=2)
    L, L1 = P.layout(pb), P.layout(P.Problem(ndim=1, n=(58, 1, 1), dx=(1 / 58, 1, 1), materials=pb.materials))
    line = np.zeros((L.nfields, 58))
    for dst, src in [(L.phi(0), L1.phi(0)), (L.rho(0), L1.rho(0)), (L.rho(1), L1.rho(1)), (L.p, L1.p),
                     (L.u(d), L1.u(0))]:
        line[dst] = row[src].ravel()
    for q, (i, j) in enumerate(P.vbar_components(2)):
        line[L.V(q)] = 1.0 if i == j else 0.0
    line = torch.as_tensor(line, device="cuda")
    W = (line[:, None, :] if d == 0 else line[:, :, None]).expand(L.nfields, n[1], n[0]).contiguous()
    g.set_primitive(W)
    before = g.state.clone()
    g.sweep(1e-6, d)
    U = g.state
    ref = U[:, :1, :] if d == 0 else U[:, :, :1]
    assert bool((U == ref).all())
    assert bool((U[L.E] != before[L.E]).any(dim=1 - d).all())


@pytest.mark.parametrize("integ", ["split", "rk3"])
@pytest.mark.parametrize("copies", [192, 193])
def test_wide_tiles_match_narrow(S, copies, integ):
    """a y sweep of a grid past the cache (eight columns by eight waves) against
    the same columns of a small one; 61 columns leave a part of a tile, and a
    part of eight.  The same stages in another instance: a few roundings"""
    import torch

    def grid(nx):
        pb = P.Problem(ndim=2, n=(nx, 130, 1), dx=(1 / 61, 1 / 130, 1), bc=(P.BC_PERIODIC,) * 3,
                       materials=[P.water_sg(), P.solid_c2(yield_stress=0.05e9)], thinc=1)
        return pb, S.Grid(pb)

    pb, g = grid(61)
    W = torch.as_tensor(P.random_smooth_state(pb, seed=4, solid_strain=1e-3), device="cuda")
    g.set_primitive(W)
    pb2, h = grid(61 * copies)
    assert (2 * 8 * P.layout(pb).nfields * h.pb.ncell > 2**28) == (copies > 192)
    h.set_primitive(W.reshape(-1, 130, 61).repeat(1, 1, copies))
    dt = g.dt_cfl()
    for a in (g, h):
        if integ == "rk3":
            a.set_integrator("rk3")
            a.advance(dt)
        else:
            a.sweep(dt, 1)
    ref = to_np(g.state).reshape(-1, 130, 61)
    out = to_np(h.state).reshape(-1, 130, copies, 61)
    for k in (0, 1, 7, copies // 2, copies - 1):
        assert_parity(out[:, :, k], ref, 1e-13, f"copy {k}", P.layout(pb))


@pytest.mark.parametrize("slots", [1, 63, 64, 65, 256, 257, 1024, 1025, 2048, 2049])
def test_wave_speed_reduction_finds_its_slot(S, slots):
    """one row of 58 cells a slot after a fused x sweep; the fastest row is the
    last, then a NaN in the first"""
    import torch

    pb = P.Problem(ndim=2, n=(58, slots, 1), dx=(1 / 58, 1 / 58, 1), materials=[P.water_sg(), P.solid_c2()], thinc=1)
    L = P.layout(pb)
    W = P.blank_prim(pb)
    W[L.phi(0)], W[L.rho(0)], W[L.rho(1)], W[L.p] = 1.0 - 1e-6, 1000.0, 2700.0, 1e5
    W[L.p][..., -1, :] = 1e9
    g, h = S.Grid(pb), S.Grid(pb)
    g.set_primitive(W)
    for bad in (False, True):
        g.set_step_index(1)  # y, then x with the sources and the wave speed
        if bad:
            U = g.state.clone()
            U[L.E, 0, 0] = float("nan")
            g.set_conserved(U)
            g.set_step_index(1)
        g.advance(1e-9)
        s = g.max_wavespeed()
        h.set_conserved(g.state)
        t = h.max_wavespeed()  # from the state, 256 cells a slot
        if bad:
            assert np.isnan(s).any() and np.isnan(t).any()
        else:
            # (two evaluations of the same closures: some tens of roundings)
            np.testing.assert_allclose(s[:2], t[:2], rtol=1e-13)
            assert s[0] > 2000.0  # the last row's 2653: the others' is 1625


@pytest.mark.parametrize("cells", [1, 255, 256, 257, 65536 * 8 - 256, 65536 * 8, 65536 * 8 + 1])
def test_wave_speed_of_a_state(S, cells):
    """256 cells a slot, up to 2048 slots in one reduction: the last cell's is found"""
    pb = P.Problem(ndim=1, n=(cells, 1, 1), dx=(1.0, 1, 1), materials=[P.water_sg(), P.air()], thinc=0)
    L = P.layout(pb)
    W = P.blank_prim(pb)
    W[L.phi(0)], W[L.rho(0)], W[L.rho(1)], W[L.p] = 1.0 - 1e-6, 1000.0, 1.0, 1e5
    W[L.u(0)][..., -1] = -700.0
    g = S.Grid(pb)
    g.set_primitive(W)
    W1 = W[..., -1:]
    from oracle import pyoracle as O

    o = O.Oracle(pb.replace(n=(1, 1, 1)))
    np.testing.assert_allclose(g.max_wavespeed()[0], o.max_wavespeed(o.prim_to_cons(np.ascontiguousarray(W1)))[0],
                               rtol=1e-13)


@pytest.mark.parametrize("mats", ["solid_gas", "gas_solid_exponents"])
@pytest.mark.parametrize("k", [0, 1])
def test_adjoint_general_instance_matches_dual_numbers(S, mats, k):
    """materials outside the adjoint's compiled profile, on a smooth periodic
    field: the bars of the profile's own dual-number test"""
    import torch

    from oracle import pyoracle as O

    n = (40, 36)
    pb = P.Problem(ndim=2, n=n + (1,), dx=(1 / n[0], 1 / n[1], 1), bc=(P.BC_PERIODIC,) * 3,
                   materials=MATERIALS[mats][0], thinc=1, limiter=P.LIM_VANALBADA)
    g = S.Grid(pb)
    g.set_primitive(P.random_smooth_state(pb, seed=6, solid_strain=3e-3))
    U = to_np(g.state).copy()
    dt = g.dt_cfl()
    v, w = directions(U, 70 + k)
    solid = 0 if mats == "solid_gas" else 1
    slots = [(1 - solid, 0), (1 - solid, 1), (solid, 2), (solid, 3)]
    dpar = np.zeros((5, 2, 4))
    for j, (mat, col) in enumerate(slots):
        dpar[1 + j, mat, col] = 1.0
    dU = np.zeros((5,) + U.shape)
    dU[0] = v
    _, T = O.Oracle(pb).step_dual(U, dU, dpar, dt, k)
    dp = torch.zeros(12, dtype=torch.float64, device="cuda")
    lam = to_np(g.adjoint_step(U, w, dt, k, dp))
    grad = g.adjoint_params(dp)
    lhs = float(np.sum(w * T[0]))
    assert abs(lhs - float(np.sum(lam * v))) <= 1e-7 * abs(lhs)
    for j, (mat, col) in enumerate(slots):
        lhs = float(np.sum(w * T[1 + j]))
        assert abs(lhs - float(grad[mat, col])) <= 1e-9 * max(abs(lhs), abs(float(grad[mat, col])), 1e-300), (mat, col)

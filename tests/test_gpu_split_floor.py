"""The App. B split of a JWL mixture in the cells of a detonation front whose
pressure function cancels strongly (the Newton steps end at the rounding noise
of the residual there): GPU against the oracle's bisection."""
import numpy as np
import pytest

from paper_2009_14555_amd import problems as P
from tests.parity_util import field_rel_diff


def front_state(nx, ny, seed, traces):
    """a rate stick with a reaction zone of 20 rows at rest ahead and moving
    behind; traces: the mixture's share of the confiner"""
    pb, W = P.rate_stick(nx, ny, seed=seed)
    L = P.layout(pb)
    x, y = P.cell_centres(pb)
    xi = np.clip((y - 0.4 * ny * pb.dx[1]) / (20 * pb.dx[1]) + 0.5, 0.0, 1.0)
    front = xi * xi * (3.0 - 2.0 * xi)
    inside = W[L.phi(0)] > 0.5
    # progress and pressure of the front everywhere, the confiner's traces included
    W[L.lam] = front
    W[L.p] = np.where(inside, 27e9 * (1.0 - front) + 1e5, W[L.p])
    W[L.phi(0)] = np.where(inside, W[L.phi(0)], traces)
    W[L.u(1)] = np.where(inside, 1500.0 * (1.0 - front), 0.0)
    return pb, W


@pytest.mark.gpu
@pytest.mark.parametrize("traces", [1e-6, 1e-3])
@pytest.mark.parametrize("nx,ny", [(40, 90), (61, 64)])
def test_split_at_the_noise_floor_matches_bisection(nx, ny, traces):
    from oracle import pyoracle as O
    from paper_2009_14555_amd import solver as S

    pb, W = front_state(nx, ny, 3, traces)
    o = O.Oracle(pb)
    g = S.Grid(pb)
    g.set_primitive(W)
    U = o.prim_to_cons(W)
    for k in range(2):
        dt = o.dt_cfl(U)
        U = o.step(U, dt, k)
        g.advance(dt)
        # the parity bound of every stored field against the oracle
        assert np.all(field_rel_diff(g.state.cpu().numpy(), U, P.layout(pb)) <= 1e-10)

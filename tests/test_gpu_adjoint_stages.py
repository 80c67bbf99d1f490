"""Every reverse stage of the adjoint against central differences of the stage of
the calibrated step that it reverses, in both instances of the reverse stages
(see tests/adjoint_stages.hip); states and acceptance as in
tests/test_gpu_adjoint_units.py."""
import ctypes as C
import os

import numpy as np
import pytest

from tests.test_gpu_adjoint_units import HERE, STAGES, env, inputs, scale_of  # noqa: F401  (env: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gs", [0, 1])
@pytest.mark.parametrize("d", [0, 1])
@pytest.mark.parametrize("stage", list(STAGES))
def test_stage_against_finite_differences(env, stage, d, gs):  # noqa: F811
    units, D, states = env
    lib = C.CDLL(os.path.join(HERE, "libdimp_adjstages.so"))
    ni, no = C.c_int(), C.c_int()
    assert units.unit_sizes(STAGES[stage], C.byref(ni), C.byref(no)) == 0
    ptr = lambda a: a.ctypes.data_as(C.POINTER(C.c_double))  # noqa: E731
    for si, (pb, U, W) in enumerate(states):
        rng = np.random.default_rng(200 + si)
        X, sc = inputs(stage, d, U, W, rng, 400)
        V = rng.standard_normal(X.shape) * sc
        WY = rng.standard_normal((X.shape[0], no.value))
        X, V, WY = (np.ascontiguousarray(a, dtype=np.float64) for a in (X, V, WY))
        assert X.shape[1] == ni.value
        mats = (D.dimp_material * 2)(*[D.material(m) for m in pb.materials])
        opt, dx = D.options(pb), (C.c_double * 2)(*pb.dx[:2])
        best = None
        for eps in (1e-7, 1e-9):
            out = np.zeros(2 * X.shape[0])
            assert lib.stage_run(gs, STAGES[stage], d, mats, C.byref(opt), dx, C.c_double(0.3), X.shape[0], ptr(X),
                                 ptr(V), ptr(WY), C.c_double(eps), ptr(out)) == 0
            fd, ad = out[0::2], out[1::2]
            rel = np.abs(fd - ad) / np.maximum(np.maximum(np.abs(fd), np.abs(ad)), 1e-300)
            q = (np.median(rel), np.quantile(rel, 0.9))
            best = q if best is None or q[0] < best[0] else best
        assert best[0] < 1e-5 and best[1] < 1e-3, (stage, d, gs, si, best)

"""The stages' reciprocal, quotient, root and exponential against extended
precision: rounded as the IEEE operations (and no further off than the library's
exponential) that they stand in place of."""
import ctypes as C
import os

import numpy as np
import pytest

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

"""Kernels whose stages read the parameters anew from the kernel's arguments take
them first: their launcher does not compile for any other signature."""
import os
import subprocess

import pytest

from paper_2009_14555_amd import build as B

KERNEL = """
#include "dimp_device.hpp"
__global__ void k(%s) {}
void f(const dimp::Params& P, double* out) { dimp::launch_params(k, dim3(1), dim3(64), 0, nullptr, %s); }
"""


@pytest.mark.parametrize("params,args,ok", [("dimp::Params P, const double* o, int n", "P, out, 3", True),
                                            ("int n, dimp::Params P", "3, P", False),
                                            ("const double* o, dimp::Params P", "P, out", False),
                                            ("dimp::Params P, const double* o", "P", False)])
def test_launcher_takes_params_first(tmp_path, params, args, ok):
    src = tmp_path / "k.hip"
    src.write_text(KERNEL % (params, args))
    flags = [f for f in B.FLAGS if f not in ("-shared", "-Wall")]
    r = subprocess.run([B.HIPCC, *flags, "-fsyntax-only", "--offload-host-only", "-I", B.CSRC, str(src)],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr


@pytest.mark.parametrize("name", ["dimp_sweeps.hpp", "dimp_patches.hpp"])
def test_sweeps_are_launched_by_it(name):
    src = open(os.path.join(B.CSRC, name)).read()
    assert "launch_params(" in src and "hipLaunchKernelGGL" not in src

"""The general conversion of a state with a history slot (any materials) stays in
registers: no private memory per lane."""
import re
import subprocess

import pytest

from paper_2009_14555_amd import build as B

KERNEL = """
#include "dimp_stencil.hpp"
using namespace dimp;
__global__ __launch_bounds__(256) void k(Params P, const double* U, double* W) {
  using L = Lay<2, 2, HIST>;
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nc = P.ncell;
  if (c >= nc) return;
  double u[L::F], w[L::F], H[6], J2;
  for (int f = 0; f < L::F; ++f) u[f] = U[f * nc + c];
  Thermo<2, HIST> T;
  cons_to_prim<2, 2, HIST>(P, u, w, T, H, J2);
  for (int f = 0; f < L::F; ++f) W[f * nc + c] = w[f];
}
"""


@pytest.mark.parametrize("rx", [1, 2])
def test_conversion_needs_no_private_memory(tmp_path, rx):
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(KERNEL.replace("HIST", str(rx)))
    flags = [f for f in B.FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", "-I", B.CSRC, str(src), "-o", str(out)], check=True,
                   capture_output=True)
    sizes = re.findall(r"\.private_segment_fixed_size:\s*(\d+)", out.read_text())
    assert sizes == ["0"]

"""The factorisation without general interchanges, for systems with and without a
declared one: the compiler finds no subscript outside its array (no GPU).
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_02876_amd", "csrc")

SOURCE = """
#include <hip/hip_runtime.h>
#include "erk.h"
using namespace ens;
__global__ void step(const double* y, const double* p, double h, double* o) {
  PlainMat<SYSTEM, double> F;
  o[0] = ros_factor_plain<SYSTEM, METHOD, double>(y, p, h, F);
}
"""


@pytest.mark.parametrize("system", ["Robertson", "Linear", "Hires"])
@pytest.mark.parametrize("method", ["Rodas4", "Ros23"])
def test_subscripts_in_bounds(tmp_path, system, method):
    src = tmp_path / "check.hip"
    src.write_text(SOURCE.replace("SYSTEM", system).replace("METHOD", method))
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only",
                        "-std=c++17", "-Werror=array-bounds", "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"), str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

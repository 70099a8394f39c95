"""The checkpointed given-mesh kernels keep four blocks of 256 lanes on a compute
unit: at most 40 KB of its 160 KB of LDS a block (the compiler's report, no GPU).
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_02876_amd", "csrc")

SOURCE = """
#include <hip/hip_runtime.h>
#include "erk.h"
namespace ens {
template __global__ void erk_forward_kernel<KERNEL, true, false, false>(const FwdArgs);
}
"""


@pytest.mark.parametrize("kernel", [
    "Lorenz, Tsit5, double, MODE_FROZEN", "Lorenz, Tsit5, float, MODE_REFRESH",
    "Robertson, Ros23, double, MODE_FROZEN"])
def test_lds_leaves_room_for_four_blocks(tmp_path, kernel):
    src = tmp_path / "check.hip"
    src.write_text(SOURCE.replace("KERNEL", kernel))
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-c", "-O1",
                        "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops",
                        "-Rpass-analysis=kernel-resource-usage", "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"), str(src), "-o",
                        str(tmp_path / "check.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lds = [int(x) for x in re.findall(r"LDS Size \[bytes/block\]: (\d+)", r.stderr)]
    assert lds and max(lds) <= 40960, lds

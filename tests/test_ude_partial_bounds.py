"""The UDE sweep's weight-gradient partial of a wavefront, written and read as
one row of UDE_NP floats of the tile storage, lies inside that row (checked by
the compiler, no GPU).
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_02876_amd", "csrc")

SOURCE = """
#include <hip/hip_runtime.h>
#include <type_traits>
#include "ude.h"
using Tile = decltype(ens::UdeLds::tile);
static_assert(std::rank<Tile>::value == 2 &&
              std::extent<Tile, 0>::value == ens::UDE_WAVES &&
              std::extent<Tile, 1>::value >= ens::UDE_NP, "a row holds a partial");
"""


def test_a_row_holds_a_partial(tmp_path):
    src = tmp_path / "check.hip"
    src.write_text(SOURCE)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only",
                        "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                        str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

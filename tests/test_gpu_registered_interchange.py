"""Registered systems of d >= 6 that change rows often: after some failed attempts
in a row a wavefront stops trying the factorisation without interchanges for a
few steps.  A registered copy of HIRES (with and without the Jacobian's pattern;
no declared interchange) against the built-in one, bit for bit: rate constants
under which rows change places in hardly any step, in nearly every one, or in
some trajectories of each wavefront, over enough steps that the attempts stop
and start again; records, checkpointed ones, replays, solves and gradients.
"""
import os
import re

import numpy as np
import pytest
import torch

from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_2609_02876_amd", "csrc", "systems.h")


def _source(rows):
    body = re.search(r"struct Hires \{(.*?)\n\};", open(HEADER).read(), re.S).group(1)
    pattern = re.search(r"  static constexpr unsigned JAC_ROWS.*?;\n", body).group(0)
    body = body[body.index("  template <class T>"):].replace("__device__ static inline",
                                                            "__device__ static")
    body = re.sub(r"#pragma unroll\n.*?J\[i\] = T\(0\);",
                  " ".join(f"J[{i}] = T(0);" for i in range(64)), body)
    return "struct System {\n" + (pattern if rows else "") + body + "\n};\n"


@pytest.fixture(scope="module")
def systems():
    for rows in (False, True):
        B.register_system(f"gpu_interchange_hires_{int(rows)}", _source(rows), 8, 12,
                          jacobian=True)


@pytest.mark.parametrize("method", ["rodas4", "ros23"])
@pytest.mark.parametrize("which", ["few", "most", "some"])
@pytest.mark.parametrize("rows", [False, True])
def test_equals_the_built_in_system(systems, rows, which, method):
    n, t1, rtol = 200, 60.0, 1e-4
    print(f"case registered hires rows={rows} {method} {which}", flush=True)
    y0, p = W.hires(n, 3)
    many = {"few": np.zeros(n, bool), "most": np.ones(n, bool),
            "some": np.random.default_rng(2).random(n) < 0.1}[which]
    p[:, 2] = np.where(many, 4.0 * p[:, 4], 0.2 * p[:, 4])
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), dtype=torch.float64, device="cuda")
    y0, p = dev(y0), dev(p)
    times = [0.4 * t1, t1]
    out = []
    for system in ("hires", f"gpu_interchange_hires_{int(rows)}"):
        a = (system, method, y0, p, 0.0, t1, rtol, 1e-4 * rtol)
        rec = B.ensemble_record(*a, save_times=times, steps_hint=8192)
        h, S = B.ensemble_mesh_export(rec)
        ck = B.ensemble_record(*a, save_times=times, steps_hint=8192, ckpt_every=16)
        rep = B.ensemble_replay_mesh(system, method, y0, p, 0.0, t1, h, S, save_times=times,
                                     ckpt_every=16)
        ys, status = B.ensemble_solve(*a, save_times=times)
        got = [h, S, rec.status, rec.n_trial(), rec.y_save, ck.y_save, rep.y_save, ys, status]
        for hd in (rec, ck, rep):
            got += list(B.ensemble_adjoint(hd))
        out.append([t.clone() for t in got])
    assert int(out[0][2].abs().max()) == 0 and int(out[0][1].max()) > 20
    for a, b in zip(*out):
        assert torch.equal(a, b)

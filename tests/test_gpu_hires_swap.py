"""The one interchange the HIRES factorisation makes without going to the
general path (rows 1 and 3 in column 1), alone, beside the others and beside
none: rate constants under which steps of a given size make it, make another
one (rows 2 and 3 in column 2), both or neither, in ensembles of one kind and
of all.  Each lane against the oracle on the same mesh (1e-11 of its norm) and,
bit for bit, against itself alone.
"""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import oracle_mesh
from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method,t1", [("rodas4", 0.9), ("ros23", 2.0)])
@pytest.mark.parametrize("which", ["neither", "swap", "other", "both", "mixed"])
@pytest.mark.parametrize("ckpt", [0, 16])
def test_swap(method, t1, which, ckpt):
    n = 70
    print(f"case {method} {which} ckpt {ckpt}", flush=True)
    y0, p = W.hires(n, 3)
    kind = np.arange(n) % 4 if which == "mixed" else np.full(
        n, ["neither", "swap", "other", "both"].index(which))
    p[:, 2] = np.where(kind & 1, 1.5 * p[:, 4], 0.2 * p[:, 4])
    p[:, 5] = np.where(kind & 2, 0.05 * p[:, 0], p[:, 5])
    p[:, 8] = 2.0 * p[:, 0]
    S = (1 + np.arange(n) % 3).astype(np.int32)
    h = np.zeros((3, n))
    for l in range(n):
        h[:S[l], l] = t1 / S[l]
    dev = lambda a, t=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=t, device="cuda")

    def run(idx):
        return B.ensemble_replay_mesh("hires", method, dev(y0[idx].T), dev(p[idx].T), 0.0, t1,
                                      dev(h[:, idx]), dev(S[idx], torch.int32),
                                      save_times=[0.3 * t1, t1], ckpt_every=ckpt)

    hd = run(np.arange(n))
    gp, gy, _ = (a.cpu().numpy() for a in B.ensemble_adjoint(hd))
    gp_o, gy_o, _ = O.adjoint(O.HIRES, {"rodas4": O.RODAS, "ros23": O.ROS23}[method], y0, p,
                              oracle_mesh(hd))
    for a, b in ((gp.T, gp_o), (gy.T, gy_o)):
        e = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
        print(f"  worst {e.max():.2e}")
        assert e.max() <= 1e-11
    for l in (0, 1, 2, 3, 63, 69):
        one = B.ensemble_adjoint(run(np.array([l])))
        assert np.array_equal(one[0][:, 0].cpu().numpy(), gp[:, l])
        assert np.array_equal(one[1][:, 0].cpu().numpy(), gy[:, l])

"""The Rosenbrock paths with and without row interchanges, at the border
between them: wavefronts in which no lane, one lane, some or all lanes meet a
column whose largest entry is off the diagonal.  A trajectory's results may not
depend on its neighbours' path: each lane's gradient in a mixed ensemble equals,
bit for bit, the one it gets alone, and the oracle's on the same mesh (1e-11 of
its norm).
"""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import oracle_mesh
from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("method", ["rodas4", "ros23"])
@pytest.mark.parametrize("which", ["none", "one", "some", "all"])
@pytest.mark.parametrize("system", ["linear", "hires"])
def test_lane_is_its_own(system, which, method):
    n = 70
    print(f"case {system} {method} {which}", flush=True)
    rng = np.random.default_rng(8)
    many = {"none": np.zeros(n, bool), "one": np.arange(n) == 17,
            "some": rng.random(n) < 0.3, "all": np.ones(n, bool)}[which]
    if system == "linear":
        # W = [[1/(gamma h) + a, w], [-w, 1/(gamma h) + a]]: rows change places
        # once w exceeds the diagonal
        y0 = rng.normal(size=(n, 2))
        p = np.stack([np.full(n, 0.2), np.where(many, 9.0, 0.01)], 1)
        t1, rtol = 4.0, 1e-2
    else:
        # column 1 holds p2 and p4 (in balance in the model): p2 well above p4
        y0, p = W.hires(n, 3)
        p[:, 2] = np.where(many, 4.0 * p[:, 4], 0.2 * p[:, 4])
        t1, rtol = 20.0, 1e-4
    run = lambda idx: B.ensemble_record(system, method, _dev(y0[idx].T), _dev(p[idx].T), 0.0, t1,
                                        rtol, 1e-2 * rtol, save_times=[0.4 * t1, t1],
                                        steps_hint=512)
    hd = run(np.arange(n))
    gp, gy, ll = (a.cpu().numpy() for a in B.ensemble_adjoint(hd))
    assert np.all(hd.status.cpu().numpy() == 0)
    gp_o, gy_o, ll_o = O.adjoint({"linear": O.LINEAR, "hires": O.HIRES}[system],
                                 {"rodas4": O.RODAS, "ros23": O.ROS23}[method], y0, p,
                                 oracle_mesh(hd))
    for a, b in ((gp.T, gp_o), (gy.T, gy_o)):
        e = np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)
        print(f"  worst {e.max():.2e}")
        assert e.max() <= 1e-11
    for l in (0, 17, 18, 63, 64, 69):
        one = B.ensemble_adjoint(run(np.array([l])))
        assert np.array_equal(one[0][:, 0].cpu().numpy(), gp[:, l])
        assert np.array_equal(one[1][:, 0].cpu().numpy(), gy[:, l])

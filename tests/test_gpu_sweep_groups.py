"""Full-tape sweep by groups of four steps: trajectories of one wavefront with
every remainder of the step count modulo the group and the page (1 .. 35 steps),
on given uniform meshes, against the FP64 oracle on the same meshes (FP64 bar
1e-11; FP32 1e-4 of each trajectory's gradient, floored at the ensemble's rms).
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W
from gpu_helpers import oracle_mesh

pytestmark = pytest.mark.gpu

SY = {"lorenz": O.LORENZ, "vdp": O.VDP, "robertson": O.ROBERTSON, "hires": O.HIRES}
ME = {"tsit5": O.TSIT5, "vern7": O.VERN7, "rodas4": O.RODAS, "ros23": O.ROS23}


@pytest.mark.parametrize("system,method,dtype,t1", [
    ("lorenz", "tsit5", "f64", 0.2), ("vdp", "vern7", "f64", 0.5), ("vdp", "tsit5", "f32", 0.5),
    ("robertson", "ros23", "f64", 0.3), ("hires", "rodas4", "f64", 1.0)])
def test_every_remainder(system, method, dtype, t1):
    n = 35
    print(f"case {system} {method} {dtype}", flush=True)
    y0, p = W.GENERATORS[system](n, 4)
    if dtype == "f32":
        y0, p = (a.astype(np.float32).astype(np.float64) for a in (y0, p))
    S = np.arange(1, n + 1, dtype=np.int32)[np.random.default_rng(1).permutation(n)]
    cap = int(S.max())
    h = np.zeros((cap, n))
    for l in range(n):
        h[:S[l], l] = t1 / S[l]
    tt = torch.float64 if dtype == "f64" else torch.float32
    dev = lambda a, t=tt: torch.tensor(np.ascontiguousarray(a), dtype=t, device="cuda")
    hd = B.ensemble_replay_mesh(system, method, dev(y0.T), dev(p.T), 0.0, t1,
                                dev(h, torch.float64), dev(S, torch.int32),
                                save_times=[0.0, 0.37 * t1, t1])
    gp, gy, ll = (t.cpu().numpy().astype(np.float64) for t in B.ensemble_adjoint(hd))
    assert np.all(hd.status.cpu().numpy() == 0)
    gp_o, gy_o, ll_o = O.adjoint(SY[system], ME[method], y0, p, oracle_mesh(hd))
    tol = 1e-11 if dtype == "f64" else 1e-4
    for a, b in ((gp.T, gp_o), (gy.T, gy_o)):
        norm = np.linalg.norm(b, axis=1)
        e = np.linalg.norm(a - b, axis=1) / np.maximum(norm, np.sqrt(np.mean(norm ** 2)))
        print(f"  worst {e.max():.2e}")
        assert e.max() <= tol
    assert np.abs(ll - ll_o).max() <= tol * np.abs(ll_o).max()

"""UDE kernels at the edges of their work split: 32 trajectories a wavefront,
128 a block (one trajectory, a wavefront and a block less and more one),
segments of 16 steps with trajectories of several segment counts, and weights
small enough for the tanh series alone and large enough for both branches.
Against the FP64 oracle on the oracle's mesh; the bar is the FP32 one, 1e-4 of
each quantity's scale.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL32 = 1e-4
T1 = 3.0
ST = [0.0, 0.4, 0.4, 1.7, 3.0]


def _dev(a, dtype=torch.float32):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


@pytest.mark.parametrize("ckpt", [0, 16])
@pytest.mark.parametrize("wscale", [0.1, 1.0])
@pytest.mark.parametrize("n", [1, 31, 33, 127, 129])
def test_ude_split(n, wscale, ckpt):
    print(f"case ude n={n} weights x{wscale} ckpt={ckpt}", flush=True)
    rng = np.random.default_rng(7)
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    y0 = f32(rng.uniform(0.5, 2.0, (n, 2)))
    th = f32(W.ude_weights(3, scale=wscale))
    ref = O.record(O.LV_UDE, O.TSIT5, y0, th, 0.0, T1, 1e-6, 1e-6, save_t=ST, params_shared=True)
    assert np.all(ref["status"] == O.ST_OK)
    gp_o, gy_o, ll_o = O.adjoint(O.LV_UDE, O.TSIT5, y0, th, ref, params_shared=True)
    g_o = gp_o.sum(axis=0)
    cap = int(ref["S"].max())
    hd = B.ensemble_replay_mesh("ude", "tsit5", _dev(y0.T), _dev(th), 0.0, T1,
                                _dev(ref["h"][:, :cap].T, torch.float64),
                                torch.tensor(ref["S"], dtype=torch.int32, device="cuda"),
                                save_times=ST, params_shared=True, ckpt_every=ckpt)
    gp, gy, ll = (t.cpu().numpy().astype(np.float64) for t in B.ensemble_adjoint(hd))
    assert np.all(hd.status.cpu().numpy() == 0)
    ys, ys_o = hd.y_save.cpu().numpy(), np.transpose(ref["y_save"], (1, 2, 0))
    for name, a, b in (("states", ys, ys_o), ("weights", gp, g_o), ("y0", gy, gy_o.T),
                       ("loss", ll, ll_o)):
        e = np.abs(a - b).max() / np.abs(b).max()
        print(f"  {name} {e:.2e}")
        assert e <= TOL32

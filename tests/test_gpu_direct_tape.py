"""Records that write each taped step at once (small ensembles) against those
that stage whole lines (large ones): the first trajectories of an ensemble,
recorded alone and as part of a large one, have the same steps, states and
gradients bit for bit -- with tapes that overflow their reserved pages, with
the longest reserve that still goes either way, and with save times at the
start, inside and at the end of the span (the save states of a small ensemble
are formed by several blocks).
"""
import pytest
import torch

from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("system,method,dtype,t1,ckpt,hint,sizes", [
    ("lorenz", "tsit5", "f64", 1.0, 0, 16, (257, 65536, 65537)),     # overflows
    ("lorenz", "tsit5", "f64", 1.0, 0, 512, (63, 32768, 32769)),     # tapes 16 KiB apart
    ("vdp", "vern7", "f32", 2.0, 0, 64, (1000, 65537)),
    ("lorenz", "vern7", "f64", 1.0, 16, 32, (257, 65536, 65537)),
    ("robertson", "rodas4", "f64", 10.0, 0, 16, (257, 65537)),
    ("robertson", "ros23", "f64", 10.0, 16, 64, (257, 65537)),
    ("hires", "rodas4", "f64", 5.0, 0, 64, (65, 65537)),
])
def test_small_and_large_agree(system, method, dtype, t1, ckpt, hint, sizes):
    tt = torch.float64 if dtype == "f64" else torch.float32
    y0, p = (torch.tensor(a.T.copy(), dtype=tt, device="cuda")
             for a in W.GENERATORS[system](sizes[-1], 3))
    times = [0.0, 0.2 * t1, 0.21 * t1, 0.7 * t1, t1]
    atol = 1e-10 if system in ("robertson", "hires") else 1e-8
    rtol = 1e-5 if dtype == "f32" else 1e-6
    pool = torch.empty(8 << 30, dtype=torch.uint8, device="cuda")
    ref = None
    for n in reversed(sizes):
        print(f"case {system} {method} {dtype} ckpt {ckpt} n {n}", flush=True)
        hd = B.ensemble_record(system, method, y0[:, :n].contiguous(), p[:, :n].contiguous(),
                               0.0, t1, rtol, atol, save_times=times, pool=pool,
                               steps_per_traj=hint, ckpt_every=ckpt)
        gp, gy, ll = B.ensemble_adjoint(hd)
        got = [hd.y_save, hd.steps(), hd.n_trial(), hd.status, gp, gy, ll]
        got = [g.clone() for g in got]
        assert int(hd.status.abs().max()) == 0
        if ref is None:
            ref = got
            if hint == 16:
                assert int(hd.steps().max()) > hint
            continue
        for a, b in zip(got, ref):
            assert torch.equal(a, b[..., :n])

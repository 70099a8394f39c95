"""Where a record's steps go when the reserved pages run out: no reserved page
at all, one, and enough, must give the same steps, states and gradients bit
for bit, for the records that write at once (small ensembles) and those that
stage lines (large ones), full and checkpointed, and for given meshes; and a
pool without room ends exactly the trajectories that found none.
"""
import pytest
import torch

from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu


def inputs(system, n, dtype=torch.float64):
    return (torch.tensor(a.T.copy(), dtype=dtype, device="cuda")
            for a in W.GENERATORS[system](n, 7))


def outputs(hd, loss="sumsq"):
    gp, gy, ll = B.ensemble_adjoint(hd, loss)
    return [t.clone() for t in (hd.y_save, hd.steps(), hd.n_trial(), hd.status, gp, gy, ll)]


@pytest.mark.parametrize("system,method,n,ckpt,t1", [
    ("lorenz", "tsit5", 65, 0, 0.05), ("lorenz", "tsit5", 65600, 0, 0.05),
    ("lorenz", "vern7", 300, 16, 0.05), ("lorenz", "vern7", 65600, 16, 0.05),
    ("robertson", "ros23", 300, 0, 1e-4), ("robertson", "rodas4", 65600, 0, 1e-4)])
def test_any_reserve(system, method, n, ckpt, t1):
    print(f"case {system} {method} {n} ckpt {ckpt}", flush=True)
    y0, p = inputs(system, n)
    times = [0.3 * t1, t1]
    args = (system, method, y0, p, 0.0, t1, 1e-6, 1e-10)
    full = B.ensemble_record(*args, save_times=times, steps_hint=64, ckpt_every=ckpt)
    ref = outputs(full)
    assert int(full.status.abs().max()) == 0 and 1 <= int(full.steps().max()) <= 16
    # no reserved page: the whole tape in the overflow area, a page each
    fixed = full.rec.links - full.pool.data_ptr()
    pool = torch.empty(fixed + 512 + int(1.05 * n * (full.rec.page_bytes + 8)),
                       dtype=torch.uint8, device="cuda")
    none = B.ensemble_record(*args, save_times=times, pool=pool, ckpt_every=ckpt)
    assert none.rec.static_pages == 0
    for a, b in zip(outputs(none), ref):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,ckpt", [(65, 0), (65600, 0), (300, 16), (65600, 16)])
def test_one_page_then_overflow(n, ckpt):
    print(f"case {n} ckpt {ckpt}", flush=True)
    y0, p = inputs("lorenz", n)
    args = ("lorenz", "tsit5", y0, p, 0.0, 2.0, 1e-6, 1e-8)
    pool = torch.empty(2 << 30, dtype=torch.uint8, device="cuda")
    full = B.ensemble_record(*args, pool=pool, steps_per_traj=256, ckpt_every=ckpt)
    ref = outputs(full)
    h, S = (t.clone() for t in B.ensemble_mesh_export(full))
    one = B.ensemble_record(*args, pool=pool, steps_per_traj=16, ckpt_every=ckpt)
    assert one.rec.static_pages == 1 and int(one.steps().max()) > 32
    for a, b in zip(outputs(one), ref):
        assert torch.equal(a, b)
    h2, S2 = B.ensemble_mesh_export(one)
    assert torch.equal(S2, S) and torch.equal(h2, h)
    rep = B.ensemble_replay_mesh("lorenz", "tsit5", y0, p, 0.0, 2.0, h, S, pool=pool,
                                 steps_per_traj=16, ckpt_every=ckpt)
    got = outputs(rep)
    for k in (0, 1, 4, 5, 6):      # all but the trial counts and status
        assert torch.equal(got[k], ref[k])


def test_no_room_left():
    n = 300
    y0, p = inputs("lorenz", n)
    args = ("lorenz", "tsit5", y0, p, 0.0, 2.0, 1e-6, 1e-8)
    full = B.ensemble_record(*args, steps_hint=256)
    S = full.steps().clone()
    pages = (S + 15) // 16
    extra = int((pages - 1).sum()) - 10          # ten overflow pages too few
    fixed = full.rec.links - full.pool.data_ptr()
    pool = torch.empty(fixed + 512 + n * full.rec.page_bytes +
                       extra * (full.rec.page_bytes + 8), dtype=torch.uint8, device="cuda")
    hd = B.ensemble_record(*args, pool=pool, steps_per_traj=16)
    short = hd.status == 4
    assert 0 < int(short.sum()) <= 10
    assert torch.equal(hd.steps()[~short], S[~short])
    assert bool((hd.steps()[short] % 16 == 0).all())
    assert bool(hd.y_save[:, :, short].isnan().all())

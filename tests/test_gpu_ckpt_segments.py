"""Checkpointed sweep: the replayed records of a block side by side in the
scratch, at ragged and single-trajectory blocks, with trajectories of different
segment counts and failed ones between them, every record size (16 bytes, 32,
80).  Per-trajectory results against the full tape's, bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2609_02876_amd import binding as B
from paper_2609_02876_amd import workloads as W

pytestmark = pytest.mark.gpu


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=12345.0), torch.nan_to_num(b, nan=12345.0)) and \
        torch.equal(torch.isnan(a), torch.isnan(b))


@pytest.mark.parametrize("n", [1, 63, 255, 257, 300])
@pytest.mark.parametrize("system,method,dtype,t1,K", [
    ("lorenz", "tsit5", torch.float64, 3.0, 16), ("lorenz", "vern7", torch.float64, 5.0, 64),
    ("vdp", "tsit5", torch.float32, 6.3, 32), ("robertson", "rodas4", torch.float64, 1e5, 64),
    ("hires", "rodas4", torch.float64, 100.0, 32)])
def test_segments_equal_full_tape(system, method, dtype, t1, K, n):
    print(f"case {system} {method} n={n} K={K}", flush=True)
    y0, p = W.GENERATORS[system](n, 11)
    y0 = y0.copy()
    p = p.copy()
    if system == "lorenz":   # step counts from about one segment to several
        p[:, 1] = np.linspace(2.0, 60.0, n)
    if n > 5:
        y0[5, 0] = np.nan    # a failed trajectory among the block's
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), dtype=dtype, device="cuda")
    st = [0.0, 0.3 * t1, 0.3 * t1, 0.77 * t1, t1]
    got = []
    for ck in (0, K):
        hd = B.ensemble_record(system, method, dev(y0), dev(p), 0.0, t1, 1e-6, 1e-9,
                               save_times=st, steps_hint=512, ckpt_every=ck)
        got.append(B.ensemble_adjoint(hd) + (hd.y_save, hd.status))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert _same(a, b)
    assert int((got[0][-1] != 0).sum()) == (1 if n > 5 else 0)

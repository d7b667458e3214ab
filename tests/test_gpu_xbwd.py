"""The reverse loop in one group of workgroups per XCD (xbwd_kernel.h), at the
sizes where it can go wrong: the edges of each variant's padded 4H and of its
16 units per workgroup, and batches that leave groups empty, with one row, a
full row tile, a second one, and just past what the groups hold.  Every
gradient of each cell against the fp64 oracle, scaled as in test_gpu_bwd, at
its tolerances; a second run gives the same bits."""
import numpy as np
import pytest

import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import say, to_device
from tests.test_gpu_bwd import GRAD_TOL, compare, oracle_grads, upstream
from tests.test_gpu_bwd_cells import oracle_grads as cell_oracle
from tests.test_gpu_cells import gru_device

pytestmark = pytest.mark.gpu

CASES = [
    ("f32", 15, 9, "lstm"), ("f32", 128, 1, "gru"), ("f32", 129, 8, "rnn"), ("f32", 256, 129, "lstm"),
    ("f32", 257, 128, "gru"), ("f32", 511, 33, "lstm"), ("f32", 512, 256, "rnn"), ("f32", 200, 257, "lstm"),
    ("bf16", 17, 5, "lstm"), ("bf16", 128, 256, "rnn"), ("bf16", 129, 16, "lstm"), ("bf16", 256, 140, "gru"),
    ("bf16", 257, 64, "lstm"), ("bf16", 512, 128, "lstm"), ("bf16", 513, 3, "gru"), ("bf16", 1000, 130, "lstm"),
    ("bf16", 1024, 70, "rnn"), ("bf16", 1025, 20, "lstm"),
]


@pytest.mark.parametrize("dt,H,B,cell", CASES)
def test_edges(dt, H, B, cell):
    import torch
    D, T = 20, 9
    say(f"case xbwd {dt} H={H} B={B} {cell}")
    dh, dc, ds = upstream(6300 + H, B, H, T)
    if cell == "lstm":
        inp = workloads.random_case(6400 + H + B, B, D, H, T, dtype=dt)
        dev = to_device(inp)
        go = oracle_grads(inp, dh.astype(np.float64), dc.astype(np.float64), ds.astype(np.float64))
        keys = ("dx", "dW", "dU", "db", "dh0", "dc0")
    else:
        inp = workloads.random_cell_case(cell, 6400 + H + B, B, D, H, T, dtype=dt)
        dev = (*gru_device(inp), None)
        go = cell_oracle(inp, dh, ds)
        keys = ("dx", "dW", "dU", "db", "dh0")
    t = lambda a: torch.from_numpy(a).cuda()
    m = ld.LstmDyn(B, D, H, T, dt, "persistent", cell=cell)
    runs = []
    for _ in range(2):
        m.forward_train(*dev)
        runs.append(m.backward(*dev, t(dh), t(dc) if cell == "lstm" else None, t(ds)))
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    compare({k: runs[0][k].cpu().numpy().astype(np.float64) for k in keys}, go, GRAD_TOL[dt], keys=keys)
    for k in keys:
        assert torch.equal(runs[0][k], runs[1][k]), k
    m.close()

"""fp32 loops with at most four rows per group (products of four rows, loop.h): the
batches on both sides of that line (32 and 33 rows with eight groups), with one row,
groups of one row beside groups of none, at every variant's width, rows that end
one by one.  Final state, sequence and every gradient against the fp64 oracle at
the forward's and the backward's fp32 tolerances; the forward for training and
the loop with termination against the plain forward bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import max_err, say, to_device
from tests.test_gpu_bwd import GRAD_TOL, compare, oracle_grads, upstream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,B", [(33, 1), (64, 5), (65, 31), (128, 32), (129, 33), (256, 32), (255, 4), (257, 8),
                                 (384, 30), (385, 32), (512, 25), (385, 16), (400, 3), (512, 1), (511, 9), (512, 16)])
def test_edges(H, B):
    import torch
    D, T = 12, 10
    say(f"case few rows H={H} B={B}")
    inp = workloads.random_case(6700 + H + B, B, D, H, T, dtype="f32")
    inp.lengths[:] = np.random.default_rng(H).permutation(np.linspace(0, T, B).round().astype(np.int32))
    dev = to_device(inp)
    m = ld.LstmDyn(B, D, H, T, "f32", "persistent")
    h, c, seq = m.forward_seq(*dev)
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    ho, co, so = oracle.forward_inputs(inp, seq=True)
    assert max(max_err(a.cpu().numpy(), o) for a, o in ((h, ho), (c, co), (seq, so))) <= 1e-5
    h2, c2, steps = m.forward_stop(*dev, torch.zeros(H, device="cuda"), -1.0)
    dh, dc, ds = upstream(6800 + H, B, H, T)
    t = lambda a: torch.from_numpy(a).cuda()
    h3, c3, seq3 = m.forward_train(*dev, with_seq=True)
    g = m.backward(*dev, t(dh), t(dc), t(ds))
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    for a, b in ((h2, h), (c2, c), (h3, h), (c3, c), (seq3, seq)):
        assert torch.equal(a, b)
    assert np.array_equal(steps.cpu().numpy(), inp.lengths)
    go = oracle_grads(inp, dh.astype(np.float64), dc.astype(np.float64), ds.astype(np.float64))
    compare({k: g[k].cpu().numpy().astype(np.float64) for k in go}, go, GRAD_TOL["f32"], keys=tuple(go))
    m.close()

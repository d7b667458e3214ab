"""The passes around the backward's GEMMs (bwd.hip: operands side by side, column
sums, gradients to the caller's layout) at the widths where they branch: D and
H no multiples of 4, x not aligned to a whole vector, more than one workgroup of
db, more rows than one workgroup takes, no row at all.  Gradients against the
fp64 oracle, scaled as in test_gpu_bwd, at its tolerances."""
import numpy as np
import pytest

import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import say, to_device
from tests.test_gpu_bwd import GRAD_TOL, compare, oracle_grads, upstream
from tests.test_gpu_bwd_cells import oracle_grads as cell_oracle
from tests.test_gpu_cells import gru_device

pytestmark = pytest.mark.gpu

CASES = [  # dt, D, H, B, T, cell, x shifted by 4 bytes
    ("f32", 1, 5, 2, 3, "lstm", False), ("f32", 8, 260, 5, 7, "gru", True), ("f32", 12, 300, 3, 40, "lstm", False),
    ("f32", 7, 64, 33, 5, "rnn", False), ("bf16", 3, 17, 4, 6, "lstm", False), ("bf16", 4, 18, 5, 9, "gru", False),
    ("bf16", 12, 260, 3, 30, "lstm", True), ("bf16", 8, 513, 2, 4, "rnn", False), ("bf16", 64, 40, 96, 33, "lstm", False),
    ("bf16", 2, 1536, 3, 5, "lstm", False),
]


@pytest.mark.parametrize("dt,D,H,B,T,cell,shift", CASES)
def test_widths(dt, D, H, B, T, cell, shift):
    import torch
    say(f"case operands {dt} D={D} H={H} B={B} T={T} {cell} shift={shift}")
    dh, dc, ds = upstream(7100 + H, B, H, T)
    lstm = cell == "lstm"
    if lstm:
        inp = workloads.random_case(7200 + H + B, B, D, H, T, dtype=dt)
        dev = list(to_device(inp))
        go = oracle_grads(inp, dh.astype(np.float64), dc.astype(np.float64), ds.astype(np.float64))
    else:
        inp = workloads.random_cell_case(cell, 7200 + H + B, B, D, H, T, dtype=dt)
        dev = [*gru_device(inp), None]
        go = cell_oracle(inp, dh, ds)
    bwd = list(dev)  # the forward's x is 16-byte aligned, the backward's need not be
    if shift:
        x = dev[0]
        n = 4 // x.element_size()
        buf = torch.empty(x.numel() + n, dtype=x.dtype, device=x.device)
        bwd[0] = buf[n:].view(x.shape)
        bwd[0].copy_(x)
    keys = ("dx", "dW", "dU", "db", "dh0") + (("dc0",) if lstm else ())
    t = lambda a: torch.from_numpy(a).cuda()
    m = ld.LstmDyn(B, D, H, T, dt, "persistent", cell=cell)
    m.forward_train(*dev)
    g = m.backward(*bwd, t(dh), t(dc) if lstm else None, t(ds))
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    compare({k: g[k].cpu().numpy().astype(np.float64) for k in keys}, go, GRAD_TOL[dt], keys=keys)
    # no row runs a step: the weights' gradients are zero, the state's its own
    dev[1] = bwd[1] = torch.zeros_like(dev[1])
    m.forward_train(*dev)
    g = m.backward(*bwd, t(dh), t(dc) if lstm else None, t(ds))
    torch.cuda.synchronize()
    for k in ("dx", "dW", "dU", "db"):
        assert not g[k].any(), k
    assert torch.equal(g["dh0"], t(dh))
    m.close()


@pytest.mark.parametrize("dt,H", [("f32", 40), ("bf16", 200)])
def test_rows_of_this_call(dt, H):
    """The GEMMs take as many rows as this forward kept, which a kernel hands to the
    host while the reverse loop runs: batches of very different sums of lengths,
    one after another on one handle, give what a fresh handle gives, bit for bit."""
    import torch
    B, D, T = 24, 12, 60
    say(f"case rows of this call {dt} H={H}")
    dh, dc, _ = upstream(7300 + H, B, H, T)
    t = lambda a: torch.from_numpy(a).cuda()
    m = ld.LstmDyn(B, D, H, T, dt, "persistent")
    for k, hi in enumerate((T, 1, 30, 0, T, 2)):
        dev = to_device(workloads.random_case(7310 + k, B, D, H, T, dtype=dt, lo=hi // 2, hi=hi))
        m.forward_train(*dev)
        g = m.backward(*dev, t(dh), t(dc))
        f = ld.LstmDyn(B, D, H, T, dt, "persistent")
        f.forward_train(*dev)
        g2 = f.backward(*dev, t(dh), t(dc))
        torch.cuda.synchronize()
        for n in g:
            assert torch.equal(g[n], g2[n]), (k, n)
        f.close()
    m.close()

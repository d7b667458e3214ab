"""The one-workgroup forward (small.hip; H <= 32) at the edges of its variants (D, B)
and of its look-ahead in x: one to five steps, rows that end early, sequence and
termination.  Against the fp64 oracle at the forward's tolerances (1e-5 with
fp32 data, 3e-3 with bf16 data)."""
import numpy as np
import pytest

import oracle
import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import max_err, say, to_device

pytestmark = pytest.mark.gpu

TOL = {workloads.F32: 1e-5, workloads.BF16: 3e-3}


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("dt,B,D,H", [("f32", 16, 16, 32), ("f32", 17, 17, 31), ("f32", 64, 64, 5), ("f32", 1, 33, 32),
                                      ("bf16", 16, 32, 32), ("bf16", 64, 128, 32), ("bf16", 2, 33, 7)])
def test_edges(dt, B, D, H, T):
    import torch
    say(f"case small {dt} B={B} D={D} H={H} T={T}")
    inp = workloads.random_case(9100 + B + D + T, B, D, H, T, dtype=dt)
    m = ld.LstmDyn(B, D, H, T, dt, "persistent")
    dev = to_device(inp)
    h, c, seq = m.forward_seq(*dev)
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    ho, co, so = oracle.forward_inputs(inp, seq=True)
    assert max(max_err(a.cpu().numpy(), o) for a, o in ((h, ho), (c, co), (seq, so))) <= TOL[dt]
    h2, c2, steps = m.forward_stop(*dev, torch.zeros(H, device="cuda"), -1.0)
    torch.cuda.synchronize()
    assert torch.equal(h, h2) and torch.equal(c, c2)
    assert np.array_equal(steps.cpu().numpy(), inp.lengths)
    assert m.query(ld.Q_STEPS_EXECUTED) == int(inp.lengths.max())
    m.close()


@pytest.mark.parametrize("dt,D", [("f32", 64), ("bf16", 128)])
def test_x_is_gathered_once(dt, D):
    """A step of 64 rows waits for the gathers of x: 12 us with four waves that
    each take all of it (fp32; bf16 17), 17 and 29 with eight, 5.2 where the
    workgroup takes it once; the bound lies between."""
    T = 200
    say(f"case small step time {dt} D={D}")
    inp = workloads.random_case(9300 + D, 64, D, 32, T, dtype=dt, lo=T)
    m = ld.LstmDyn(64, D, 32, T, dt, "persistent")
    m.set_option(ld.OPT_TIMING, 1)
    dev = to_device(inp)
    times = []
    for _ in range(5):
        m.forward(*dev)
        times.append(m.query(ld.Q_TIME_LOOP_NS) / T / 1e3)
    say("  us a step: " + " ".join(f"{t:.2f}" for t in times))
    assert min(times) <= 9.0
    m.close()

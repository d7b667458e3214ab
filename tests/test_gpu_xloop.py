"""The loop in one group of workgroups per XCD (xloop_kernel.h), at the sizes
where it can go wrong: the edges of each variant's hidden width (one unit
below, at and above the padded K), batches that leave groups empty, with one
row, with a full row tile, with a second one, and just past what the groups
hold (the device-wide loop).  The final state and the output sequence against
the fp64 oracle at the forward's tolerances (1e-5 with fp32 data, 3e-3 with
bf16 data), the forward for training and the halting read-out against the
plain forward bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import max_err, say, to_device

pytestmark = pytest.mark.gpu

TOL = {workloads.F32: 1e-5, workloads.BF16: 3e-3}

CASES = [(dt, H, B) for dt, widths in (("f32", (63, 65, 128, 129, 256, 257, 384, 385, 512, 513)),
                                       ("bf16", (36, 128, 129, 257, 384, 511, 513, 768, 769, 1024, 1025)))
         for H, B in zip(widths, (5, 9, 1, 129, 8, 128, 33, 256, 17, 64, 140))] + [
    ("f32", 100, 257), ("bf16", 600, 256), ("bf16", 1022, 131), ("bf16", 1000, 2)]


@pytest.mark.parametrize("dt,H,B", CASES)
def test_edges(dt, H, B):
    import torch
    D, T = 24, 7
    inp = workloads.random_case(6100 + H + B, B, D, H, T, dtype=dt)
    say(f"case xloop {dt} H={H} B={B}")
    m = ld.LstmDyn(B, D, H, T, dt, "persistent")
    dev = to_device(inp)
    h, c, seq = m.forward_seq(*dev)
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    ho, co, so = oracle.forward_inputs(inp, seq=True)
    errs = [max_err(a.cpu().numpy(), o) for a, o in ((h, ho), (c, co), (seq, so))]
    say("  max errors h, c, seq: " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) <= TOL[dt]
    h2, c2, seq2 = m.forward_train(*dev, with_seq=True)
    v = torch.zeros(H, device="cuda")
    h3, c3, steps = m.forward_stop(*dev, v, -1.0)
    torch.cuda.synchronize()
    assert m.query(ld.Q_STEPS_EXECUTED) == int(inp.lengths.max())
    for a, b in ((h2, h), (c2, c), (seq2, seq), (h3, h), (c3, c)):
        assert torch.equal(a, b)
    assert np.array_equal(steps.cpu().numpy(), inp.lengths)
    m.close()


@pytest.mark.parametrize("T", [16, 252])
def test_noalloc_with_and_without_room_for_packed_u(T):
    """The allocation-free forward leaves the packed copy of U out where its
    scratch has no room for it (T = 252) and then reads U itself: the same bits
    as the handle's forward either way."""
    import torch
    B, D, H = 64, 32, 512
    inp = workloads.random_case(6200, B, D, H, T, dtype="bf16", hi=20 if T > 20 else T)
    dev = to_device(inp)
    m = ld.LstmDyn(B, D, H, T, "bf16", "persistent")
    h, c = m.forward(*dev)
    oh, oc = torch.empty_like(h), torch.empty_like(c)
    st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    say(f"case xloop noalloc T={T}")
    ld.lstm_dyn_forward_noalloc(B, D, H, T, ld.BF16, *(t.data_ptr() for t in dev), oh.data_ptr(),
                                oc.data_ptr(), st.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert int(st[0]) == ld.OK
    assert torch.equal(h, oh) and torch.equal(c, oc)
    m.close()


@pytest.mark.parametrize("dt,H,B", [("bf16", 512, 256), ("f32", 130, 200), ("bf16", 800, 256)])
def test_rows_ending_in_later_tiles(dt, H, B):
    """Rows end one by one while a group has two row tiles, forward and back: a
    lane whose row has ended must not wait for a row of another tile, whose
    slot other workgroups may already have marked for a later step."""
    import torch
    D, T = 16, 300
    inp = workloads.random_case(6500 + H, B, D, H, T, dtype=dt)
    inp.lengths[:] = np.maximum(T - np.arange(B), 1)
    m = ld.LstmDyn(B, D, H, T, dt, "persistent")
    m.set_option(ld.OPT_TIMEOUT_US, 200000)
    dev = to_device(inp)
    say(f"case xloop rows ending {dt} H={H} B={B}")
    h, c = m.forward(*dev)
    dh = torch.ones(B, H, device="cuda")
    m.forward_train(*dev)
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    m.backward(*dev, dh, dh)
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    rows = [0, 17, B // 2, B - 1]
    sub = workloads.Inputs(x=inp.x[rows], lengths=inp.lengths[rows], W=inp.W, U=inp.U, b=inp.b, h0=inp.h0[rows],
                           c0=inp.c0[rows], dtype=inp.dtype)
    ho, co = oracle.forward_inputs(sub)
    assert max_err(h.cpu().numpy()[rows], ho) <= TOL[dt] and max_err(c.cpu().numpy()[rows], co) <= TOL[dt]
    m.close()

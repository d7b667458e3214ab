"""Which loop a size takes (LSTM_DYN_Q_LAST_LOOP), forward and back, on both sides
of each line of the dispatch, and the number of workgroups that its launch has
(LSTM_DYN_Q_GROUPS)."""
import numpy as np
import pytest

import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import say, to_device

pytestmark = pytest.mark.gpu

G, D_, S, SG, RG, RB, RF, RS = (ld.LOOP_GROUPED, ld.LOOP_DEVICE, ld.LOOP_STEPS, ld.LOOP_SINGLE, ld.LOOP_REVERSE_GROUPED,
                                ld.LOOP_REVERSE_BLOCKS, ld.LOOP_REVERSE_FEW, ld.LOOP_REVERSE_STEPS)

CASES = [  # dt, B, H, mode: forward, workgroups, forward for training, backward
    ("f32", 64, 32, "persistent", SG, 1, S, RG), ("f32", 65, 32, "persistent", G, 8 * 8, G, RG),
    ("f32", 8, 256, "persistent", G, 32 * 8, G, RG), ("f32", 256, 512, "persistent", G, 32 * 8, G, RG),
    ("f32", 1, 512, "persistent", G, 32 * 8, G, RG), ("f32", 16, 385, "persistent", G, 25 * 8, G, RG),
    ("f32", 257, 512, "persistent", D_, 128, D_, RS), ("f32", 17, 513, "persistent", D_, 129, D_, RS),
    ("f32", 5, 64, "per_step", S, 16, S, RS),
    ("bf16", 37, 100, "persistent", G, 25 * 8, G, RG), ("bf16", 257, 512, "persistent", D_, 128, D_, RB),
    ("bf16", 257, 300, "persistent", D_, 75, D_, RF), ("bf16", 20, 768, "persistent", G, 32 * 8, G, RG),
    ("bf16", 257, 768, "persistent", D_, 192, D_, RF), ("bf16", 20, 1023, "persistent", G, 32 * 8, G, RG),
    ("bf16", 20, 1024, "persistent", G, 32 * 8, G, RB), ("bf16", 20, 1026, "persistent", D_, 129, D_, RF),
    ("bf16", 20, 1025, "persistent", D_, 129, D_, RS), ("bf16", 20, 1280, "persistent", D_, 160, D_, RF),
    ("bf16", 20, 2048, "persistent", D_, 256, D_, RB), ("bf16", 9, 200, "per_step", S, 50, S, RS),
]


@pytest.mark.parametrize("dt,B,H,mode,fwd,groups,train,bwd", CASES)
def test_loop_of_size(dt, B, H, mode, fwd, groups, train, bwd):
    import torch
    say(f"case loop {dt} B={B} H={H} {mode}")
    inp = workloads.random_case(9500 + B + H, B, 8, H, 3, dtype=dt)
    inp.lengths[:] = np.where(np.arange(B) < 16, 3, 2)  # the last step has at most 16 rows
    dev = to_device(inp)
    m = ld.LstmDyn(B, 8, H, 3, dt, mode)
    assert m.query(ld.Q_LAST_LOOP) == 0
    m.forward(*dev)
    assert (m.query(ld.Q_LAST_LOOP), m.query(ld.Q_GROUPS)) == (fwd, groups)
    m.forward_stop(*dev, torch.zeros(H, device="cuda"), -1.0)
    assert m.query(ld.Q_LAST_LOOP) == fwd
    m.forward_train(*dev)
    assert m.query(ld.Q_LAST_LOOP) == train
    d = torch.ones(B, H, device="cuda")
    m.backward(*dev, d, d)
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    assert m.query(ld.Q_LAST_LOOP) == bwd
    m.close()


@pytest.mark.parametrize("dt,B,D,H,T", [("bf16", 20, 24, 1000, 3), ("bf16", 64, 40, 512, 5), ("f32", 9, 30, 500, 3),
                                        ("f32", 64, 16, 32, 4)])
def test_training_workspace(dt, B, D, H, T):
    """A handle with the grouped reverse loop reserves for training what it uses:
    the kept states and rows, the GEMMs' operands and results, the column sums,
    U packed, the exchange of dz; no operands of a product per step."""
    say(f"case training workspace {dt} B={B} D={D} H={H} T={T}")
    dev = to_device(workloads.random_case(9700 + H, B, D, H, T, dtype=dt))
    m = ld.LstmDyn(B, D, H, T, dt, "persistent")
    before = m.query(ld.Q_WORKSPACE_BYTES)
    m.forward_train(*dev)
    got = m.query(ld.Q_WORKSPACE_BYTES) - before
    e = 2 if dt == "bf16" else 4
    rows, slots = B * T, -(-B // 8) * 8
    need = 8 * rows * H + 4 * rows * D + 16 * (D + H) * H + 16 * D * H * e // 4 + 64 * 16 * H   # states, dx, dW dU, W, sums
    if dt == "bf16":
        need += 2 * rows * (D + 5 * H)                                    # dz, x and h in fp16
    pad = next(w for w in (512, 1024, 2048, 4096) if w >= 4 * H)          # 4H as the compiled variants pad it
    need += e * (H + 32) * pad + 4 * e * slots * pad + 4 * H              # U packed, dz exchanged, U's scales
    if dt == "bf16":
        need += 8 * slots * (pad // 32)
    if H <= 32:
        need += 16 * H * (-(-B // 16) * 16)                               # pre-activations of a step
    need += 24 * 256                                                      # each array starts at a multiple of 256 bytes
    say(f"  {got} bytes, at most {need} used")
    assert got <= need
    m.close()


@pytest.mark.parametrize("dt,H", [("bf16", 512), ("f32", 256)])
def test_two_handles_on_two_streams(dt, H):
    """Two handles whose launches each take every CU, forward and back on streams of
    their own without a wait between them: each gives what it gives alone."""
    import torch
    B, D, T = 40, 32, 50
    say(f"case two streams {dt} H={H}")
    d = torch.ones(B, H, device="cuda")
    dev = [to_device(workloads.random_case(9800 + k, B, D, H, T, dtype=dt)) for k in range(2)]
    ms = [ld.LstmDyn(B, D, H, T, dt, "persistent") for _ in range(2)]
    alone = []
    for m, a in zip(ms, dev):
        m.set_option(ld.OPT_TIMEOUT_US, 500000)
        h, c = m.forward(*a)
        m.forward_train(*a)
        alone.append({"h": h, "c": c, **m.backward(*a, d, d)})
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = [None, None]
    for rep in range(5):
        for k in (0, 1):
            with torch.cuda.stream(streams[k]):
                h, c = ms[k].forward(*dev[k])
                ms[k].forward_train(*dev[k])
                got[k] = {"h": h, "c": c, **ms[k].backward(*dev[k], d, d)}
        torch.cuda.synchronize()
        for k in (0, 1):
            assert ms[k].query(ld.Q_LAST_STATUS) == ld.OK
            for n in alone[k]:
                assert torch.equal(got[k][n], alone[k][n]), (rep, k, n)
    for m in ms:
        m.close()

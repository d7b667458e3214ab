"""Performance cases of the variable-length recurrent loop: what is timed, on
which inputs, and how exact the results have to be.

A case is a dict of plain values:
  op       "forward" (final state), "seq" (and the output sequence), "stop"
           (rows end on a halting read-out of their state) or "train" (the
           forward for training, then the backward)
  cell     "lstm", "gru" or "rnn"
  dtype    "f32" or "bf16" (x, W and U; state, biases and gradients are fp32)
  B D H T  batch rows, input width, hidden width, padded number of steps
  lengths  how long the rows are: "full", "uniform", "geometric" or "lognormal"
  dseq     op "train": the loss also takes a gradient of the output sequence

prepare() makes the handle a program keeps for its shape, the weights and one
batch; run() is one call (op "train": two) of the LstmDyn class.
"""
import math

import torch

from paper_1810_08061_amd import LstmDyn

_GATES = {"lstm": 4, "gru": 3, "rnn": 1}   # columns of W and U per hidden unit
_BIAS = {"lstm": 4, "gru": 6, "rnn": 1}    # bias entries per hidden unit


def _case(name, op, cell, dtype, B, D, H, T, lengths, dseq=False):
    c = {"op": op, "cell": cell, "dtype": dtype, "B": B, "D": D, "H": H, "T": T,
         "lengths": lengths, "dseq": dseq}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a few short sequences through a narrow layer, where
        # launches, the host's work and one step's latency are all there is
        _case("tiny_f32", "forward", "lstm", "f32", 4, 16, 32, 20, "uniform"),
        # an ordinary fp32 layer: classify a small ragged batch from its final state
        _case("lstm256_f32", "forward", "lstm", "f32", 32, 256, 256, 100, "uniform"),
        # the paper's RNN benchmark (hidden 256, batch 128, 128 steps, outputs kept)
        _case("paper256_seq_f32", "seq", "lstm", "f32", 128, 64, 256, 128, "full"),
        # an ordinary bf16 layer: encode a ragged batch
        _case("lstm512_bf16", "forward", "lstm", "bf16", 64, 512, 512, 200, "uniform"),
        # serving traffic: most requests short, a few very long ones
        _case("skewed1024_bf16", "forward", "lstm", "bf16", 128, 1024, 1024, 500, "geometric"),
        # the largest: a wide layer over a large batch of long documents
        _case("large2048_bf16", "forward", "lstm", "bf16", 256, 1024, 2048, 1000, "lognormal"),
        # a decoder loop that leaves on the device once every row has ended
        _case("stop1024_bf16", "stop", "lstm", "bf16", 64, 512, 1024, 256, "uniform"),
        # another cell at sizes that are no multiple of any tile, outputs kept
        _case("gru750_seq_bf16", "seq", "gru", "bf16", 37, 200, 750, 61, "uniform"),
        # training steps: fp32 ...
        _case("train256_f32", "train", "lstm", "f32", 32, 256, 256, 100, "uniform"),
        # ... fp32 at odd sizes, another cell, a loss on every output ...
        _case("train333_rnn_f32", "train", "rnn", "f32", 21, 77, 333, 45, "uniform", True),
        # ... bf16, a loss on every output ...
        _case("train512_bf16", "train", "lstm", "bf16", 64, 512, 512, 200, "uniform", True),
        # ... and the largest
        _case("train2048_bf16", "train", "lstm", "bf16", 256, 1024, 2048, 1000, "lognormal"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        op = rng.choice(["forward", "forward", "seq", "stop", "train", "train"])
        cell = rng.choice(["lstm", "lstm", "gru", "rnn"])
        dtype = rng.choice(["f32", "bf16"])
        B, D, T = log(1, 256), log(16, 1024), log(8, 1000)
        H = log(24, 1024 if dtype == "f32" else 2048)
        if rng.random() < 0.5:   # half the layers have widths programs like to choose
            D = max(16, (D + 8) // 16 * 16)
            H = max(32, (H + 32) // 64 * 64)
        c = _case(None, op, cell, dtype, B, D, H, T,
                  rng.choice(["full", "uniform", "geometric", "lognormal"]), rng.random() < 0.5)
        if op != "train":
            c["dseq"] = False
        w, top = work(c), work(listed()[-1])
        # (fp32 operations run at a sixteenth of the bf16 rate)
        if w["flops"] * (16 if dtype == "f32" else 1) <= top["flops"] and w["bytes"] <= top["bytes"]:
            return c


def _length(case, u):
    """A row's length from u in (0, 1), a tensor of fp64."""
    T, kind = case["T"], case["lengths"]
    if kind == "full":
        L = torch.full_like(u, T)
    elif kind == "uniform":          # 0 to T
        L = torch.floor(u * (T + 1))
    elif kind == "geometric":        # mean T / 12, at least one step
        L = torch.ceil(torch.log1p(-u) / math.log1p(-min(0.9, 12.0 / T)))
    else:                            # lognormal about T / 7, as document lengths are
        L = torch.round(torch.exp(math.log(max(1.0, T * 0.148)) + 0.8 * math.sqrt(2.0) * torch.erfinv(2 * u - 1)))
        L = torch.clamp(L, min=1)
    return torch.clamp(L, 0, T)


def _longest(case):
    """Batches of skewed lengths hold one row of the full length."""
    return case["lengths"] in ("geometric", "lognormal")


def _batch(case, seed):
    """Inputs in the library's layouts, on the GPU."""
    B, D, H, T, cell = case["B"], case["D"], case["H"], case["T"], case["cell"]
    g, nb = _GATES[cell], _BIAS[cell]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    et = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(*shape, std=1.0, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype).mul_(std)

    u = torch.rand((B,), generator=gen, device="cuda", dtype=torch.float64).clamp_(1e-9, 1 - 1e-9)
    L = _length(case, u).to(torch.int32)
    if _longest(case):
        L[0] = T
    # the plain tanh recurrence is initialised as torch.nn.RNN is (variance 1 / 3H)
    std = 1.0 / math.sqrt(3 * H if cell == "rnn" else H)
    s = {"x": normal(B, T, D, dtype=et), "lengths": L,
         "W": normal(D, g * H, std=std).to(et), "U": normal(H, g * H, std=std).to(et)}
    if cell == "lstm":
        b = torch.zeros(4 * H, device="cuda")
        b[H:2 * H] = 1.0
    else:
        b = normal(nb * H, std=math.sqrt(0.1))
    s["b"] = b
    s["h0"] = normal(B, H, std=math.sqrt(0.1))
    s["c0"] = normal(B, H, std=math.sqrt(0.1)) if cell == "lstm" else None
    if case["op"] == "stop":
        # An end marker in feature 0 of x (-1, then +1 at a row's last step for
        # seven rows of ten) drives hidden unit 0, which the read-out looks at;
        # the other units move the score a little.
        x, W, U = s["x"], s["W"], s["U"]
        W[0] = 0
        W[:, 0::H] = 0
        U[:, 0::H] = 0
        if cell == "lstm":
            W[0, 2 * H] = 4.0
            b[0], b[H], b[3 * H] = 6.0, -6.0, 6.0
        elif cell == "gru":
            W[0, 2 * H] = 4.0
            b[0::H] = 0.0
            b[H] = -8.0
        else:
            W[0, 0] = 4.0
            b[0] = 0.0
        x[:, :, 0] = -1.0
        end = torch.floor(torch.rand((B,), generator=gen, device="cuda") * L).long()
        some = torch.rand((B,), generator=gen, device="cuda") < 0.7
        rows = torch.arange(B, device="cuda")
        x[rows, end.clamp(0, T - 1), 0] = torch.where(some, 1.0, -1.0).to(et)
        v = normal(H, std=0.1 / math.sqrt(H))
        v[0] = 2.0
        s["stop_v"], s["stop_c"] = v, -0.5
    if case["op"] == "train":
        s["d_out_h"] = normal(B, H)
        s["d_out_c"] = normal(B, H) if cell == "lstm" else None
        s["d_seq"] = normal(B, T, H) if case["dseq"] else None
    return s


def prepare(case, seed):
    s = _batch(case, seed)
    s["op"] = case["op"]
    s["model"] = LstmDyn(case["B"], case["D"], case["H"], case["T"], case["dtype"], "persistent",
                         case["cell"])
    return s


def run(s):
    m, op = s["model"], s["op"]
    a = (s["x"], s["lengths"], s["W"], s["U"], s["b"], s["h0"], s["c0"])
    if op == "forward":
        h, c = m.forward(*a)
        return {"h": h, "c": c}
    if op == "seq":
        h, c, seq = m.forward_seq(*a)
        return {"h": h, "c": c, "seq": seq}
    if op == "stop":
        h, c, steps = m.forward_stop(*a, s["stop_v"], s["stop_c"])
        return {"h": h, "c": c, "steps": steps}
    out = m.forward_train(*a, with_seq=s["d_seq"] is not None)
    got = {"h": out[0], "c": out[1]}
    if s["d_seq"] is not None:
        got["seq"] = out[2]
    got.update(m.backward(*a, s["d_out_h"], s["d_out_c"], s["d_seq"]))
    return got


def _mean_steps(case):
    """Expected sum of the rows' lengths."""
    n = 4096
    u = (torch.arange(n, dtype=torch.float64) + 0.5) / n
    mean = float(_length(case, u).mean())
    B = case["B"]
    total = mean * B
    if case["op"] == "stop":   # seven rows of ten end halfway on average
        total *= 0.65
    if _longest(case):
        total += case["T"] - mean
    return max(total, 1.0)


def work(case):
    B, D, H, T, cell, op = (case[k] for k in ("B", "D", "H", "T", "cell", "op"))
    g, e = _GATES[cell], 2 if case["dtype"] == "bf16" else 4
    steps = _mean_steps(case)
    flops = steps * 2 * g * H * (D + H)
    weights = (D + H) * g * H
    bias = _BIAS[cell] * H * 4
    states = 4 * B * H * (4 if cell == "lstm" else 3)   # h0, c0 in; h, c out
    nbytes = steps * D * e + weights * e + bias + states + 4 * B
    if op == "seq" or (op == "train" and case["dseq"]):
        nbytes += 4 * B * T * H
    if op == "stop":
        nbytes += 4 * H + 4 * B
    if op == "train":
        flops *= 3     # and the gradients of the inputs and of the weights
        nbytes += 4 * B * T * D + 4 * weights + bias + 4 * B * H * (4 if cell == "lstm" else 2)
        if case["dseq"]:
            nbytes += steps * H * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # about four times what an implementation with the same operands is off the
    # fp64 result over these ranges (7e-7 and 3e-4 for most, 5e-4 for the tanh
    # RNN's gradients): fp32 sums in another order, and with bf16 data 16-bit
    # operands of the recurrent product, rounded again at every step
    return {"rel": 5e-6} if case["dtype"] == "f32" else {"rel": 2e-3}


def _step(cell, zx, h, c, U, b, H):
    """One step in fp64 from zx = x W: (h', c', what the backward needs)."""
    if cell == "lstm":
        i, f, g, o = (zx + h @ U + b).split(H, dim=1)
        i, f, g, o = i.sigmoid(), f.sigmoid(), g.tanh(), o.sigmoid()
        c2 = f * c + i * g
        return o * c2.tanh(), c2, (i, f, g, o)
    if cell == "gru":
        a, e = zx + b[:3 * H], h @ U + b[3 * H:]
        r, u = (a[:, :H] + e[:, :H]).sigmoid(), (a[:, H:2 * H] + e[:, H:2 * H]).sigmoid()
        n = (a[:, 2 * H:] + r * e[:, 2 * H:]).tanh()
        return (1 - u) * n + u * h, c, (r, u, n, e[:, 2 * H:])
    h2 = (zx + h @ U + b).tanh()
    return h2, c, (h2,)


def _back(cell, kept, h, c, dh, dc):
    """(gradient of x W, gradient of h U, dh other than through U, dc) of one step."""
    if cell == "lstm":
        i, f, g, o = kept
        t = (f * c + i * g).tanh()
        dct = dc + dh * o * (1 - t * t)
        dz = torch.cat([dct * g * i * (1 - i), dct * c * f * (1 - f), dct * i * (1 - g * g),
                        dh * t * o * (1 - o)], 1)
        return dz, dz, torch.zeros_like(dh), dct * f
    if cell == "gru":
        r, u, n, en = kept
        dn = dh * (1 - u) * (1 - n * n)
        dr, du = dn * en * r * (1 - r), dh * (h - n) * u * (1 - u)
        return torch.cat([dr, du, dn], 1), torch.cat([dr, du, dn * r], 1), dh * u, dc
    dz = dh * (1 - kept[0] * kept[0])
    return dz, dz, torch.zeros_like(dh), dc


def exact(case, seed):
    """What run() returns, in fp64 with plain torch."""
    s = _batch(case, seed)
    B, D, H, T, cell, op = (case[k] for k in ("B", "D", "H", "T", "cell", "op"))
    W, U, b = s["W"].double(), s["U"].double(), s["b"].double()
    h = s["h0"].double()
    c = s["c0"].double() if cell == "lstm" else torch.zeros_like(h)
    # rows by length, longest first: the rows of step t are the first n[t]
    L, order = torch.sort(s["lengths"], descending=True, stable=True)
    h, c = h[order].clone(), c[order].clone()
    x = s["x"]
    last = int(L[0])
    n = (L[None, :] > torch.arange(max(last, 1), device="cuda")[:, None]).sum(1).tolist()
    seq = torch.zeros((B, T, H), device="cuda", dtype=torch.float64) \
        if op == "seq" or (op == "train" and case["dseq"]) else None
    train, stop = op == "train", op == "stop"
    ended = torch.zeros(B, dtype=torch.bool, device="cuda")
    steps = L.clone()
    kept = []
    for t in range(last):
        k = n[t]
        zx = x[order[:k], t].double() @ W
        h2, c2, gates = _step(cell, zx, h[:k], c[:k], U, b, H)
        if train:
            kept.append((h[:k].clone(), c[:k].clone(), gates))
        if stop:
            live = ~ended[:k, None]
            h[:k], c[:k] = torch.where(live, h2, h[:k]), torch.where(live, c2, c[:k])
            now = (h[:k] @ s["stop_v"].double() + s["stop_c"] > 0) & ~ended[:k]
            steps[:k][now] = t + 1
            ended[:k] |= now
        else:
            h[:k], c[:k] = h2, c2
        if seq is not None:
            seq[order[:k], t] = h2

    def back(v):   # to batch order
        out = torch.empty_like(v)
        out[order] = v
        return out

    got = {"h": back(h), "c": back(c) if cell == "lstm" else torch.zeros_like(h)}
    if seq is not None:
        got["seq"] = seq
    if stop:
        got["steps"] = back(steps)
    if not train:
        return got
    dh = s["d_out_h"].double()[order].clone()
    dc = s["d_out_c"].double()[order].clone() if cell == "lstm" else torch.zeros_like(dh)
    g = _GATES[cell]
    dx = torch.zeros((B, T, D), device="cuda", dtype=torch.float64)
    dW, dU = torch.zeros_like(W), torch.zeros_like(U)
    db_x = torch.zeros(g * H, device="cuda", dtype=torch.float64)
    db_h = torch.zeros_like(db_x)
    for t in reversed(range(last)):
        k = n[t]
        hp, cp, gates = kept.pop()
        d = dh[:k]
        if s["d_seq"] is not None:
            d = d + s["d_seq"][order[:k], t].double()
        dzx, dzh, direct, dcp = _back(cell, gates, hp, cp, d, dc[:k])
        dh[:k], dc[:k] = dzh @ U.t() + direct, dcp
        xt = x[order[:k], t].double()
        dW += xt.t() @ dzx
        dU += hp.t() @ dzh
        db_x += dzx.sum(0)
        db_h += dzh.sum(0)
        dx[order[:k], t] = dzx @ W.t()
    got.update({"dx": dx, "dW": dW, "dU": dU, "dh0": back(dh),
                "db": torch.cat([db_x, db_h]) if cell == "gru" else db_x})
    if cell == "lstm":
        got["dc0"] = back(dc)
    return got

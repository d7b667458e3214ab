"""The fp32 input projection (gemm.hip) on either side of the line between its
small and large tiles (one 128 x 128 tile of the valid rows per CU, 256 CUs; three
quarters of that for D of five runs of 16), with each length of a block of K, and
at ragged edges: D and 4H no multiples of a block of K, a tile or a vector, one
row, rows just past a tile.  Output sequence and final state of the forward
against the fp64 oracle at its fp32 tolerance (1e-5)."""
import numpy as np
import pytest

import oracle
import paper_1810_08061_amd as ld
import workloads
from tests.gpu_util import max_err, say, to_device

pytestmark = pytest.mark.gpu

CASES = [  # D, H, B, T: large tiles
    (9, 257, 256, 14),   # 9 x 28 = 252: small
    (9, 257, 256, 15),   # 9 x 30 = 270: large
    (20, 256, 256, 16),  # 8 x 32 = 256: small
    (20, 256, 241, 17),  # 8 x 33 = 264: large
    (30, 259, 241, 17),  # 9 x 33 = 297: large
    (68, 256, 256, 12),  # 8 x 24 = 192: small
    (68, 256, 241, 13),  # 8 x 25 = 200: large
    (68, 256, 253, 15),  # 8 x 30 = 240: large
    (68, 256, 241, 17),  # 8 x 33 = 264: large
    (50, 256, 241, 17),  # 8 x 33 = 264: large, blocks of 32
    (64, 256, 241, 17),  # the same, whole vectors
    (97, 257, 241, 17),  # 9 x 33 = 297: large, blocks of 16, seven of them
    (255, 130, 241, 29), # 5 x 55 = 275: large, blocks of 32
    (1, 33, 1, 1), (64, 40, 65, 1), (130, 70, 129, 2),
]


@pytest.mark.parametrize("D,H,B,T", CASES)
def test_tiles(D, H, B, T):
    import torch
    say(f"case inproj f32 D={D} H={H} B={B} T={T}")
    inp = workloads.random_case(8100 + D + H, B, D, H, T, dtype="f32")
    inp.lengths[:] = T
    m = ld.LstmDyn(B, D, H, T, "f32", "persistent")
    h, c, seq = m.forward_seq(*to_device(inp))
    torch.cuda.synchronize()
    assert m.query(ld.Q_LAST_STATUS) == ld.OK
    ho, co, so = oracle.forward_inputs(inp, seq=True)
    errs = [max_err(a.cpu().numpy(), o) for a, o in ((h, ho), (c, co), (seq, so))]
    say("  max errors h, c, seq: " + " ".join(f"{e:.2e}" for e in errs))
    assert max(errs) <= 1e-5
    m.close()

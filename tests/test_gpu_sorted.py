"""One-shot calls whose workgroups sort the rows themselves (a few rows per CU) against a stored plan, whose rows are
ordered by the pre-pass and handed out by tickets: a row's result does not depend on who computes it, so every bit is
the same.  Every query block has to turn up exactly once in either order."""
import numpy as np
import pytest
import torch

import paper_2509_25401_amd as pkg
from gpu_utils import down_bits, up_u8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,bq,bk,B,H,L,keep,cached", [
    (64, 64, 64, 1, 257, 100, 0.7, 0.3),        # 514 rows; two blocks a head
    (64, 128, 128, 1, 257, 90, 1.0, 0.5),       # 257 rows: one more than CUs, one symbol byte each
    (128, 128, 128, 1, 24, 6144, 0.2, 0.0),     # 1152 rows: the most for 512 workgroups, no flags
    (128, 128, 128, 1, 24, 4608, 0.3, 0.5625),  # fewer computed rows than workgroups: the others move cached rows
    (64, 64, 128, 1, 32, 4096, 0.1, 0.2),       # 2048 rows: the longest lists
    (64, 64, 64, 1, 4, 8192, 0.3, 0.6),         # four symbol words a row
    (128, 64, 64, 1, 7, 2600, 0.4, 0.3),        # 287 rows, 41 symbols each: an odd number of bytes, parts of unequal size
    (128, 64, 128, 2, 11, 2049, 0.5, 0.9),      # one token in the last block, nearly everything cached
    (64, 128, 64, 1, 20, 4000, 0.3, 0.1),
    (64, 128, 128, 1, 24, 4000, 0.3, 0.0),      # 96 rows per XCD: one for each of three workgroups per CU
    (64, 128, 128, 1, 24, 4608, 0.3, 0.04),     # some 104 computed rows: the first eight or so workgroups have a second one
    (64, 128, 64, 1, 24, 6000, 0.2, 0.0),       # 141 rows: nearly half of the 96 have a second one
    (64, 64, 128, 1, 24, 3584, 0.3, 0.0),       # 168 rows on 128 workgroups: the last round on the first and third of a CU
    (64, 64, 64, 1, 24, 4608, 0.2, 0.0),        # 216 rows: the last round from the end
    (128, 64, 64, 1, 24, 3584, 0.3, 0.0),
])
def test_sorted_rows_match_a_stored_plan(D, bq, bk, B, H, L, keep, cached):
    print(f"[case] sorted D={D} {bq}x{bk} B={B} H={H} L={L}", flush=True)
    Tq, Tk = -(-L // bq), -(-L // bk)
    rng = np.random.default_rng(B * H * L + D)
    mask = (rng.random((B, H, Tq, Tk)) < keep).astype(np.uint8)
    mask[0, 0, 0] = 1                                        # a row that keeps everything,
    mask[0, H // 2, Tq - 1] = 0                              # one that keeps nothing
    flags = None
    if cached > 0:
        flags = (rng.random((B, H, Tq)) < cached).astype(np.uint8)
        flags[0, 0] = 1                                      # a head without a computed row
        flags[0, H // 2, Tq - 1] = 0
    packed, dflags = up_u8(pkg.sparse_attn_pack_mask(mask)), up_u8(flags)
    g = torch.Generator(device="cuda").manual_seed(L)
    Q, K, V, C0, C1 = (torch.randn(B, H, L, D, device="cuda", generator=g).bfloat16() for _ in range(5))
    plan = pkg.SparseAttnPlan(dflags, packed, B, H, L, bq, bk)

    def both(one_shot, planned):
        outs = []
        for call in (one_shot, planned):
            O = torch.full((B, H, L, D), 3.0, dtype=torch.bfloat16, device="cuda")
            call(O)
            torch.cuda.synchronize()
            outs.append(down_bits(O))
        assert (outs[0] == outs[1]).all()
        return outs[0]

    for cache in (None, C0):                                 # cached rows left alone, or copied
        got = both(lambda O: pkg.sparse_attn_fwd(Q, K, V, dflags, packed, cache, O, bq, bk),
                   lambda O: plan.run(Q, K, V, cache, O))
    if flags is not None:
        rows = np.repeat(flags != 0, bq, axis=2)[:, :, :L]
        assert (got[rows] == down_bits(C0)[rows]).all()
        coef = [1.0, 2.0]
        both(lambda O: pkg.sparse_attn_fwd_forecast(Q, K, V, dflags, packed, [C0, C1], coef, O, bq, bk),
             lambda O: plan.run_forecast(Q, K, V, [C0, C1], coef, O))
    empty = got[0, H // 2, (Tq - 1) * bq:]
    assert (empty == 0).all()
    plan.destroy()

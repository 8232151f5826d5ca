"""GPU tests of the reusable plan (sparse_attn_plan_*): the stored pre-pass must drive the same kernel to the same
bits as the one-shot call, run after run, and symbols at granularity n must decode as Section 3.4 defines."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_25401_amd as pkg
from paper_2509_25401_amd import synth
from gpu_utils import DeviceCase, dev, up_bf16, up_u8, down_bits, oracle_full, check_against_oracle, prepass_ran

pytestmark = pytest.mark.gpu


def fresh_O(w, fill=0x4242):
    return torch.from_numpy(np.full(w.Q.shape, fill, dtype=np.uint16).view(np.int16)).view(torch.bfloat16).to(dev())


@pytest.mark.parametrize("D,bq,bk", [(128, 128, 128), (64, 64, 128), (128, 128, 64)])
def test_plan_reproduces_the_one_shot_call_bit_for_bit(D, bq, bk):
    w = synth.random_case(synth.BASE_SEED + 90 + D + bq, 2, 3, 1024, D, bq, bk, keep=0.4, cached_frac=0.3)
    case = DeviceCase(w)
    want = case.run()
    flags, mask = case.flags.clone(), case.mask.clone()
    plan = pkg.SparseAttnPlan(flags, mask, w.B, w.H, w.L, bq, bk)
    torch.cuda.synchronize()
    flags.fill_(1)                        # the plan holds its own decoded copy: the symbol arrays may change
    mask.zero_()
    for rep in range(3):                  # the queue counters are reset for every run
        O = fresh_O(w)
        plan.run(case.Q, case.K, case.V, case.Oc, O)
        torch.cuda.synchronize()
        assert (down_bits(O) == want).all(), f"run {rep} differs from the one-shot call"
    ref, ref_bits = oracle_full(w)
    check_against_oracle(w, want, ref, ref_bits, f"plan D{D} {bq}x{bk}")
    plan.destroy()


@pytest.mark.parametrize("D,bq,bk,n_terms", [(128, 128, 128, 2), (64, 64, 64, 3)])
def test_plan_with_forecast_reproduces_the_one_shot_forecast(D, bq, bk, n_terms):
    """Stored plan + Taylor forecast in the cache branch: the same bits as sparse_attn_fwd_forecast (whose parity
    with the oracle is checked where that entry point is tested), run after run."""
    w = synth.random_case(synth.BASE_SEED + 95 + n_terms, 1, 4, 1152, D, bq, bk, keep=0.5, cached_frac=0.4)
    rng = np.random.default_rng(synth.BASE_SEED + 96 + n_terms)
    terms = [up_bf16(w.O_cache)] + [up_bf16(synth.normal_bf16(rng, w.Q.shape)) for _ in range(n_terms - 1)]
    coef = pkg.sparse_taylor_coefficients(n_terms - 1, 3.0)
    case = DeviceCase(w)
    want = fresh_O(w)
    pkg.sparse_attn_fwd_forecast(case.Q, case.K, case.V, case.flags, case.mask, terms, coef, want, bq, bk)
    plan = pkg.SparseAttnPlan(case.flags, case.mask, w.B, w.H, w.L, bq, bk)
    torch.cuda.synchronize()
    rows = np.repeat(w.cache_flags != 0, bq, axis=2)
    assert rows.any() and (~rows).any()
    for rep in range(2):
        O = fresh_O(w)
        plan.run_forecast(case.Q, case.K, case.V, terms, coef, O)
        torch.cuda.synchronize()
        assert (down_bits(O) == down_bits(want)).all(), f"run {rep} differs from the one-shot forecast"
    # and it is not the plain copy: the forecast moved the cached blocks away from term 0
    assert (down_bits(want)[rows] != w.O_cache[rows]).any()
    plan.destroy()


@pytest.mark.parametrize("n,L", [(2, 1024), (3, 896), (4, 2048)])
def test_granularity_decodes_like_the_expanded_symbols(n, L):
    B, H, D, blk = 1, 2, 128, 128
    T = L // blk
    sT = -(-T // n)
    rng = np.random.default_rng(synth.BASE_SEED + 95 + n)
    w = synth.random_case(synth.BASE_SEED + 96 + n, B, H, L, D, blk, blk, keep=1.0, cached_frac=0.0, with_cache_tensor=True)
    coarse_flags = (rng.random((B, H, sT)) < 0.3).astype(np.uint8)
    coarse_M = (rng.random((B, H, sT, sT)) < 0.5).astype(np.uint8)
    coarse_M[..., 0] = 1                                           # every row keeps something
    f, m = oracle.expand_granularity(coarse_flags, coarse_M, n, T, T)
    ref, ref_bits = oracle.sparse_attention(w.Q, w.K, w.V, f, oracle.pack_symbols(m), w.O_cache, blk, blk)
    Q, K, V, Oc = up_bf16(w.Q), up_bf16(w.K), up_bf16(w.V), up_bf16(w.O_cache)
    plan = pkg.SparseAttnPlan(up_u8(coarse_flags), up_u8(pkg.sparse_attn_pack_mask(coarse_M)), B, H, L, blk, blk, granularity=n)
    O = fresh_O(w)
    plan.run(Q, K, V, Oc, O)
    torch.cuda.synchronize()
    got = down_bits(O)
    w.cache_flags, w.M_s = f, m
    check_against_oracle(w, got, ref, ref_bits, f"granularity {n}")
    # the same tiles through the one-shot call with symbols expanded to granularity 1: identical bits
    O1 = fresh_O(w)
    pkg.sparse_attn_fwd(Q, K, V, up_u8(f), up_u8(pkg.sparse_attn_pack_mask(m)), Oc, O1, blk, blk)
    torch.cuda.synchronize()
    assert (down_bits(O1) == got).all()
    plan.destroy()


def test_plan_without_symbols_is_dense_attention_and_skips_the_prepass_time():
    w = synth.random_case(synth.BASE_SEED + 99, 1, 4, 4608, 128, 128, 128, keep=1.0)
    case = DeviceCase(w)
    plan = pkg.SparseAttnPlan(None, None, w.B, w.H, w.L, 128, 128)
    O = fresh_O(w)
    plan.run(case.Q, case.K, case.V, None, O)
    torch.cuda.synchronize()
    O1 = fresh_O(w)
    pkg.sparse_attn_fwd(case.Q, case.K, case.V, None, None, None, O1, 128, 128)
    torch.cuda.synchronize()
    assert (down_bits(O) == down_bits(O1)).all()
    # timing, for the log only: stored plan vs pre-pass on every call
    def timed(fn, reps=20):
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            fn()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / reps
    t_plan = timed(lambda: plan.run(case.Q, case.K, case.V, None, O))
    t_shot = timed(lambda: pkg.sparse_attn_fwd(case.Q, case.K, case.V, None, None, None, O1, 128, 128))
    print(f"[plan] 4608 tokens x 4 heads dense: stored plan {t_plan * 1e3:.1f} us/call, one-shot {t_shot * 1e3:.1f} us/call", flush=True)
    plan.destroy()


def test_caller_supplied_workspace_and_scratch_release():
    """sparse_attn_fwd_workspace writes the bits of the one-shot call using only the caller's buffer (a buffer one
    byte short is refused); releasing the library's scratch of the stream leaves the next one-shot call working."""
    # 1112 rows of five words: more than the attention kernel sees to itself, so the pre-pass fills the buffer
    w = synth.random_case(synth.BASE_SEED + 97, 2, 4, 8833, 64, 64, 64, keep=0.1, cached_frac=0.3)
    case = DeviceCase(w)
    want = case.run()
    need = pkg.sparse_attn_workspace_bytes(w.B, w.H, w.L, w.block_q, w.block_k)
    ws = torch.full((need + 512,), 0xAB, dtype=torch.uint8, device=dev())
    base = (-ws.data_ptr()) % 256
    O = fresh_O(w)
    pkg.sparse_attn_fwd_workspace(case.Q, case.K, case.V, case.flags, case.mask, case.Oc, O, w.block_q, w.block_k,
                                  ws[base:base + need])
    torch.cuda.synchronize()
    assert (down_bits(O) == want).all()
    assert (ws[base:base + need] != 0xAB).any(), "the call did without the workspace"
    assert (ws[base + need:] == 0xAB).all() and (ws[:base] == 0xAB).all(), "wrote outside the workspace"
    with pytest.raises(pkg.SparseAttnError):
        pkg.sparse_attn_fwd_workspace(case.Q, case.K, case.V, case.flags, case.mask, case.Oc, O, w.block_q, w.block_k,
                                      ws[base:base + need - 1])
    pkg.sparse_attn_release_scratch()
    pkg.sparse_attn_release_scratch()          # nothing left to free: still fine
    assert (case.run() == want).all()


# (B, H, L, D, block_q, block_k, keep or None for no mask, cached share, one-shot route): rows around what the chip runs at a
# time (512 workgroups, 1024 for 64-row blocks of 64 channels) and around where the one-shot call changes its way to hand them
# out, fewer rows than queues, heads that do not fill the queues
ROUTES = [
    (1, 1, 50, 64, 64, 64, None, 0.0, "dealt"),
    (1, 5, 130, 128, 128, 64, 0.6, 0.3, "dealt"),
    (1, 9, 2100, 64, 64, 64, 0.3, 0.3, "sorted"),
    (2, 24, 1344, 64, 64, 64, 0.4, 0.4, "sorted"),       # 1008 rows
    (2, 24, 1400, 64, 64, 64, 0.4, 0.4, "sorted"),       # 1056 rows
    (1, 31, 2100, 128, 128, 128, 0.3, 0.0, "sorted"),    # 527 rows
    (1, 31, 2100, 128, 128, 128, None, 0.0, "dealt"),    # 527 equal rows: some workgroups take two
    (1, 31, 4300, 64, 128, 128, None, 0.0, "list"),      # 1054 equal rows
    (1, 17, 4300, 64, 128, 128, None, 0.5, "list"),      # flags alone
    (1, 24, 1409, 128, 64, 64, None, 0.0, "dealt"),      # 288 blocks of 128 rows: done in 256-row blocks whatever the caller's
    (2, 30, 2500, 128, 128, 128, None, 0.0, "list"),     # 600 blocks of 256 rows: some workgroups take three
    (1, 2, 8300, 64, 64, 64, 0.1, 0.2, "dealt"),         # five words a row, 130 bits in rows of 17 bytes
    (1, 16, 8300, 64, 64, 64, 0.05, 0.2, "list"),        # 2080 such rows: five words are too many to sort
    (2, 24, 3100, 64, 64, 64, 0.3, 0.3, "list"),         # 2352 rows: too many to sort
    (1, 24, 6300, 64, 128, 64, 0.2, 0.3, "list"),        # 1200 rows of 128: more than two and a quarter per workgroup
    (1, 25, 6017, 128, 128, 128, 0.2, 0.2, "list"),      # 1200, queues of three and four heads, one row in the last block
    (1, 24, 1330, 128, 64, 128, 0.4, 0.0, "sorted"),     # 504 rows of 64 x 128 channels: 64-key sub-tiles
    (1, 24, 2040, 128, 64, 64, 0.4, 0.3, "sorted"),      # 768, some cached: the same, one round and a half
    (1, 24, 2050, 128, 64, 64, 0.4, 0.3, "sorted"),      # 792: 32-key sub-tiles
    (2, 22, 3100, 128, 64, 64, 0.1, 0.3, "list"),        # 2156
    (1, 1, 33100, 64, 64, 64, 0.04, 0.2, "dealt"),       # 518 rows of 17 words; the plan decodes them in a kernel of its own
]


@pytest.mark.parametrize("B,H,L,D,bq,bk,keep,cached,route", ROUTES)
def test_dealt_rows_and_work_list_agree(B, H, L, D, bq, bk, keep, cached, route):
    """The one-shot call deals few rows out by workgroup number or sorts them in its workgroups, and decodes them in place;
    beyond, and in a stored plan, they go through the work list.  Same rows, same bits; the symbols start at an odd byte."""
    print(f"[case] routes B={B} H={H} L={L} D={D} {bq}x{bk} keep={keep} cached={cached}", flush=True)
    w = synth.random_case(synth.BASE_SEED + 120 + L, B, H, L, D, bq, bk, keep=1.0 if keep is None else keep,
                          cached_frac=cached, with_cache_tensor=True)
    if keep is None:
        w.M_s = None
    elif w.cache_flags is None or not w.cache_flags[0, 0, 0]:
        w.M_s[0, 0, 0] = 0                  # a computed row without a kept block
    case = DeviceCase(w)
    if case.mask is not None:
        raw = torch.zeros(case.mask.numel() + 3, dtype=torch.uint8, device=dev())
        odd = raw[3:].view(case.mask.shape)
        odd.copy_(case.mask)
        case.mask = odd
    got = case.run()
    assert prepass_ran(case) == (route == "list")
    plan = pkg.SparseAttnPlan(case.flags, case.mask, w.B, w.H, w.L, bq, bk)
    for rep in range(3):
        O = fresh_O(w)
        plan.run(case.Q, case.K, case.V, case.Oc, O)
        torch.cuda.synchronize()
        assert (down_bits(O) == got).all(), f"run {rep} of the plan differs from the one-shot call"
    plan.destroy()
    ref, ref_bits = oracle_full(w)
    check_against_oracle(w, got, ref, ref_bits, f"routes {B}x{H}x{L}")


@pytest.mark.parametrize("profile", ["growing", "staircase", "spiky"])
@pytest.mark.parametrize("D,bq,bk", [(128, 64, 64), (128, 64, 128), (128, 128, 64), (64, 64, 64)])
def test_bits_do_not_depend_on_the_blocks_when_the_reference_moves(D, bq, bk, profile):
    """Dense attention in the caller's blocks (a stored plan) and in the kernel's own (one-shot call, 272 blocks of 128
    rows): same bits, also where the exponent's reference is raised in the middle of a row.  "staircase": every
    64 keys are four times louder than the 64 before, so the first 32 of them raise it and the next 32 follow."""
    B, H, L = 1, 17, 2000
    print(f"[case] blocks D={D} {bq}x{bk} {profile}", flush=True)
    w = synth.random_case(synth.BASE_SEED + 330 + D + bq, B, H, L, D, bq, bk, keep=1.0)
    pos = np.arange(L, dtype=np.float32)[None, None, :, None]
    scale = {"growing": 0.1 + 2.9 * pos / L, "staircase": 0.05 * 4.0 ** np.minimum(pos // 64, 3),
             "spiky": np.where(pos % 97 == 0, 12.0, 0.5)}[profile].astype(np.float32)
    w.K = synth.f32_to_bf16_bits(synth.bf16_bits_to_f32(w.K) * scale)
    w.M_s = None
    case = DeviceCase(w)
    got = case.run()
    plan = pkg.SparseAttnPlan(None, None, B, H, L, bq, bk)
    O = fresh_O(w)
    plan.run(case.Q, case.K, case.V, None, O)
    torch.cuda.synchronize()
    plan.destroy()
    ref, _ = oracle_full(w)
    err = np.abs(synth.bf16_bits_to_f32(got).astype(np.float64) - ref)
    # weights are rounded to bf16 (relative 2^-9), the same ones in the product and in the sum it is divided by, and so
    # is the result: at most 3 * 2^-9 of the largest value, however few keys a row's weight lies on
    assert err.max() <= 3 * 2.0 ** -9 * np.abs(synth.bf16_bits_to_f32(w.V)).max()
    differ = (down_bits(O) != got).sum()
    assert differ == 0, f"{differ} of {got.size} values depend on the blocks"


def test_plan_is_intact_behind_runs_that_overlapped():
    """Two runs of one plan that overlap in time share its queue counters and leave out blocks of their outputs.  What
    follows them, ordered behind both, is right: the counters are back at zero when the last workgroup of both ends."""
    w = synth.random_case(synth.BASE_SEED + 340, 1, 24, 4608, 128, 128, 128, keep=0.4, cached_frac=0.3)
    case = DeviceCase(w)
    plan = pkg.SparseAttnPlan(case.flags, case.mask, w.B, w.H, w.L, 128, 128)
    want, O = fresh_O(w), fresh_O(w)
    plan.run(case.Q, case.K, case.V, case.Oc, want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for rep in range(20):
        for st in streams:
            plan.run(case.Q, case.K, case.V, case.Oc, O, stream=st)
        torch.cuda.synchronize()
        got = fresh_O(w)
        plan.run(case.Q, case.K, case.V, case.Oc, got)
        torch.cuda.synchronize()
        assert (down_bits(got) == down_bits(want)).all(), f"run behind the {rep}-th overlapping pair"
    plan.destroy()


@pytest.mark.parametrize("n", [1, 2, 3])
def test_symbols_decoded_in_front_of_the_queues(n):
    """202 rows of 7 words per queue: at granularity 1 the queue's workgroup decodes them, else a kernel of its own; both
    give the bits of the one-shot call with the symbols expanded to tiles."""
    B, H, L, D, blk = 1, 3, 12900, 64, 64
    T = -(-L // blk)
    sT = -(-T // n)
    rng = np.random.default_rng(synth.BASE_SEED + 350 + n)
    w = synth.random_case(synth.BASE_SEED + 351 + n, B, H, L, D, blk, blk, keep=1.0, cached_frac=0.0, with_cache_tensor=True)
    coarse_flags = (rng.random((B, H, sT)) < 0.3).astype(np.uint8)
    coarse_M = (rng.random((B, H, sT, sT)) < 0.1).astype(np.uint8)
    coarse_flags[0, 0, 1], coarse_M[0, 0, 1] = 0, 0                # computed rows without a kept block
    f, m = oracle.expand_granularity(coarse_flags, coarse_M, n, T, T)
    Q, K, V, Oc = up_bf16(w.Q), up_bf16(w.K), up_bf16(w.V), up_bf16(w.O_cache)
    packed = up_u8(pkg.sparse_attn_pack_mask(coarse_M))
    raw = torch.zeros(packed.numel() + 1, dtype=torch.uint8, device=dev())
    odd = raw[1:].view(packed.shape)
    odd.copy_(packed)
    plan = pkg.SparseAttnPlan(up_u8(coarse_flags), odd, B, H, L, blk, blk, granularity=n)
    O, O1 = fresh_O(w), fresh_O(w)
    plan.run(Q, K, V, Oc, O)
    pkg.sparse_attn_fwd(Q, K, V, up_u8(f), up_u8(pkg.sparse_attn_pack_mask(m)), Oc, O1, blk, blk)
    torch.cuda.synchronize()
    plan.destroy()
    assert (down_bits(O) == down_bits(O1)).all()
    c = np.repeat(f != 0, blk, axis=2)[:, :, :L]
    assert (down_bits(O)[c] == w.O_cache[c]).all()
    empty = np.repeat((f == 0) & ~m.any(axis=-1), blk, axis=2)[:, :, :L]
    assert empty.any() and (down_bits(O)[empty] == 0).all()


@pytest.mark.parametrize("D,bk,L", [(64, 64, 2900), (128, 128, 2900),       # 1104 rows: sorted by the workgroups
                                    (64, 64, 5500), (128, 128, 5500)])      # 2064: work list
def test_skewed_rows_of_64_row_blocks(D, bk, L):
    """A tenth of the rows keeps nine tenths of the key blocks, the others 5 %: long rows, fine buckets and a queue whose
    grid has four workgroups per CU.  Every block once, same bits as the plan's."""
    B, H, bq = 1, 24, 64
    w = synth.random_case(synth.BASE_SEED + 360 + D, B, H, L, D, bq, bk, keep=1.0, cached_frac=0.1)
    rng = np.random.default_rng(synth.BASE_SEED + 361 + D)
    p = np.where(rng.random((B, H, w.M_s.shape[2], 1)) < 0.1, 0.9, 0.05)
    w.M_s = (rng.random(w.M_s.shape) < p).astype(w.M_s.dtype)
    case = DeviceCase(w)
    got = case.run()
    assert prepass_ran(case) == (L == 5500)
    plan = pkg.SparseAttnPlan(case.flags, case.mask, B, H, L, bq, bk)
    O = fresh_O(w)
    plan.run(case.Q, case.K, case.V, case.Oc, O)
    torch.cuda.synchronize()
    plan.destroy()
    assert (down_bits(O) == got).all()
    # a row with a single kept block of K keys is a mean of that many values: the usual bar, and per value the bound of
    # rounded weights and a rounded result
    ref, ref_bits = oracle_full(w)
    c = np.repeat(w.cache_flags != 0, bq, axis=2)[:, :, :L]
    assert (got[c] == ref_bits[c]).all()
    err = np.abs(synth.bf16_bits_to_f32(got).astype(np.float64) - ref)[~c]
    assert err.max() <= 3 * 2.0 ** -9 * np.abs(synth.bf16_bits_to_f32(w.V)).max() and err.mean() <= 1e-3

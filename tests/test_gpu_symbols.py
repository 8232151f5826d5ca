"""GPU parity of the symbol generation (sparse_symbols_update) against the fp64 oracle.

The kernels decide in fp32, the oracle in fp64.  A yes/no decision is compared wherever the oracle's deciding
quantity is further from its threshold than fp32 rounding can move it (and than a near-tie in the ascending order
could move it); the remaining, undecidable entries must be rare."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_25401_amd as pkg
from paper_2509_25401_amd import synth
from gpu_utils import dev, up_bf16, down_bits, check_against_oracle
from helpers import compare_symbols

pytestmark = pytest.mark.gpu

def f32(x):
    return float(np.float32(x))


def run_gpu(Q, K, block, text, tau_c, tau_kv, s_q=0.0):
    B, H, L, D = Q.shape
    T = -(-L // block)
    flags = torch.full((B, H, T), 0xAA, dtype=torch.uint8, device=dev())
    mask = torch.full((B, H, T, (T + 7) // 8), 0xAA, dtype=torch.uint8, device=dev())
    pkg.sparse_symbols_update(up_bf16(Q), up_bf16(K), flags, mask, block, text, tau_c, tau_kv, s_q)
    torch.cuda.synchronize()
    return flags.cpu().numpy(), mask.cpu().numpy()


def compare(ref, flags, mask, T, label, max_ambiguous=0.02, require_identical=True):
    """On the structured test inputs the fp32 kernels reproduce every decision of the fp64 oracle, so the raw
    symbols are required to be identical; the margin rule of helpers.compare_symbols stays in force underneath
    (it is what the statement "a decision within rounding of its threshold may differ" means)."""
    bits = oracle.unpack_symbols(mask, T)
    if T % 8:    # padding bits of the last byte are zero
        assert (mask[..., -1] & ((1 << (8 - T % 8)) - 1) == 0).all(), f"{label}: padding bits set"
    compare_symbols(ref, flags, bits, label, max_ambiguous, require_identical)
    return bits


@pytest.mark.parametrize("B,H,L,D,block,text,tau_c,tau_kv", [
    (1, 2, 1024, 128, 128, 256, 0.5, 0.1),        # 8 blocks, 2 text
    (2, 3, 2560, 128, 128, 128, 0.3, 0.2),        # 20 blocks, 1 text block, row groups with a ragged tail
    (1, 2, 4160, 64, 64, 192, 0.6, 0.05),         # 65 blocks (more than one lane pass), D = 64, 3 text blocks
    (1, 2, 8320, 128, 64, 256, 0.4, 0.3),         # 130 blocks at block 64, D = 128
    (1, 1, 33280, 64, 128, 512, 0.5, 0.15),       # 260 blocks (more than 256: two thread passes), 4 text blocks
])
def test_symbols_match_oracle(B, H, L, D, block, text, tau_c, tau_kv):
    tau_c, tau_kv = f32(tau_c), f32(tau_kv)
    Q, K = synth.structured_qk(synth.BASE_SEED + L + D, B, H, L, D, block)
    ref = oracle.update_symbols(Q, K, block, text, tau_c, tau_kv)
    flags, mask = run_gpu(Q, K, block, text, tau_c, tau_kv)
    compare(ref, flags, mask, L // block, f"L{L}_D{D}_b{block}")
    assert (flags[..., : text // block] == 0).all()


def test_threshold_extremes_and_degrade_rule():
    B, H, L, D, block, text = 1, 2, 2048, 128, 128, 256
    Q, K = synth.structured_qk(synth.BASE_SEED + 7, B, H, L, D, block)
    T, nt = L // block, text // block
    flags, mask = run_gpu(Q, K, block, text, 0.0, 0.0)
    assert flags.sum() == 0 and (oracle.unpack_symbols(mask, T) == 1).all()
    flags, mask = run_gpu(Q, K, block, text, 1.0, 0.0)
    assert (flags[..., nt:] == 1).all() and (flags[..., :nt] == 0).all()
    # degrade: with tau_c = 1 only the 2 text blocks of 16 need computation (0.125)
    flags, _ = run_gpu(Q, K, block, text, 1.0, 0.0, s_q=0.25)
    assert (flags == 1).all()
    flags, _ = run_gpu(Q, K, block, text, 1.0, 0.0, s_q=0.0625)
    assert (flags[..., :nt] == 0).all()
    # tau_kv = 1 skips every block whose cumulative sum stays <= 1: everything except possibly the largest
    _, mask = run_gpu(Q, K, block, text, 0.0, 1.0)
    assert oracle.unpack_symbols(mask, T).sum(axis=-1).max() <= 1


def test_uniform_map_closed_form_and_repeatability():
    """Q = 0: all entries tie, ties go by index, so exactly the first floor(tau * count) entries are taken."""
    B, H, L, D, block, text = 1, 2, 2560, 128, 128, 512       # 20 blocks, 4 text, 16 vision
    _, K = synth.structured_qk(synth.BASE_SEED + 8, B, H, L, D, block)
    Q = np.zeros_like(K)
    flags, mask = run_gpu(Q, K, block, text, f32(0.33), f32(0.27))
    assert (flags[:, :, :4] == 0).all() and (flags[:, :, 4:9] == 1).all() and (flags[:, :, 9:] == 0).all()
    bits = oracle.unpack_symbols(mask, 20)
    assert (bits[..., :5] == 0).all() and (bits[..., 5:] == 1).all()
    flags2, mask2 = run_gpu(Q, K, block, text, f32(0.33), f32(0.27))
    assert (flags2 == flags).all() and (mask2 == mask).all()


def test_video_size_symbols_and_the_attention_they_drive():
    """Full sequence length of the video workload (258 blocks, 2 of them text), 4 heads; then the symbols the GPU
    wrote drive the attention kernel, checked against the oracle run on the ORACLE's symbols over the rows where
    both sets of symbols agree."""
    B, H, L, D, block, text = 1, 4, 33024, 128, 128, 256
    tau_c, tau_kv = f32(0.5), f32(0.2)
    Q, K = synth.structured_qk(synth.BASE_SEED + 9, B, H, L, D, block)
    V = synth.normal_bf16(np.random.default_rng(synth.BASE_SEED + 10), (B, H, L, D))
    Oc = synth.normal_bf16(np.random.default_rng(synth.BASE_SEED + 11), (B, H, L, D))
    ref = oracle.update_symbols(Q, K, block, text, tau_c, tau_kv)
    T = L // block
    dQ, dK, dV, dOc = up_bf16(Q), up_bf16(K), up_bf16(V), up_bf16(Oc)
    flags = torch.zeros((B, H, T), dtype=torch.uint8, device=dev())
    mask = torch.zeros((B, H, T, (T + 7) // 8), dtype=torch.uint8, device=dev())
    pkg.sparse_symbols_update(dQ, dK, flags, mask, block, text, tau_c, tau_kv)
    O = torch.zeros_like(dQ)
    pkg.sparse_attn_fwd(dQ, dK, dV, flags, mask, dOc, O, block, block)
    torch.cuda.synchronize()
    bits = compare(ref, flags.cpu().numpy(), mask.cpu().numpy(), T, "video33k")
    same = (flags.cpu().numpy() == ref["cache_flags"]) & (bits == ref["M_s"]).all(axis=-1)      # [B,H,T]
    assert same.mean() > 0.95
    rng = np.random.default_rng(5)
    cand = np.argwhere(same)
    items = cand[rng.choice(len(cand), size=24, replace=False)]
    flat = np.array([(b * H + h) * T + i for b, h, i in items], dtype=np.int64)
    got = down_bits(O)
    ref_o, ref_bits = oracle.sparse_attention_blocks(Q, K, V, ref["cache_flags"], oracle.pack_symbols(ref["M_s"]), Oc,
                                                     block, block, flat)
    n_cached = 0
    for n, (b, h, i) in enumerate(items):
        rows = slice(i * block, (i + 1) * block)
        if ref["cache_flags"][b, h, i]:
            assert (got[b, h, rows] == Oc[b, h, rows]).all()
            n_cached += 1
        else:
            err = np.abs(synth.bf16_bits_to_f32(got[b, h, rows]).astype(np.float64) - ref_o[n])
            assert err.max() <= 1e-2 and err.mean() <= 1e-3
    print(f"[symbols] video33k pipeline: {len(items)} sampled blocks ({n_cached} cached) match the oracle", flush=True)


@pytest.mark.parametrize("L,D,block,text", [(1000, 128, 128, 128), (4200, 64, 64, 128), (2561, 128, 128, 256)])
def test_short_last_block(L, D, block, text):
    B, H = 1, 2
    T = -(-L // block)
    Q, K = synth.structured_qk(synth.BASE_SEED + 500 + L, B, H, T * block, D, block)
    Q, K = np.ascontiguousarray(Q[:, :, :L]), np.ascontiguousarray(K[:, :, :L])
    tau_c, tau_kv = f32(0.5), f32(0.2)
    ref = oracle.update_symbols(Q, K, block, text, tau_c, tau_kv)
    flags, mask = run_gpu(Q, K, block, text, tau_c, tau_kv)
    compare(ref, flags, mask, T, f"ragged L{L}_D{D}_b{block}", max_ambiguous=0.05)


def run_gpu_granular(Q, K, bq, bk, n, text, tau_c, tau_kv, s_q=0.0):
    B, H, L, D = Q.shape
    Tq, Tk = -(-L // (n * bq)), -(-L // (n * bk))
    flags = torch.full((B, H, Tq), 0xAA, dtype=torch.uint8, device=dev())
    mask = torch.full((B, H, Tq, (Tk + 7) // 8), 0xAA, dtype=torch.uint8, device=dev())
    pkg.sparse_symbols_update(up_bf16(Q), up_bf16(K), flags, mask, bq, text, tau_c, tau_kv, s_q, block_k=bk, granularity=n)
    torch.cuda.synchronize()
    return flags, mask


@pytest.mark.parametrize("L,D,bq,bk,n,text", [
    (4096, 128, 128, 128, 2, 256),        # pooled blocks of 256 tokens: 16 x 16 symbols
    (6000, 128, 128, 128, 3, 500),        # 384-token pooled blocks, short last one, text ends inside a pooled block
    (4096, 64, 64, 128, 1, 256),          # b_q != b_k: 64 x 32 map, the contribution metric is carried over
    (5000, 128, 128, 64, 2, 300),         # b_q = 2 b_k with granularity 2, nothing lines up
    (16640, 64, 64, 64, 4, 512),          # 65 pooled blocks of 256 tokens
])
def test_granular_symbols_match_oracle(L, D, bq, bk, n, text):
    """Section 3.3 with granularity n and b_q != b_k: maps of ceil(L/(n b_q)) x ceil(L/(n b_k)) pooled blocks."""
    B, H = 1, 2
    tau_c, tau_kv = f32(0.5), f32(0.2)
    pool = n * max(bq, bk)
    Lp = -(-L // pool) * pool
    Q, K = synth.structured_qk(synth.BASE_SEED + 900 + L + n, B, H, Lp, D, n * min(bq, bk))
    Q, K = np.ascontiguousarray(Q[:, :, :L]), np.ascontiguousarray(K[:, :, :L])
    ref = oracle.update_symbols(Q, K, bq, text, tau_c, tau_kv, block_k=bk, granularity=n)
    flags, mask = run_gpu_granular(Q, K, bq, bk, n, text, tau_c, tau_kv)
    Tk = -(-L // (n * bk))
    mask_h = mask.cpu().numpy()
    if Tk % 8:
        assert (mask_h[..., -1] & ((1 << (8 - Tk % 8)) - 1) == 0).all(), "padding bits set"
    # (with b_k = 2 b_q two neighbouring query blocks inherit the same contribution: exact ties, which the oracle
    # reports as undecidable although both sides break them by index; identical symbols are required regardless)
    compare_symbols(ref, flags.cpu().numpy(), oracle.unpack_symbols(mask_h, Tk), f"granular L{L} {bq}x{bk} n{n}",
                    max_ambiguous=0.05 if bq >= bk else 0.2, require_identical=True)
    assert (flags.cpu().numpy()[..., : -(-text // (n * bq))] == 0).all()


@pytest.mark.parametrize("L,D,bq,bk,n,text", [(4096, 128, 128, 128, 2, 256), (3000, 64, 64, 128, 3, 200)])
def test_granular_symbols_drive_the_plan_they_were_made_for(L, D, bq, bk, n, text):
    """Update then Dispatch at granularity n: sparse_symbols_update writes exactly the arrays that
    sparse_attn_plan_create reads, and the attention they drive matches the oracle run on the oracle's own symbols
    expanded to tiles."""
    B, H = 1, 2
    tau_c, tau_kv = f32(0.4), f32(0.3)
    pool = n * max(bq, bk)
    Lp = -(-L // pool) * pool
    Q, K = synth.structured_qk(synth.BASE_SEED + 950 + L, B, H, Lp, D, n * min(bq, bk))
    Q, K = np.ascontiguousarray(Q[:, :, :L]), np.ascontiguousarray(K[:, :, :L])
    rng = np.random.default_rng(synth.BASE_SEED + 951)
    V, Oc = synth.normal_bf16(rng, Q.shape), synth.normal_bf16(rng, Q.shape)
    ref = oracle.update_symbols(Q, K, bq, text, tau_c, tau_kv, block_k=bk, granularity=n)
    flags, mask = run_gpu_granular(Q, K, bq, bk, n, text, tau_c, tau_kv)
    Tq, Tk = -(-L // bq), -(-L // bk)
    sTk = -(-L // (n * bk))
    assert (flags.cpu().numpy() == ref["cache_flags"]).all()
    assert (oracle.unpack_symbols(mask.cpu().numpy(), sTk) == ref["M_s"]).all()
    assert ref["cache_flags"].any() and not ref["cache_flags"].all()
    plan = pkg.SparseAttnPlan(flags, mask, B, H, L, bq, bk, granularity=n)
    dQ, dK, dV, dOc = up_bf16(Q), up_bf16(K), up_bf16(V), up_bf16(Oc)
    O = torch.zeros_like(dQ)
    plan.run(dQ, dK, dV, dOc, O)
    torch.cuda.synchronize()
    f, m = oracle.expand_granularity(ref["cache_flags"], ref["M_s"], n, Tq, Tk)
    ref_o, ref_bits = oracle.sparse_attention(Q, K, V, f, oracle.pack_symbols(m), Oc, bq, bk)
    got = down_bits(O)
    c = np.repeat(f != 0, bq, axis=2)[:, :, :L]
    assert (got[c] == Oc[c]).all(), "cached blocks are not bit exact"
    # The block-structured queries and keys make the softmax peaked, so outputs are single V rows of magnitude up to
    # 4 rather than averages: the bf16 rounding of the output alone is then up to 2^-7 = 7.8e-3 (half a unit in the
    # last place in [2, 4)), and the unit-variance tolerance applies relative to the magnitude of the value.
    err = np.abs(synth.bf16_bits_to_f32(got).astype(np.float64) - ref_o)[~c]
    bound = 1e-2 * np.maximum(1.0, np.abs(ref_o[~c]))
    print(f"[parity] update->dispatch at granularity {n}: max-abs {err.max():.3e} mean-abs {err.mean():.3e}", flush=True)
    assert (err <= bound).all() and err.mean() <= 1e-3
    plan.destroy()


# blocks per sequence around the register tiers of the threshold search (32, 64, 128, 272, 512; 64, 128 and 320 for the
# flags) and the 16- and 32-row tiles of the map; `repeat`: blocks that repeat, so that equal entries have to be ranked
@pytest.mark.parametrize("T,short,D,repeat", [
    (2, 0, 64, False), (16, 3, 128, False), (17, 0, 64, True), (32, 0, 128, False), (33, 20, 64, False), (64, 0, 128, True), (65, 1, 64, False),
    (128, 0, 64, False), (129, 0, 64, True), (272, 0, 64, False), (273, 63, 64, True), (320, 0, 64, False), (321, 0, 128, False),
    (512, 0, 64, True), (513, 5, 64, False)])
def test_search_tiers(T, short, D, repeat):
    B, H, block = 1, 2, 64
    L = T * block - short
    Q, K = synth.structured_qk(synth.BASE_SEED + 300 + T, B, H, T * block, D, block)
    if repeat:
        for x in (Q, K):
            v = x.reshape(B, H, T, block, D)
            v[:, :, 2::5] = v[:, :, 1:2]
    Q, K = np.ascontiguousarray(Q[:, :, :L]), np.ascontiguousarray(K[:, :, :L])
    for tau_c, tau_kv in ((f32(0.5), f32(0.3)), (f32(0.35), f32(0.7))):
        ref = oracle.update_symbols(Q, K, block, block, tau_c, tau_kv)
        flags, mask = run_gpu(Q, K, block, block, tau_c, tau_kv)
        # (blocks that repeat are near-ties for the fp64 oracle: it may order them by their last bits; it calls at most 6.6 % of
        # the entries of these shapes undecidable)
        compare(ref, flags, mask, T, f"T{T} D{D} repeat={repeat}", max_ambiguous=0.1 if repeat else 0.05, require_identical=False)


@pytest.mark.parametrize("T,D", [(20, 128), (32, 64), (33, 128), (65, 64), (129, 64), (273, 64), (321, 128), (513, 64)])
def test_equal_entries_are_taken_in_index_order_in_every_tier(T, D):
    """Q = 0: all entries of a row tie, and so do C and G: exactly the first floor(tau * count) blocks are skipped and
    cached.  The thresholds lie half an entry away from a whole number of entries."""
    B, H, block = 1, 2, 64
    _, K = synth.structured_qk(synth.BASE_SEED + 700 + T, B, H, T * block, D, block)
    for share in (0.12, 0.47):
        n_kv, n_c = int(share * T), int(share * (T - 1))
        flags, mask = run_gpu(np.zeros_like(K), K, block, block, f32((n_c + 0.5) / (T - 1)), f32((n_kv + 0.5) / T))
        bits = oracle.unpack_symbols(mask, T)
        assert (bits[..., :n_kv] == 0).all() and (bits[..., n_kv:] == 1).all()
        assert (flags[..., 0] == 0).all() and (flags[..., 1:1 + n_c] == 1).all() and (flags[..., 1 + n_c:] == 0).all()


@pytest.mark.parametrize("D,T", [(64, 3), (128, 32), (64, 33), (128, 64), (64, 65), (128, 129), (64, 273), (128, 512), (64, 513)])
def test_search_ends_early_at_the_same_place(D, T):
    """The threshold search stops where one entry is left to decide on and passes over bits that every entry agrees in: at
    thresholds from nothing to everything the skipped blocks of a row are the longest prefix of its ascending order whose
    sum fits (fp64 map; sums and order up to fp32 rounding of a row of T entries)."""
    print(f"[case] search D={D} T={T}", flush=True)
    block, text = 64, 64
    rng = np.random.default_rng(T)
    Q, K = synth.structured_qk(synth.BASE_SEED + T, 1, 2, T * block, D, block)
    K[0, 1, : (T // 2) * block] = 0                          # equal entries: half of the second head's keys are nothing
    pool = lambda x: torch.from_numpy(synth.bf16_bits_to_f32(x)).double().view(1, 2, T, block, D).mean(3)
    P = torch.softmax(pool(Q) @ pool(K).transpose(2, 3) / D ** 0.5, dim=3).numpy()
    slack = 4e-7 * T ** 0.5 + 2e-6                           # relative: exponentials, their sum, the sum of a prefix
    ascending = np.sort(P, axis=3)
    for tau in (0.0, 1e-6, 0.3 / T, 1.5 / T, float(rng.uniform(0.05, 0.3)), 0.5, float(rng.uniform(0.7, 0.99)), 0.99999, 1.0):
        tau = f32(tau)
        _, mask = run_gpu(Q, K, block, text, 0.5, tau)
        kept = oracle.unpack_symbols(mask, T).astype(bool)
        skipped = np.where(kept, 0.0, P).sum(3)
        n = (~kept).sum(3)
        assert (skipped <= tau * (1 + slack) + 1e-12).all()
        following = np.take_along_axis(ascending, np.minimum(n, T - 1)[..., None], 3)[..., 0]
        assert (np.where(n < T, skipped + following, np.inf) >= tau * (1 - slack) - 1e-12).all() or tau == 1.0
        largest = np.where(kept, 0.0, P).max(3)
        smallest = np.where(kept, P, np.inf).min(3)
        assert (largest <= smallest * (1 + 1e-5)).all()

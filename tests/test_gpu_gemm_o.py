"""GPU parity of the sparse output projection (GEMM-O) against its CPU oracle.

Bar per element: |got - ref| <= 2^-8 |ref| + 2e-3 (one bf16 rounding of the result; fp32 accumulation of
up to 3072 products of O(1) terms and the bf16 addend contribute well below the absolute term)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_25401_amd as pkg
from paper_2509_25401_amd import synth
from gpu_utils import up_bf16, up_u8, down_bits

pytestmark = pytest.mark.gpu


def _case(seed, B, H, L, D, C_out, bq, cached):
    r = np.random.default_rng(seed)
    O = synth.normal_bf16(r, (B, H, L, D))
    W = synth.f32_to_bf16_bits((r.standard_normal((C_out, H * D)) / np.sqrt(H * D)).astype(np.float32))
    bias = synth.normal_bf16(r, (C_out,))
    flags = (r.random((B, H, L // bq)) < cached).astype(np.uint8) if cached is not None else None
    return O, W, bias, flags


def _run(O, W, bias, flags, select, addend, bq, in_place=False):
    B, H, L, D = O.shape
    C_out = W.shape[0]
    Out = torch.from_numpy(np.full((B, L, C_out), 0x4242, dtype=np.uint16).view(np.int16)).view(torch.bfloat16).to("cuda:0")
    ad = None if addend is None else up_bf16(addend)
    if in_place:
        Out.copy_(ad)
        ad = Out
    pkg.sparse_gemm_o(up_bf16(O), up_bf16(W), None if bias is None else up_bf16(bias), up_u8(flags), select, ad, Out, bq)
    torch.cuda.synchronize()
    return down_bits(Out)


def _check(got_bits, ref, ref_bits, label):
    got = synth.bf16_bits_to_f32(got_bits).astype(np.float64)
    err = np.abs(got - ref)
    tol = np.abs(ref) * 2.0 ** -8 + 2e-3
    exact = (got_bits == ref_bits).mean()
    print(f"[parity] {label}: max-abs {err.max():.3e}, bit-identical to the rounded oracle: {exact * 100:.2f}%", flush=True)
    assert (err <= tol).all(), f"{label}: max violation {(err - tol).max()}"
    assert exact > 0.97


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq", [64, 128])
def test_both_stages_small_cases_all_variants(D, bq):
    print(f"[case] gemm_o small D={D} bq={bq}", flush=True)
    B, H, L, C_out = 2, 5, 384, 256
    O, W, bias, flags = _case(30 + D + bq, B, H, L, D, C_out, bq, cached=0.4)
    flags[0, :, 0] = 1            # a token block with every head cached: stage 2 is addend + bias only
    flags[1, :, 1] = 0            # and one with none cached: stage 1 is zero
    # stage 1: cached bias
    got1 = _run(O, W, None, flags, 1, None, bq)
    ref1, ref1_bits = oracle.gemm_o(O, W, None, flags, 1, None, bq)
    _check(got1, ref1, ref1_bits, f"gemm_o stage1 D={D} bq={bq}")
    assert (got1[1, bq:2 * bq] == 0).all()
    # stage 2 on top of the kernel's own cached bias
    got2 = _run(O, W, bias, flags, 0, got1, bq)
    ref2, ref2_bits = oracle.gemm_o(O, W, bias, flags, 0, got1, bq)
    _check(got2, ref2, ref2_bits, f"gemm_o stage2 D={D} bq={bq}")
    # in place: addend == Out
    assert (_run(O, W, bias, flags, 0, got1, bq, in_place=True) == got2).all()
    # Equation 3: both stages together reproduce the dense projection (up to the bf16 rounding of B_c)
    dense, _ = oracle.gemm_o(O, W, bias, None, 0, None, bq)
    err = np.abs(synth.bf16_bits_to_f32(got2).astype(np.float64) - dense)
    assert (err <= np.abs(dense) * 2.0 ** -8 + np.abs(ref1).max() * 2.0 ** -8 + 2e-3).all()


def test_dense_without_flags_and_poisoned_skipped_heads():
    print("[case] gemm_o dense / poison", flush=True)
    B, H, L, D, C_out, bq = 1, 6, 256, 128, 384, 128
    O, W, bias, flags = _case(40, B, H, L, D, C_out, bq, cached=0.5)
    got = _run(O, W, bias, None, 0, None, bq)
    ref, ref_bits = oracle.gemm_o(O, W, bias, None, 0, None, bq)
    _check(got, ref, ref_bits, "gemm_o dense")
    # NaN in every O block that stage 2 must skip: the result stays finite and unchanged
    clean = _run(O, W, bias, flags, 0, None, bq)
    Op = O.copy()
    skip = np.repeat(flags != 0, bq, axis=2)
    Op[skip] = 0x7FC0
    assert (_run(Op, W, bias, flags, 0, None, bq) == clean).all()


def test_image_dit_shape_stage2_with_config3_flags():
    print("[case] gemm_o image-DiT shape", flush=True)
    w = synth.config_image_cache_skip()
    B, H, L, D, C_out, bq = 1, w.H, w.L, w.D, 3072, w.block_q
    O, W, bias, _ = _case(41, B, H, L, D, C_out, bq, cached=None)
    Bc = synth.normal_bf16(np.random.default_rng(42), (B, L, C_out))
    got = _run(O, W, bias, w.cache_flags, 0, Bc, bq)
    ref, ref_bits = oracle.gemm_o(O, W, bias, w.cache_flags, 0, Bc, bq)
    _check(got, ref, ref_bits, "gemm_o image-DiT stage2")


@pytest.mark.parametrize("D,bq,L", [(128, 128, 1000), (64, 64, 200), (128, 64, 513), (64, 128, 90)])
def test_short_last_token_block(D, bq, L):
    """ceil(L / block_q) token blocks; nothing past token L - 1 may be read from O or the addend or written to Out."""
    rng = np.random.default_rng(70 + L)
    B, H, C = 1, 3, 256
    Tq = -(-L // bq)
    O = synth.normal_bf16(rng, (B, H, L, D))
    W = synth.f32_to_bf16_bits((rng.standard_normal((C, H * D)) / np.sqrt(H * D)).astype(np.float32))
    flags = (rng.random((B, H, Tq)) < 0.4).astype(np.uint8)
    addend = synth.normal_bf16(rng, (B, L, C))
    pad = 256
    obuf = np.full((H * L + pad, D), 0x7FC0, dtype=np.uint16)        # NaN behind the last head
    obuf[:H * L] = O.reshape(H * L, D)
    dO = up_bf16(obuf)[:H * L].view(1, H, L, D)
    abuf = np.full((L + pad, C), 0x7FC0, dtype=np.uint16)
    abuf[:L] = addend[0]
    dA = up_bf16(abuf)[:L].view(1, L, C)
    outbuf = torch.from_numpy(np.full((L + pad, C), 0x4242, dtype=np.uint16).view(np.int16)).view(torch.bfloat16).to("cuda:0")
    Out = outbuf[:L].view(1, L, C)
    for select in (0, 1):
        pkg.sparse_gemm_o(dO, up_bf16(W), None, up_u8(flags), select, dA, Out, bq)
        torch.cuda.synchronize()
        whole = down_bits(outbuf)
        assert (whole[L:] == 0x4242).all(), "rows past the end of Out were written"
        got = synth.bf16_bits_to_f32(whole[:L]).astype(np.float64)[None]
        assert np.isfinite(got).all(), "something past the end of O or the addend was read"
        ref, _ = oracle.gemm_o(O, W, None, flags, select, addend, bq)
        err = np.abs(got - ref)
        assert (err <= np.abs(ref) * 2.0 ** -8 + 2e-3).all(), f"select {select}: max violation {err.max()}"


@pytest.mark.parametrize("D,bq,n_terms,L", [(128, 128, 2, 640), (64, 64, 3, 384), (128, 128, 1, 400), (128, 64, 4, 330)])
def test_output_initialised_by_op_reuse_in_one_call(D, bq, n_terms, L):
    """sparse_gemm_o_reuse = OP_reuse(B_c) + stage 2 in one kernel: bit-identical to the two calls it replaces
    (the forecast is rounded to bf16 exactly as the element-wise kernel rounds it), and within the bar of the oracle
    that composes the two definitions.  One token block has every head cached (pure addend + bias path), the last
    block may be short."""
    print(f"[case] gemm_o fused reuse D={D} bq={bq} terms={n_terms} L={L}", flush=True)
    B, H, C_out = 2, 6, 384
    r = np.random.default_rng(700 + D + bq + n_terms)
    O = synth.normal_bf16(r, (B, H, L, D))
    W = synth.f32_to_bf16_bits((r.standard_normal((C_out, H * D)) / np.sqrt(H * D)).astype(np.float32))
    bias = synth.normal_bf16(r, (C_out,))
    Tq = -(-L // bq)
    flags = (r.random((B, H, Tq)) < 0.6).astype(np.uint8)
    flags[0, :, 1] = 1                                   # nothing selected in this token block
    terms = [synth.normal_bf16(r, (B, L, C_out)) for _ in range(n_terms)]
    coef = [float(c) for c in oracle.taylor_coefficients(n_terms - 1, 2.0)] if n_terms > 1 else [0.75]
    dO, dW, db, df = up_bf16(O), up_bf16(W), up_bf16(bias), up_u8(flags)
    dterms = [up_bf16(t) for t in terms]
    # the two calls
    fc = torch.empty_like(dterms[0])
    pkg.sparse_op_reuse(dterms, coef, fc)
    two = torch.empty_like(fc)
    pkg.sparse_gemm_o(dO, dW, db, df, 0, fc, two, bq)
    # the one call, out of place and in place (terms[0] is Out)
    one = torch.from_numpy(np.full((B, L, C_out), 0x4242, dtype=np.uint16).view(np.int16)).view(torch.bfloat16).to("cuda:0")
    pkg.sparse_gemm_o_reuse(dO, dW, db, df, dterms, coef, one, bq)
    inplace = dterms[0].clone()
    pkg.sparse_gemm_o_reuse(dO, dW, db, df, [inplace] + dterms[1:], coef, inplace, bq)
    torch.cuda.synchronize()
    assert (down_bits(one) == down_bits(two)).all(), "fused call differs from op_reuse + gemm_o"
    assert (down_bits(inplace) == down_bits(two)).all(), "in-place fused call differs"
    ref, ref_bits = oracle.gemm_o_reuse(O, W, bias, flags, terms, coef, bq)
    # The forecast is rounded to bf16 before it is added: where its fp64 value lies within fp32 rounding of a
    # rounding boundary the kernel's fp32 sum may land on the neighbouring bf16 value (as in the element-wise kernel's
    # own test), which moves the result by one unit in the last place of the forecast; everywhere else the usual bar.
    f64, _ = oracle.op_reuse(terms, coef)
    got = synth.bf16_bits_to_f32(down_bits(one)).astype(np.float64)
    err = np.abs(got - ref)
    tol = np.abs(ref) * 2.0 ** -8 + 2e-3
    loose = tol + np.abs(f64) * 2.0 ** -7
    exact = (down_bits(one) == ref_bits).mean()
    print(f"[parity] gemm_o_reuse D={D} bq={bq} terms={n_terms}: max-abs {err.max():.3e}, beyond the usual bar "
          f"{(err > tol).mean() * 100:.3f}%, bit-identical to the rounded oracle {exact * 100:.2f}%", flush=True)
    assert (err <= loose).all() and (err > tol).mean() < 2e-3 and exact > 0.97


# every tile of the dispatch at its edges: (B, H, L, D, C_out, block_q, cached share or None for no flags)
TILE_CASES = [
    (1, 1, 1, 64, 128, 64, None),            # one stage, one token
    (2, 3, 129, 128, 384, 64, None),         # 128 x 128 tiles, one token in the last
    (1, 2, 4097, 64, 2048, 128, None),       # 256 x 128 tiles (528 of 128 x 128), two stages
    (1, 3, 8191, 64, 1152, 128, None),       # 256 x 256 tiles, last column tile half full, three stages
    (1, 1, 11300, 128, 1536, 128, None),     # 256 x 256 tiles and the last token tiles done with the small ones
    (1, 64, 300, 64, 256, 128, 0.9),         # as many heads as the bitmap holds, short last block
    (2, 7, 700, 128, 384, 128, 0.7),
    (2, 7, 700, 128, 384, 64, 0.7),          # 64 x 256 tiles, last column tile half full
    (1, 5, 450, 64, 640, 64, 0.8),
    (1, 3, 6100, 64, 640, 64, 0.6),          # 64-token blocks, 288 tiles of 256 channels, the last one half full
    (1, 3, 6100, 64, 3584, 64, 0.6),         # 1344 of them: 128 channels where computed heads are selected
]


@pytest.mark.parametrize("B,H,L,D,C_out,bq,cached", TILE_CASES)
def test_every_tile_at_its_edges(B, H, L, D, C_out, bq, cached):
    """Plain, with an addend, and with one to four terms of the cached bias (where the loads of the first two are in
    flight during the reduction), for both values of the selector."""
    print(f"[case] gemm_o tiles B={B} H={H} L={L} D={D} C={C_out} bq={bq} cached={cached}", flush=True)
    O, W, bias, _ = _case(80 + L, B, H, L, D, C_out, bq, None)
    flags = None
    if cached is not None:
        flags = (np.random.default_rng(81 + L).random((B, H, -(-L // bq))) < cached).astype(np.uint8)
        flags[0, :, 0] = 1                   # a block without a computed head
        flags[0, :, -1] = 0                  # one without a cached head
    r = np.random.default_rng(82 + L)
    terms = [synth.normal_bf16(r, (B, L, C_out)) for _ in range(4)]
    for select in (0, 1):
        ref, ref_bits = oracle.gemm_o(O, W, bias, flags, select, None, bq)
        _check(_run(O, W, bias, flags, select, None, bq), ref, ref_bits, f"select {select}")
    ref, ref_bits = oracle.gemm_o(O, W, bias, flags, 0, terms[0], bq)
    _check(_run(O, W, bias, flags, 0, terms[0], bq), ref, ref_bits, "addend")
    for n in (1, 2, 3, 4):
        coef = pkg.sparse_taylor_coefficients(n - 1, 2.0)
        ref, ref_bits = oracle.gemm_o_reuse(O, W, bias, flags, terms[:n], coef, bq)
        Out = torch.zeros((B, L, C_out), dtype=torch.bfloat16, device="cuda:0")
        pkg.sparse_gemm_o_reuse(up_bf16(O), up_bf16(W), up_bf16(bias), up_u8(flags), [up_bf16(t) for t in terms[:n]], coef,
                                Out, bq)
        torch.cuda.synchronize()
        # the forecast bias is rounded to bf16 before it is added: where its fp32 sum and the oracle's fp64 sum lie on two
        # sides of a rounding boundary it differs by one step, at most 2^-7 of its size
        got = synth.bf16_bits_to_f32(down_bits(Out)).astype(np.float64)
        forecast = sum(np.abs(c * synth.bf16_bits_to_f32(t).astype(np.float64)) for c, t in zip(coef, terms))
        assert (np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + forecast * 2.0 ** -7 + 2e-3).all(), f"{n} terms"
        assert (down_bits(Out) == ref_bits).mean() > 0.97


@pytest.mark.parametrize("bq,cached", [(128, 0.6), (64, 0.6), (128, None)])
def test_bias_at_any_two_byte_address(bq, cached):
    """The bias is read in pieces of 16 bytes and needs no more than its own alignment."""
    B, H, L, D, C_out = 1, 3, 300, 64, 384
    O, W, bias, _ = _case(95, B, H, L, D, C_out, bq, None)
    flags = None if cached is None else (np.random.default_rng(96).random((B, H, -(-L // bq))) < cached).astype(np.uint8)
    if flags is not None:
        flags[0, :, 0] = 1                   # a block without a computed head
    buf = torch.zeros(C_out + 1, dtype=torch.bfloat16, device="cuda:0")
    odd = buf[1:]
    odd.copy_(up_bf16(bias))
    assert odd.data_ptr() % 4 == 2
    add = synth.normal_bf16(np.random.default_rng(97), (B, L, C_out))
    for a in (None, add):
        ref, ref_bits = oracle.gemm_o(O, W, bias, flags, 0, a, bq)
        Out = torch.zeros((B, L, C_out), dtype=torch.bfloat16, device="cuda:0")
        pkg.sparse_gemm_o(up_bf16(O), up_bf16(W), odd, up_u8(flags), 0, None if a is None else up_bf16(a), Out, bq)
        torch.cuda.synchronize()
        _check(down_bits(Out), ref, ref_bits, f"odd bias bq={bq}")

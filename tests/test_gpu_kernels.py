"""GPU: kernels and dispatch branches at the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt, make_weights
from tests._parity import CONF_TOL, PROB_RTOL, assert_logits_close, decisive, lockstep_ssd, make_pair, to_gpu

pytestmark = pytest.mark.gpu


# vocabularies around the cut of the reduction: one block per row (fewer than four slices of 1024), the fewest slices,
# ragged slices, sixteen of them; fp32 weights take the same reduction behind their own GEMM
@pytest.mark.parametrize("vocab,dtype", [(3072, "bf16"), (4096, "bf16"), (4112, "fp16"), (20016, "bf16"), (5136, "fp32")])
def test_confidence_reduction_over_vocabulary_slices(vocab, dtype):
    shape = ModelShape(3, 256, 4, 4, 704, vocab, dtype=dtype)
    orc, ctx = make_pair(shape, 21, 64, max_k=4, norm_gain_std=0.1, init_std=0.2 if dtype == "fp32" else 0.08)
    prompt = make_prompt(vocab, 20, 3).tolist()
    o = OracleSSD(orc)
    o.prefill(prompt)
    ctx.ssd_prefill(prompt)
    conf_o, det = o.layer_confidence(0)
    conf, g = ctx.ssd_layer_confidence(0, 1, detail=True)
    np.testing.assert_allclose(conf[0], conf_o, atol=CONF_TOL[dtype])
    np.testing.assert_allclose(g["maxprob"][0], det["maxprob"], rtol=PROB_RTOL[dtype] * 1.25)
    np.testing.assert_array_equal(ctx.ssd_layer_confidence(0, 1, static=True), conf)


@pytest.mark.parametrize("vocab", [512, 4112, 16400])
def test_equal_maxima_give_the_lowest_token(vocab):
    """Every row of the LM head exists twice: the greedy token of prompt, verify and decode passes is the lower one."""
    import paper_2604_14612_amd as ssd
    shape = ModelShape(2, 256, 4, 4, 704, vocab)
    w = make_weights(shape, 5)
    half = vocab // 2
    w["lm_head"][half:] = w["lm_head"][:half]
    ctx = ssd.Context(shape, to_gpu(w), 96, 8)
    for plen in (5, 40):
        ctx.ssd_reset()
        toks = [ctx.ssd_prefill(make_prompt(vocab, plen, 4).tolist())]
        d = ctx.ssd_draft_step(np.array([0, 1], np.uint8), 8)
        y = ctx.ssd_verify(d)
        toks += d + y
        z = ctx.ssd_copy_logits(0, 9)
        assert y == [int(np.argmax(r)) for r in z]
        ctx.ssd_accept(d, y)
        toks.append(ctx.ssd_decode())
        assert max(toks) < half


# Single-row attention: contexts at the edges of its position ranges (64 to 256 rows by head size and cache type, at most eight
# of them, then longer ones) and the MFMA kernel's chunks of 96 behind them; rows past the position hold NaN, as the
# kernels request whole ranges before they know it.
@pytest.mark.parametrize("heads,kv_heads,kv", [(4, 4, "fp32"), (4, 2, "bf16"), (2, 2, "fp32"), (2, 1, "fp16")])
@pytest.mark.parametrize("plen", [63, 95, 127, 255, 511, 1030])
def test_attention_ranges_at_their_edges(heads, kv_heads, kv, plen):
    shape = ModelShape(2, 256, heads, kv_heads, 704, 1024)      # head_dim 64 (4 heads) or 128 (2 heads)
    orc, ctx = make_pair(shape, 31, plen + 24, max_k=4, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(1024, plen, 7).tolist()
    o = OracleSSD(orc)
    o.prefill(prompt)
    ctx.ssd_prefill(prompt)
    for _ in range(3):
        ctx.ssd_kv_poison_stale()
        o.decode()
        t = ctx.ssd_decode()
        assert_logits_close(ctx.ssd_copy_logits(0, 1)[0], o.last_logits[0], shape.dtype, "decode")
        if t != o.tokens[-1]:
            assert not decisive(o.last_logits[0], shape.dtype)
            o.tokens[-1] = t      # a sub-tolerance tie: the oracle goes on from the library's token
    ctx.ssd_kv_poison_stale()
    zero = np.zeros(2, np.uint8)
    d = o.draft(zero, 4)
    ctx.ssd_draft_step(zero, 4)
    o.verify(d)
    ctx.ssd_verify(d)
    assert_logits_close(ctx.ssd_copy_logits(0, 5), o.last_logits, shape.dtype, "verify")


@pytest.mark.parametrize("dtype", ["bf16", "fp16", "fp32"])
def test_logits_without_a_maximum_give_a_token_that_verification_refuses(dtype):
    """One NaN weight makes every logit NaN; an infinite clamp turns them into -inf, which no arg-max picks.  The draft steps
    chain on that token: the next one must read a row of the embedding table, and the id itself is no valid draft."""
    import paper_2604_14612_amd as ssd
    shape = ModelShape(2, 256, 4, 4, 704, 1024, dtype=dtype)
    w = make_weights(shape, 5)
    w["wd"][0][7, 11] = float("nan")
    ctx = ssd.Context(shape, to_gpu(w), 96, 8, conf_clamp=float("inf"))
    none = 0x7fffffff
    assert ctx.ssd_prefill(make_prompt(1024, 20, 4).tolist()) == none
    d = ctx.ssd_draft_step(np.zeros(2, np.uint8), 6)
    assert d == [none] * 6
    assert np.isnan(ctx.ssd_copy_logits(0, 6)).all()
    with pytest.raises(ssd.SsdError):
        ctx.ssd_verify(d)


# 8208 logits are eight slices of 1026 in the confidence reduction: the first, an inner and the last one without any finite logit
@pytest.mark.parametrize("dead", [(0, 1040), (2000, 3100), (7100, 8208)])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_a_vocabulary_slice_of_minus_infinity_adds_nothing(dtype, dead):
    """NaN rows of the LM head under an infinite clamp: logits of -inf, probability 0.  Held against Eq. 1-4 over the finite
    logits of the same row (the last tap is what the prompt's logits are taken from), in 64 bits."""
    import paper_2604_14612_amd as ssd
    vocab = 8208
    shape = ModelShape(2, 256, 4, 4, 704, vocab, dtype=dtype)
    w = make_weights(shape, 5, init_std=0.08)
    w["lm_head"][dead[0]:dead[1]] = float("nan")
    ctx = ssd.Context(shape, to_gpu(w), 96, 4, conf_clamp=float("inf"))
    first = ctx.ssd_prefill(make_prompt(vocab, 20, 4).tolist())
    z = ctx.ssd_copy_logits(0, 1)[0].astype(np.float64)
    live = np.isfinite(z)
    assert (~live).sum() == dead[1] - dead[0] and first == int(np.nanargmax(z))
    p = np.exp(z[live] - z[live].max())
    p /= p.sum()
    for static in (False, True):
        conf, g = ctx.ssd_layer_confidence(0, 1, detail=True, static=static)
        assert np.isfinite(conf).all() and np.isfinite(g["maxprob"]).all()
        np.testing.assert_allclose(g["conf"][0, -1, 1], 1.0 + (p * np.log(p + 1e-10)).sum() / np.log(vocab), atol=CONF_TOL[dtype])
        np.testing.assert_allclose(g["maxprob"][0, -1, 1], p.max(), rtol=PROB_RTOL[dtype])
        assert g["argmax"][0, -1, 1] == first


def _first_layer_kv(ctx):
    """K and V of layer 0 of an fp32 cache, [KV heads][max_seq][head_dim] each: they follow the rotary table in the workspace."""
    import torch
    s, n = ctx.shape, int(ctx.cfg.max_seq)
    off = -(-n * s.head_dim * 4 // 256) * 256
    size = s.n_kv_heads * n * s.head_dim
    kv = ctx.workspace[off:off + 2 * size * 4].view(torch.float32).cpu().double()
    return [kv[i * size:(i + 1) * size].view(s.n_kv_heads, n, s.head_dim) for i in (0, 1)]


# Tiles of the QKV launch of a prompt: 192 weight rows in 200 blocks (no K cut; all rows, and a ragged last block), 192 rows cut
# along K by two (102 and 128 blocks) and by four (34), 256 rows uncut (160 blocks) and cut (30), 128 rows uncut (468) and cut (204)
@pytest.mark.parametrize("d,kv_heads,rows,dtype", [(3200, 25, 512, "bf16"), (3200, 25, 449, "fp16"), (2176, 17, 333, "bf16"), (2048, 16, 512, "bf16"),
                                                   (2176, 17, 70, "fp16"), (5120, 20, 512, "bf16"), (2048, 2, 300, "fp16"), (4992, 39, 500, "fp16"),
                                                   (2176, 17, 450, "bf16")])
def test_prompt_qkv_launch_element_by_element(d, kv_heads, rows, dtype):
    """Every cached K and V element of the first layer against 64 bits: rotate(Wk norm(x)) and Wv norm(x) of the embedding rows.
    Bound per element: activations enter as hi + lo (2^-17 relative, fp16 better) and the fp32 sums of 2 x K products add
    rounding errors that grow with the square root of their number (below 2^-17 here), both relative to the sum of the
    absolute products; four times that in all, over both rows of a rotary pair."""
    import torch
    import paper_2604_14612_amd as ssd
    shape = ModelShape(1, d, d // 128, kv_heads, 256, 1024, dtype=dtype)
    w = make_weights(shape, 9, norm_gain_std=0.1)
    ctx = ssd.Context(shape, to_gpu(w), 520, 1)
    toks = make_prompt(1024, rows, 6).tolist()
    ctx.ssd_prefill(toks)
    k, v = _first_layer_kv(ctx)
    x = w["embed"][torch.tensor(toks)].double()
    h = x * torch.rsqrt(x.square().mean(-1, keepdim=True) + shape.rms_eps) * w["attn_norm"][0].double()
    hd, half = 128, 64
    heads = lambda t: t.view(rows, kv_heads, hd).transpose(0, 1)  # noqa: E731
    mul = lambda m: (heads(h @ m.double().t()), heads(h.abs() @ m.double().abs().t()))  # noqa: E731
    ang = torch.arange(rows, dtype=torch.float64)[:, None] * shape.rope_base ** (-torch.arange(half, dtype=torch.float64) / half)
    c, s = ang.cos(), ang.sin()
    a, mag = mul(w["wk"][0])
    want_k = torch.cat([a[..., :half] * c - a[..., half:] * s, a[..., half:] * c + a[..., :half] * s], -1)
    mag_k = (mag[..., :half] + mag[..., half:]).repeat(1, 1, 2)
    want_v, mag_v = mul(w["wv"][0])
    for name, got, want, m in (("k", k, want_k, mag_k), ("v", v, want_v, mag_v)):
        err = (got[:, :rows] - want).abs() / m
        assert err.max() <= 2.0 ** -14, (name, float(err.max()))


# fp32 and untiled fp16 rows longer than one trip of the K loop (1024 and 2048 elements), with a partial last one, as K of the
# QKV / gate-up / LM-head launches (d) and of the down projection (f); one, two and the most token rows per wave
@pytest.mark.parametrize("d,heads,f,dtype", [(1152, 9, 1040, "fp32"), (1024, 8, 2064, "fp32"), (2176, 17, 2192, "fp16")])
@pytest.mark.parametrize("k", [2, 8, 15])
def test_plain_rows_over_several_trips_of_k(d, heads, f, dtype, k):
    shape = ModelShape(2, d, heads, heads, f, 1024, dtype=dtype)
    orc, ctx = make_pair(shape, 13, 64, max_k=15, norm_gain_std=0.1)
    prompt = make_prompt(1024, 21, 8).tolist()      # 16 rows, then 5
    o = OracleSSD(orc)
    o.prefill(prompt)
    ctx.ssd_prefill(prompt)
    assert_logits_close(ctx.ssd_copy_logits(0, 1)[0], o.last_logits[0], dtype, "prompt")
    zero = np.zeros(2, np.uint8)
    d_o = o.draft(zero, k)
    ctx.ssd_draft_step(zero, k)
    o.verify(d_o)
    ctx.ssd_verify(d_o)
    assert_logits_close(ctx.ssd_copy_logits(0, k + 1), o.last_logits, dtype, "verify")
    conf_o, _ = o.layer_confidence(0)
    np.testing.assert_allclose(ctx.ssd_layer_confidence(0, 1)[0], conf_o, atol=CONF_TOL[dtype])


# Single-row products whose input is longer than what a block requests in front of its weights (8192 elements of a normalised one, 4096 at
# the LM head and where attention partials are folded, 14336 of the FFN's), and shorter than one piece per thread.
@pytest.mark.parametrize("shape,plen", [(ModelShape(1, 4352, 34, 2, 512, 528), 70), (ModelShape(1, 8448, 66, 2, 256, 528, dtype="fp16"), 5),
                                        (ModelShape(1, 1088, 17, 17, 14464, 528), 5), (ModelShape(1, 704, 11, 11, 14464, 528, dtype="fp32"), 70),
                                        (ModelShape(2, 1152, 9, 3, 320, 528, dtype="fp16"), 150)],
                         ids=["fold", "norm", "ffn", "ffn32", "short"])
def test_products_of_a_single_row(shape, plen):
    orc, ctx = make_pair(shape, 13, plen + 12, max_k=3, norm_gain_std=0.1)
    prompt = make_prompt(shape.vocab, plen, 5).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [3, 1], np.zeros(shape.n_layers, np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 3
    assert ctx.ssd_get_one_launch() == (0, 0, 0)


# Verifications on the matrix-core attention: fewer rows than a wave's four queries, groups that fill several blocks of 16, heads of 64
# (four of eight waves have output dims), contexts that end inside the first position tile, at the chunk's end and one behind it.
@pytest.mark.parametrize("heads,kv_heads,kv", [(10, 10, "fp32"), (10, 2, "bf16"), (20, 20, "bf16"), (20, 4, "fp32")])
@pytest.mark.parametrize("plen", [11, 91, 92, 187])
def test_attention_of_a_verification(heads, kv_heads, kv, plen):
    shape = ModelShape(2, 1280, heads, kv_heads, 192, 528)      # head_dim 128 (10 heads) or 64 (20 heads)
    orc, ctx = make_pair(shape, 17, plen + 40, max_k=7, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 7).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [4, 7], np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1
    assert ctx.ssd_get_one_launch() == (0, 0, 0)


# Folds of many attention partials: two ranges, the eight that are requested together, nine and more, with rows whose first ranges are all
# there is (the last ranges of a chunked context are empty for earlier rows), in one launch and -- replayed -- one after the other
@pytest.mark.parametrize("kv", ["fp32", "bf16"])
@pytest.mark.parametrize("plen", [95, 190, 760, 772, 1250])
def test_partials_folded_by_the_last_block(kv, plen):
    shape = ModelShape(2, 1280, 10, 5, 192, 528)
    orc, ctx = make_pair(shape, 19, plen + 40, max_k=7, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 7).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [7, 7, 7, 2], np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 2


# Single rows over contexts long enough for more ranges than the output projection folds: heads in groups of four and alone, both sides of the
# rule, more ranges than one share of the fold takes, ranges made longer because there would be more than blocks (22 of 80 positions, 23 of
# 144), 16-bit caches
@pytest.mark.parametrize("heads,kv_heads,plen,kv", [(20, 5, 1530, "fp32"), (20, 5, 2950, "fp32"), (20, 20, 1530, "fp32"), (10, 10, 1300, "fp32"), (10, 5, 1700, "fp32"),
                                                    (10, 10, 1700, "fp32"), (10, 5, 1700, "bf16"), (20, 5, 3400, "bf16"), (10, 10, 3220, "bf16")])
def test_single_rows_fold_many_ranges(heads, kv_heads, plen, kv):
    shape = ModelShape(1, 1280, heads, kv_heads, 192, 528)
    orc, ctx = make_pair(shape, 23, plen + 24, max_k=8, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 7).tolist()
    o = OracleSSD(orc)
    o.prefill(prompt)
    ctx.ssd_prefill(prompt)
    for i in range(3):                      # kernel by kernel, captured, replayed
        o.decode()
        got = ctx.ssd_decode()
        assert_logits_close(ctx.ssd_copy_logits(0, 1)[0], o.last_logits[0], shape.dtype, "decode %d" % i)
        if got != o.tokens[-1]:
            assert not decisive(o.last_logits[0], shape.dtype)
            break

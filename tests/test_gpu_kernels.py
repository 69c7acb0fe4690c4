"""GPU: kernels and dispatch branches at the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt, make_weights
from tests._parity import CONF_TOL, PROB_RTOL, assert_logits_close, make_pair, to_gpu

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
            return      # a sub-tolerance tie: the sequences part
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

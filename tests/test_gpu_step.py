"""GPU: single-row steps and verifications of narrow models as one launch, at the edges of their rules (csrc/ssd_rules.h:
step_blocks, rows_step_fits), against the CPU oracle.  Every test states how many of its calls are to run so."""
import threading

import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt, make_weights
from tests._parity import assert_logits_close, decisive, lockstep_ssd, make_pair, to_gpu

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_head": (ModelShape(2, 64, 1, 1, 48, 272), "fp32"),                         # 64 blocks, one row of everything
    "widest": (ModelShape(2, 1024, 8, 2, 3072, 4112), "fp32"),                      # the registers of a wave are full
    "widest16": (ModelShape(2, 1024, 16, 4, 3072, 528, dtype="fp16"), "fp16"),
    "odd": (ModelShape(3, 960, 15, 5, 1040, 496), "bf16"),                          # 15 heads in groups of three, ragged shares
    "wide_ffn": (ModelShape(2, 512, 8, 8, 3088, 528), "fp32"),                      # 16 FFN columns too many: launches per matrix
    "widest32": (ModelShape(2, 512, 8, 8, 1536, 1040, dtype="fp32"), "fp32"),
    "group8": (ModelShape(2, 512, 8, 1, 1408, 528), "fp32"),                        # eight query heads per KV head: steps by a launch per matrix
}
STEPS_PER_MATRIX, VERIFICATIONS_PER_MATRIX = ("wide_ffn", "group8"), ("wide_ffn",)


def one_launch_verifications(shape, kv, plen, ks, accepted):
    """How many of these cycles' verifications fit: two to nine rows, 128 KB of keys per head."""
    n, count = plen + 1, 0
    for k, a in zip(ks, accepted):
        count += k + 1 <= 9 and (n + k) * shape.head_dim * (4 if kv == "fp32" else 2) <= 128 * 1024
        n += a + 1
    return count


@pytest.mark.parametrize("name", sorted(SHAPES))
@pytest.mark.parametrize("plen", [1, 130])
def test_drafts_and_verification_at_the_limits(name, plen):
    shape, kv = SHAPES[name]
    orc, ctx = make_pair(shape, 31, plen + 40, max_k=6, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 6).tolist()
    mask = np.zeros(shape.n_layers, np.uint8)
    mask[1] = 1
    st = lockstep_ssd(ctx, orc, prompt, 0, [6, 1, 4], mask, shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 5
    verifications = 0 if name in VERIFICATIONS_PER_MATRIX else 2 if name == "widest16" and plen == 1 else 3   # (seven rows of fp16 over 8 positions)
    assert ctx.ssd_get_one_launch() == (0 if name in STEPS_PER_MATRIX else 11, verifications, 0)


# rows of a verification around what the kernel is compiled for (3, 5, 9; 10 take the launches per matrix), contexts of one pass over
# the cache, several passes, just below the longest one (128 KB of keys: 512 rows of 64 fp32 values, 1024 of 16 bits) and on both sides of it
@pytest.mark.parametrize("kv,plen", [("fp32", 1), ("fp32", 300), ("fp32", 490), ("fp32", 500), ("bf16", 700), ("bf16", 1003), ("bf16", 1012)])
def test_verification_of_two_to_ten_rows(kv, plen):
    shape = ModelShape(2, 512, 8, 2, 1408, 528)
    orc, ctx = make_pair(shape, 11, plen + 70, max_k=9, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 6).tolist()
    ks = [8, 1, 2, 3, 4, 5, 7, 9]
    st = lockstep_ssd(ctx, orc, prompt, 0, ks, np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 20
    fit = one_launch_verifications(shape, kv, plen, ks, st["accepted"])
    assert 3 <= fit < 7 if plen in (500, 1012) else fit == 7
    assert ctx.ssd_get_one_launch() == (sum(ks), fit, 0)


def test_verification_with_128_wide_heads_and_nine_rows():
    shape = ModelShape(2, 1024, 8, 2, 3072, 528)    # LDS and the registers are full
    orc, ctx = make_pair(shape, 12, 300, max_k=8, norm_gain_std=0.1)
    prompt = make_prompt(shape.vocab, 230, 6).tolist()   # up to 256 positions of 128 fp32 values
    ks = [8, 8, 6, 8]
    st = lockstep_ssd(ctx, orc, prompt, 0, ks, np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 14
    fit = one_launch_verifications(shape, "fp32", 230, ks, st["accepted"])
    assert fit >= 2 and ctx.ssd_get_one_launch() == (sum(ks), fit, 0)


@pytest.mark.parametrize("kv", ["fp32", "bf16"])
@pytest.mark.parametrize("plen", [511, 1300])    # up to eight ranges of one pass; longer ranges, several passes
def test_decoding_over_several_ranges(kv, plen):
    shape = ModelShape(2, 256, 4, 2, 688, 528)
    orc, ctx = make_pair(shape, 7, plen + 12, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 6).tolist()
    o = OracleSSD(orc)
    assert ctx.ssd_prefill(prompt) == o.prefill(prompt)
    for step in range(6):
        t_o, t_g = o.decode(), ctx.ssd_decode()
        assert_logits_close(ctx.ssd_copy_logits(0, 1)[0], o.last_logits[0], shape.dtype, "step %d" % step)
        assert t_g == t_o
    assert ctx.ssd_get_one_launch() == (6, 0, 0)


def test_two_contexts_decode_at_the_same_time():
    """Only one such launch may be in flight per device and process: a call that finds the other context's takes the launches
    per matrix, no wait gives up, and the results are those of a context alone -- to the last bits, which depend on the
    path, so that a token may differ where its margin is below the tolerance; what follows has other inputs then."""
    import torch
    import paper_2604_14612_amd as ssd
    shape = ModelShape(6, 512, 8, 8, 1408, 2048)
    w = to_gpu(make_weights(shape, 3, norm_gain_std=0.1))
    torch.cuda.synchronize()
    prompts = [make_prompt(shape.vocab, 20, s).tolist() for s in (1, 2)]

    def decode(ctx, prompt):
        tokens, logits = [ctx.ssd_prefill(prompt)], []
        for _ in range(100):
            tokens.append(ctx.ssd_decode())
            logits.append(ctx.ssd_copy_logits(0, 1)[0].astype(np.float64))
        return tokens, logits, ctx.ssd_get_one_launch()

    alone = [decode(ssd.Context(shape, w, 160, 1), p) for p in prompts]
    assert [a[2] for a in alone] == [(100, 0, 0)] * 2
    got, errors = [None, None], []

    def run(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                got[i] = decode(ssd.Context(shape, w, 160, 1), prompts[i])
        except Exception as e:      # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert sum(g[2][0] for g in got) >= 100 and all(g[2][2] == 0 for g in got), [g[2] for g in got]
    for (tokens, logits, _), (ref_tokens, ref_logits, _) in zip(got, alone):
        assert tokens[0] == ref_tokens[0]
        for step in range(100):
            assert_logits_close(logits[step], ref_logits[step], shape.dtype, "step %d" % step)
            if tokens[step + 1] != ref_tokens[step + 1]:
                assert not decisive(ref_logits[step], shape.dtype), step
                break

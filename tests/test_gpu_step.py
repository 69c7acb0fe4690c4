"""GPU: single-row steps of narrow models as one launch, at the edges of its rule (csrc/ssd_rules.h: step_blocks), against the
CPU oracle."""
import threading

import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt, make_weights
from tests._parity import assert_logits_close, lockstep_ssd, make_pair, to_gpu

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_head": (ModelShape(2, 64, 1, 1, 48, 272), "fp32"),                         # 64 blocks, one row of everything
    "widest": (ModelShape(2, 1024, 8, 2, 3072, 4112), "fp32"),                      # the registers of a wave are full
    "widest16": (ModelShape(2, 1024, 16, 4, 3072, 528, dtype="fp16"), "fp16"),
    "odd": (ModelShape(3, 960, 15, 5, 1040, 496), "bf16"),                          # 15 heads in groups of three, ragged shares
    "wide_ffn": (ModelShape(2, 512, 8, 8, 3088, 528), "fp32"),                      # 16 FFN columns too many: launches per matrix
    "widest32": (ModelShape(2, 512, 8, 8, 1536, 1040, dtype="fp32"), "fp32"),
    "group8": (ModelShape(2, 512, 8, 1, 1408, 528), "fp32"),                        # eight query heads per KV head: launches per matrix
}


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


# rows of a verification around what the kernel is compiled for (3, 5, 9; 10 take the launches per matrix), contexts of one pass over
# the cache, several passes, and on both sides of the longest one (128 KB of keys: 512 rows of 64 fp32 values, 1024 of 16 bits)
@pytest.mark.parametrize("kv,plen", [("fp32", 1), ("fp32", 300), ("fp32", 490), ("bf16", 700), ("bf16", 1003)])
def test_verification_of_two_to_ten_rows(kv, plen):
    shape = ModelShape(2, 512, 8, 2, 1408, 528)
    orc, ctx = make_pair(shape, 11, plen + 70, max_k=9, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 6).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [8, 1, 2, 3, 4, 5, 7, 9], np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 20


def test_verification_with_128_wide_heads_and_nine_rows():
    shape = ModelShape(2, 1024, 8, 2, 3072, 528)    # LDS and the registers are full
    orc, ctx = make_pair(shape, 12, 300, max_k=8, norm_gain_std=0.1)
    prompt = make_prompt(shape.vocab, 230, 6).tolist()   # up to 256 positions of 128 fp32 values
    st = lockstep_ssd(ctx, orc, prompt, 0, [8, 8, 6, 8], np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["draft_rows"] >= 14


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


def test_two_contexts_decode_at_the_same_time():
    """Only one such launch may be in flight per device: the other context falls back to the launches per matrix and the
    tokens are those of a context alone."""
    import torch
    import paper_2604_14612_amd as ssd
    shape = ModelShape(6, 512, 8, 8, 1408, 2048)
    w = to_gpu(make_weights(shape, 3, norm_gain_std=0.1))
    torch.cuda.synchronize()
    prompts = [make_prompt(shape.vocab, 20, s).tolist() for s in (1, 2)]
    alone = []
    for p in prompts:
        alone.append(ssd.generate_vanilla(ssd.Context(shape, w, 160, 1), p, 100))
    got, errors = [None, None], []

    def run(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                got[i] = ssd.generate_vanilla(ssd.Context(shape, w, 160, 1), prompts[i], 100)
        except Exception as e:      # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert got == alone

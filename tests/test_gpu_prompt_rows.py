"""GPU: the epilogue of the 64-column groups of prompt GEMMs (what is shared by a wave's rows is worked out once) where rows and
groups end inside a batch, against the CPU oracle: the cache rows a prompt wrote are read by the cycle behind it."""
import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt
from tests._parity import CONF_TOL, assert_logits_close, decisive, lockstep_ssd, make_pair

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": ModelShape(2, 768, 12, 4, 1408, 528),                       # two heads per 128 columns, 192-row QKV tiles
    "hd128": ModelShape(2, 768, 6, 2, 1408, 528, dtype="fp16"),
}


@pytest.mark.parametrize("name", sorted(SHAPES))
@pytest.mark.parametrize("kv", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("plen", [17, 65, 191, 321])
def test_cache_rows_of_a_prompt(name, kv, plen):
    shape = SHAPES[name]
    if kv != "fp32" and kv != shape.dtype:
        pytest.skip("the other 16-bit type: covered for bf16 weights elsewhere")
    orc, ctx = make_pair(shape, 5, plen + 16, max_k=4, norm_gain_std=0.1, kv_dtype=kv)
    prompt = make_prompt(shape.vocab, plen, 3).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [4], np.array([0, 1], np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["verify_rows"] == 5


# The last layer of a prompt block leaves keys and values of all rows and the rest for the last row only: one layer and several, the
# 64-row blocks of shapes outside the large tiles, last blocks of one row, of 16 (the 16-row path behind a block of 512) and of more.
@pytest.mark.parametrize("shape", [ModelShape(1, 512, 4, 4, 1408, 528), ModelShape(2, 256, 4, 1, 704, 640, dtype="fp16"),
                                   ModelShape(2, 256, 2, 2, 640, 576), ModelShape(3, 192, 3, 1, 336, 528, dtype="fp32"),
                                   ModelShape(1, 256, 2, 2, 688, 528, dtype="fp32"), ModelShape(2, 256, 2, 1, 688, 528, dtype="fp16")],
                         ids=["one_layer", "gqa", "blocks_of_64", "fp32", "fp32_one_layer", "fp16_untiled"])
@pytest.mark.parametrize("plen", [17, 64, 65, 80, 81, 513, 530])
def test_last_layer_of_a_prompt(shape, plen):
    orc, ctx = make_pair(shape, 9, plen + 16, max_k=4, norm_gain_std=0.1, init_std=0.08)
    prompt = make_prompt(shape.vocab, plen, 3).tolist()
    o = OracleSSD(orc)
    assert ctx.ssd_prefill(prompt) == o.prefill(prompt) or not decisive(o.last_logits[0], shape.dtype)
    assert_logits_close(ctx.ssd_copy_logits(0, 1)[0], o.last_logits[0], shape.dtype, "prompt")
    np.testing.assert_allclose(ctx.ssd_layer_confidence(0, 1)[0], o.layer_confidence(0)[0], atol=CONF_TOL[shape.dtype])
    ctx.ssd_reset()
    st = lockstep_ssd(ctx, orc, prompt, 0, [4, 1], np.zeros(shape.n_layers, np.uint8), shape.dtype)   # reads the cache rows
    assert st["unpinned_cycles"] <= 1


# K slices of unequal length and more blocks than slots: 20 and 53 stripes of K, an odd number of 128-row tiles
@pytest.mark.parametrize("shape", [ModelShape(2, 1280, 10, 2, 3392, 640), ModelShape(2, 1152, 9, 9, 3392, 640, dtype="fp16")], ids=["gqa", "mha"])
def test_uneven_k_slices(shape):
    orc, ctx = make_pair(shape, 9, 320, max_k=2, norm_gain_std=0.1, init_std=0.03)
    prompt = make_prompt(shape.vocab, 300, 3).tolist()
    st = lockstep_ssd(ctx, orc, prompt, 0, [2], np.zeros(shape.n_layers, np.uint8), shape.dtype)
    assert st["unpinned_cycles"] <= 1 and st["verify_rows"] == 3

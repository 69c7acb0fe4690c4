"""GPU: one-launch steps and verifications whose waits give up, because the launch lacks a block (a negative bound).  The other
blocks drain by themselves, nothing of them may be committed, and the call's results are those of the launches per matrix."""
import numpy as np
import pytest

from oracle import OracleSSD
from synth import ModelShape, make_prompt
from tests._parity import assert_logits_close, make_pair

pytestmark = pytest.mark.gpu

SHAPES = {
    "grouped": (ModelShape(6, 512, 8, 2, 1408, 528, dtype="fp32"), "fp32"),
    "plain": (ModelShape(4, 256, 4, 4, 688, 1024, dtype="fp32"), "fp32"),
}


# graphs: how the launches per matrix that do the work again are enqueued (steps in one launch are launched as they are)
@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_calls_that_give_up_return_the_results_of_the_other_path(name, graphs):
    shape, kv = SHAPES[name]
    orc, ctx = make_pair(shape, 21, 128, max_k=4, norm_gain_std=0.1, kv_dtype=kv)
    ctx.ssd_set_graphs(graphs)
    o = OracleSSD(orc)
    prompt = make_prompt(shape.vocab, 40, 6).tolist()
    assert ctx.ssd_prefill(prompt) == o.prefill(prompt)
    mask = np.zeros(shape.n_layers, np.uint8)
    mask[1] = 1
    calls = 0

    def call(fn):
        nonlocal calls
        ctx.ssd_set_one_launch(True, -1)      # one launch again, whatever the call before did
        calls += 1
        return fn()

    def rows(n, ref, what):
        z = ctx.ssd_copy_logits(0, n)
        for j in range(n):
            assert_logits_close(z[j], ref[j], shape.dtype, "%s row %d" % (what, j))

    for rnd in range(4):                      # the other path: kernel by kernel, captured, replayed twice
        d = call(lambda: ctx.ssd_draft_step(mask, 3))
        assert d == o.draft(mask, 3), rnd
        rows(3, o.last_draft_logits, "draft %d" % rnd)
        y = call(lambda: ctx.ssd_verify(d))
        assert y == o.verify(d), rnd
        rows(4, o.last_logits, "verify %d" % rnd)
        assert ctx.ssd_accept(d, y) == o.accept(d, y)
        ctx.ssd_kv_poison_stale()
        assert call(ctx.ssd_decode) == o.decode(), rnd
        rows(1, o.last_logits, "decode %d" % rnd)
        d, _ = call(lambda: ctx.ssd_draft_adaptive(mask, 2, 0.0))
        assert d == o.draft(mask, 2), rnd
        y = call(lambda: ctx.ssd_verify(d))
        assert y == o.verify(d), rnd
        rows(3, o.last_logits, "second verify %d" % rnd)
        assert ctx.ssd_accept(d, y) == o.accept(d, y)
        assert ctx.ssd_get_stats()["n_tokens"] == o.n
    steps, verifications, gave_up = ctx.ssd_get_one_launch()
    assert (steps, verifications, gave_up) == (0, 0, calls)
    # with the usual bound the same context goes on in one launch per step
    ctx.ssd_set_one_launch(True)
    for _ in range(3):
        assert ctx.ssd_decode() == o.decode()
        rows(1, o.last_logits, "behind")
    d = ctx.ssd_draft_step(mask, 3)
    assert d == o.draft(mask, 3) and ctx.ssd_verify(d) == o.verify(d)
    rows(4, o.last_logits, "verify behind")
    assert ctx.ssd_get_one_launch() == (steps + 6, verifications + 1, gave_up)


def test_requests_of_a_context_whose_launches_keep_giving_up():
    """Every request of a context that cannot have all CUs used to wait its bound out once."""
    shape, kv = SHAPES["plain"]
    orc, ctx = make_pair(shape, 21, 64, norm_gain_std=0.1, kv_dtype=kv)
    ctx.ssd_set_one_launch(True, -1)
    prompt = make_prompt(shape.vocab, 8, 6).tolist()
    o = OracleSSD(orc)
    want = [o.prefill(prompt)] + [o.decode() for _ in range(3)]
    for _ in range(100):
        assert [ctx.ssd_prefill(prompt)] + [ctx.ssd_decode() for _ in range(3)] == want
        ctx.ssd_reset()
    steps, _, gave_up = ctx.ssd_get_one_launch()
    assert steps == 0 and 4 <= gave_up <= 7

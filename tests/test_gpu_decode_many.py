"""GPU: decode steps that are waited for together give what as many single ones give."""
import threading

import numpy as np
import pytest

from synth import ModelShape, make_prompt, make_weights
from tests._parity import to_gpu

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_launch": (ModelShape(2, 256, 4, 2, 688, 528, dtype="fp32"), True),    # each step one launch
    "per_matrix": (ModelShape(2, 1280, 10, 2, 192, 528), False),
    "untiled": (ModelShape(2, 1088, 17, 17, 176, 528, dtype="fp16"), False),
    "one_launch_off": (ModelShape(2, 256, 4, 2, 688, 528, dtype="fp32"), False),
}
# replayed or launched makes a difference to the launches per matrix only
CASES = [("one_launch", True)] + [(name, graphs) for name in ("one_launch_off", "per_matrix", "untiled") for graphs in (True, False)]


# one step, two, whole batches of 32 and what is left over; positions that cross a change of attention's plan; the sequence full before the
# count, on its last position and with the rotary row behind it outside the table
@pytest.mark.parametrize("name,graphs", CASES)
@pytest.mark.parametrize("plen,count,room", [(1, 1, 5), (60, 2, 3), (60, 32, 40), (50, 70, 70), (118, 33, 33), (30, 40, 10), (30, 34, 1)])
def test_same_as_single_steps(name, graphs, plen, count, room):
    import paper_2604_14612_amd as ssd
    shape, one_launch = SHAPES[name]
    max_seq = plen + 1 + room          # committed tokens after the prompt: plen + 1
    ctx = ssd.Context(shape, to_gpu(make_weights(shape, 7, init_std=0.08)), max_seq, 4)
    ctx.ssd_set_graphs(graphs)
    ctx.ssd_set_one_launch(name != "one_launch_off")
    prompt = make_prompt(shape.vocab, plen, 3).tolist()
    want, fit = [], min(count, room)
    ctx.ssd_prefill(prompt)
    for _ in range(fit):
        want.append(ctx.ssd_decode())
    z, stats = ctx.ssd_copy_logits(0, 1), ctx.ssd_get_stats()
    for rep in range(3):               # kernel by kernel, captured, replayed; steps in one launch are launched each time
        before = ctx.ssd_get_one_launch()
        ctx.ssd_reset()
        ctx.ssd_prefill(prompt)
        if fit < count:
            with pytest.raises(ssd.SsdError) as e:
                ctx.ssd_decode_many(count)
            assert e.value.code == ssd.SSD_ECAPACITY
            assert ctx.ssd_get_stats()["n_tokens"] == max_seq
        else:
            assert ctx.ssd_decode_many(count) == want
        np.testing.assert_array_equal(ctx.ssd_copy_logits(0, 1), z)
        assert ctx.ssd_get_stats() == stats
        after = ctx.ssd_get_one_launch()
        assert after[0] - before[0] == (fit if one_launch else 0) and after[2] == 0
    if fit == count:                   # the calls go on from there as they do behind single steps
        assert ssd.generate_vanilla(_again(ctx), prompt, count + 1)[1:] == want


def _again(ctx):
    ctx.ssd_reset()
    return ctx


@pytest.mark.parametrize("name", ["one_launch", "per_matrix"])
def test_contexts_beside_each_other(name):
    """Steps are waited for one by one then, and the slot of the one-launch steps goes from hand to hand."""
    import paper_2604_14612_amd as ssd
    shape = SHAPES[name][0]
    ctxs = [ssd.Context(shape, to_gpu(make_weights(shape, 7 + i, init_std=0.08)), 400, 4) for i in range(2)]
    prompt = make_prompt(shape.vocab, 20, 3).tolist()
    want = [ssd.generate_vanilla(c, prompt, 300) for c in ctxs]
    got = [None, None]

    def run(i):
        for _ in range(3):
            got[i] = ssd.generate_vanilla(_again(ctxs[i]), prompt, 300)
    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == want
    assert all(c.ssd_get_stats()["n_tokens"] == 320 and c.ssd_get_one_launch()[2] == 0 for c in ctxs)


def test_bad_arguments_and_order():
    import paper_2604_14612_amd as ssd
    shape = SHAPES["one_launch"][0]
    ctx = ssd.Context(shape, to_gpu(make_weights(shape, 7)), 32, 4)
    with pytest.raises(ssd.SsdError) as e:
        ctx.ssd_decode_many(2)
    assert e.value.code == ssd.SSD_ESTATE
    ctx.ssd_prefill([1, 2, 3])
    with pytest.raises(ssd.SsdError) as e:
        ctx.ssd_decode_many(0)
    assert e.value.code == ssd.SSD_EINVAL
    ctx.ssd_draft_step(np.zeros(2, np.uint8), 2)
    with pytest.raises(ssd.SsdError) as e:
        ctx.ssd_decode_many(2)
    assert e.value.code == ssd.SSD_ESTATE


def test_steps_that_give_up():
    """Every one-launch step lacks a block: the first of a batch gives up, nothing behind it is committed, and the batch is done again."""
    import paper_2604_14612_amd as ssd
    shape = ModelShape(2, 256, 4, 2, 688, 528, dtype="fp32")
    ctx = ssd.Context(shape, to_gpu(make_weights(shape, 7, init_std=0.08)), 80, 4)
    prompt = make_prompt(shape.vocab, 20, 3).tolist()
    ctx.ssd_set_one_launch(False)
    want = ssd.generate_vanilla(ctx, prompt, 12)
    z = ctx.ssd_copy_logits(0, 1)
    ctx.ssd_set_one_launch(True, -1)
    for rep in range(2):
        ctx.ssd_set_one_launch(True, -1)    # (forgets the wait that gave up)
        ctx.ssd_reset()
        assert ssd.generate_vanilla(ctx, prompt, 12) == want
        np.testing.assert_array_equal(ctx.ssd_copy_logits(0, 1), z)
        assert ctx.ssd_get_one_launch() == (0, 0, rep + 1)

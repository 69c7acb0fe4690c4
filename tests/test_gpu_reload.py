"""GPU: a context that is given other weights, or another workspace, behind a reset.  Its launch sequences were captured with
the earlier pointers by then; what follows has to equal a fresh context bit for bit."""
import ctypes as C

import numpy as np
import pytest

from paper_2604_14612_amd.binding import ssd_weights
from synth import ModelShape, make_prompt, make_weights
from tests._parity import to_gpu

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_launch": (ModelShape(3, 512, 8, 8, 1408, 528), "fp32"),        # steps and verifications in one launch
    "per_matrix": (ModelShape(2, 512, 8, 8, 3088, 528), "fp32"),        # FFN too wide for those
}


def _request(ctx, shape, seed):
    """A prompt, two cycles, three decoded tokens: everything a caller sees of them."""
    out = [ctx.ssd_prefill(make_prompt(shape.vocab, 20, seed).tolist())]
    mask = np.zeros(shape.n_layers, np.uint8)
    mask[1] = 1
    for _ in range(2):
        d, prob = ctx.ssd_draft_step(mask, 3, want_maxprob=True)
        y = ctx.ssd_verify(d)
        out += [d, prob, y, ctx.ssd_copy_logits(0, 4).tolist(), ctx.ssd_layer_confidence(0, 4).tolist(), ctx.ssd_accept(d, y)]
    for _ in range(3):
        out += [ctx.ssd_decode(), ctx.ssd_copy_logits(0, 1).tolist()]
    ctx.ssd_reset()
    return out


def _requests(ctx, shape):
    """Four of them: kernel by kernel, captured, replayed twice."""
    return [_request(ctx, shape, s) for s in (5, 5, 6, 5)]


def _differing(a, b):
    """(request, item) of what differs; short, so that a failure does not print whole logits."""
    return [(i, j) for i in range(len(a)) for j in range(len(a[i])) if a[i][j] != b[i][j]]


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_other_weights_behind_a_reset(name):
    import paper_2604_14612_amd as ssd
    shape, kv = SHAPES[name]
    first, second = (to_gpu(make_weights(shape, s, norm_gain_std=0.1)) for s in (1, 2))
    ctx, fresh = ssd.Context(shape, first, 64, 4, kv_dtype=kv), ssd.Context(shape, second, 64, 4, kv_dtype=kv)
    before = _requests(ctx, shape)
    want = _requests(fresh, shape)
    assert _differing(before, want)
    arr = lambda n: C.cast(fresh._arrs[n], C.POINTER(C.c_void_p))  # noqa: E731
    w = ssd_weights(second["embed"].data_ptr(), second["lm_head"].data_ptr(), second["final_norm"].data_ptr(),
                    *(arr(n) for n in ("attn_norm", "wq", "wk", "wv", "wo", "mlp_norm", "wg", "wu", "wd")))
    ctx._check(ctx._l.ssd_load_weights(ctx._h, C.byref(w)))
    assert _differing(_requests(ctx, shape), want) == []


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_another_workspace_behind_a_reset(name):
    import torch
    import paper_2604_14612_amd as ssd
    shape, kv = SHAPES[name]
    ctx = ssd.Context(shape, to_gpu(make_weights(shape, 1, norm_gain_std=0.1)), 64, 4, kv_dtype=kv)
    want = _requests(ctx, shape)
    torch.cuda.synchronize()
    old = ctx.workspace
    old_bytes = old.clone()
    ctx.workspace = torch.zeros_like(old)
    torch.cuda.synchronize()
    ctx._check(ctx._l.ssd_set_workspace(ctx._h, C.c_void_p(ctx.workspace.data_ptr()), ctx.workspace.numel()))
    assert _differing(_requests(ctx, shape), want) == []
    torch.cuda.synchronize()
    assert torch.equal(old, old_bytes), "the earlier workspace was written"

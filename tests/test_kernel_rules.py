"""CPU: the integer rules of csrc/ssd_rules.h (who writes what, which index is read), compiled for the host and enumerated."""
import ctypes as C
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_14612_amd", "csrc")

WRAPPERS = r"""
#include "ssd_rules.h"
using namespace ssdk;
extern "C" {
int k_slices_of(int blocks, int slots, int stripes, double slice_bytes, int most) { return ssdk::k_slices(blocks, slots, stripes, slice_bytes, most); }
void attention_plan(int G, int Hkv, int hd, int kv_f32, int w_f32, int ctx, int M, int* out) {
    const AttnPlan p = attn_plan(AttnShape{G, Hkv, hd, kv_f32 != 0, w_f32 != 0}, ctx, M, 0, 0);
    out[0] = p.wide; out[1] = p.n_splits; out[2] = p.chunk;
}
void attention_plan_many(int G, int Hkv, int hd, int kv_f32, int w_f32, int ctx, int* out) {
    const AttnPlan p = attn_plan_many(AttnShape{G, Hkv, hd, kv_f32 != 0, w_f32 != 0}, ctx, 0, 0);
    out[0] = p.wide; out[1] = p.n_splits; out[2] = p.chunk;
}
int qkv_tile(int n_total, int m_blocks) { return qkv_tile_rows(n_total, m_blocks); }
int draft_ctx(int n, int k) { return draft_plan_ctx(n, k); }
size_t embedding_row(int tok, int V) { return embed_row(tok, V); }
int row_writers(int row) { int n = 0; for (int w = 0; w < 8; w++) rows_of_wave(w, [&](int c) { n += c == row; }); return n; }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("rules")
    src, lib = str(d / "rules.cpp"), str(d / "librules.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, "-o", lib, src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    l = C.CDLL(lib)
    l.embedding_row.restype = C.c_size_t
    return l


def kernel_source(name):
    """The body of kernel `name` in ssd_kernels.hip, comments taken out."""
    text = open(os.path.join(CSRC, "ssd_kernels.hip")).read()
    text = re.sub(r"//[^\n]*", "", text)
    a = re.search(r"void %s\(" % name, text).start()
    return text[a:text.index("\n}\n", a)]


def test_every_row_scale_of_the_16_row_kernel_has_one_writer(rules):
    """Two writers without a barrier between them leave the scale to chance: the 1 of one may land on the factor of the other."""
    assert [rules.row_writers(c) for c in range(-1, 17)] == [0] + [1] * 16 + [0]
    assert len(re.findall(r"\brs\[[^]]*\]\s*=[^=]", kernel_source("rows_mfma3_kernel"))) == 1


def test_single_row_products_request_their_first_weights_before_they_wait():
    """A value that goes to LDS in front of the first requests is waited for in front of them (loads return in order)."""
    src = kernel_source("gemv_kernel")
    first = src.index("for (int s = 0; s < D; s++) issue(s);")
    stores = [m.start() for m in re.finditer(r"\b(rope_row|res_s|red|part)\[[^]]*\](\[[^]]*\])?\s*=[^=]|reinterpret_cast<float4\*>\(xs", src)]
    assert len(stores) >= 4 and min(stores) > first


@pytest.mark.parametrize("vocab", [16, 1024, 128256])
def test_embedding_gathers_stay_inside_the_table(rules, vocab):
    """An id is a row, any other value reads the first or the last one: 0x7fffffff is what a row of NaN logits leaves as arg-max."""
    for tok in (0, 1, vocab - 1):
        assert rules.embedding_row(tok, vocab) == tok
    assert rules.embedding_row(0x7fffffff, vocab) == rules.embedding_row(vocab, vocab) == vocab - 1
    assert rules.embedding_row(-1, vocab) == rules.embedding_row(-0x80000000, vocab) == 0
    for kernel in ("embed_kernel", "embed_split_kernel", "step_finish_kernel"):
        assert "embed_row(" in kernel_source(kernel), kernel


def plan(rules, G, Hkv, hd, kv_f32, w_f32, ctx, M):
    out = (C.c_int * 3)()
    rules.attention_plan(G, Hkv, hd, kv_f32, w_f32, ctx, M, out)
    return tuple(out)


# (query heads per KV head, KV heads, head size, fp32 cache, fp32 weights)
ATTN_SHAPES = [(1, 32, 128, 1, 0), (1, 40, 128, 0, 0), (4, 8, 128, 0, 0), (8, 8, 128, 1, 0), (1, 16, 64, 1, 0), (1, 4, 64, 1, 1), (2, 2, 64, 0, 0),
               (8, 1, 128, 1, 1), (1, 80, 64, 0, 0)]


@pytest.mark.parametrize("shape", ATTN_SHAPES)
@pytest.mark.parametrize("M", [1, 2, 4, 5, 16, 64])
def test_attention_ranges_cover_the_context(rules, shape, M):
    """Every position belongs to a range, the partials fit the scratch (64 ranges, or one per 96 positions of the cache) and a
    launch that a captured sequence repeats (same plan) covers every context it is repeated for."""
    for ctx in list(range(M, 1400)) + list(range(1400, 33000, 61)):
        wide, ns, chunk = plan(rules, *shape, ctx, M)
        assert ns >= 1 and chunk >= 1 and ns * chunk >= ctx, (ctx, ns, chunk)
        assert ns <= max(64, -(-ctx // 96)), (ctx, ns)
        if wide:
            assert chunk % 16 == 0 and ns <= 16
            if M == 1 and ctx <= 4096:
                assert ns <= 8          # what the output projection folds itself


# (the LDS-staged kernel of wide 16-bit groups has one range per 96 positions instead)
@pytest.mark.parametrize("shape", [s for s in ATTN_SHAPES if s[0] <= 4 or s[4]])
def test_a_long_generation_has_few_launch_plans(rules, shape):
    """One plan per draft: as many as single steps have, one per 128 positions (steps of 16, eight ranges) and a few between."""
    decode = [plan(rules, *shape, n, 1) for n in range(600, 4091)]
    assert len(set(decode)) <= 34, sorted(set(decode))
    assert sum(a != b for a, b in zip(decode, decode[1:])) == len(set(decode)) - 1      # none comes back
    assert len({plan(rules, *shape, n, 1) for n in range(4100, 8190)}) <= 17
    draft = {plan(rules, *shape, rules.draft_ctx(n, 4), 1) for n in range(600, 4087)}
    assert draft <= set(decode)
    assert all(rules.draft_ctx(n, k) == n + k - 1 for n in (1, 9) for k in (1, 15))


def test_qkv_tiles_are_the_faster_ones_where_both_were_measured(rules):
    """(stacked weight rows, prompt rows) -> rows per tile of the faster launch."""
    measured = {(12288, 128): 192, (12288, 256): 192, (12288, 320): 192, (12288, 512): 192, (15360, 192): 256, (15360, 320): 192, (15360, 512): 256,
                (6144, 256): 192, (6144, 512): 192, (9216, 384): 256, (9216, 512): 192, (6528, 384): 192, (6528, 512): 128, (9600, 256): 192,
                (9600, 320): 128, (9600, 384): 128, (9600, 512): 192, (14976, 128): 192, (14976, 256): 128, (14976, 320): 192, (14976, 512): 128,
                (1152, 512): 192, (1920, 320): 192, (3456, 65): 192}
    for (n, rows), tile in measured.items():
        assert rules.qkv_tile(n, -(-rows // 128)) == tile, (n, rows)
    for n in range(128, 40000, 128):
        for mb in (1, 2, 3, 4):
            t = rules.qkv_tile(n, mb)
            assert t in (128, 192, 256) and n % t == 0


def test_k_slices_of_the_large_tiles(rules):
    """The cut is the faster one where two were measured, every slice has a stripe, and a launch that fills its slots is not cut."""
    rules.k_slices_of.argtypes = [C.c_int, C.c_int, C.c_int, C.c_double, C.c_int]
    measured = {(64, 64, 512 * 4096, 8): 4,            # 7B, 512 rows, output projection
                (64, 172, 512 * 4096, 8): 4,           # .. down projection
                (128, 64, 512 * 8192, 4): 2,           # .. keys and values
                (160, 80, 512 * 10240, 4): 3,          # 13B, keys and values
                (162, 128, 2 * 300 * 6912, 4): 3,      # 70B, 300 rows, the last tiles of gate/up
                (96, 128, 300 * 8192, 8): 5}           # .. output projection
    for (blocks, stripes, sums, most), ks in measured.items():
        assert rules.k_slices_of(blocks, 256, stripes, 4.0 * sums, most) == ks, (blocks, stripes)
    for slots in (256, 512):
        for blocks in range(1, 3 * slots, 7):
            for stripes in (1, 2, 3, 16, 64, 448):
                ks = rules.k_slices_of(blocks, slots, stripes, 4e6, 8)
                assert 1 <= ks <= min(8, stripes)
                if blocks % slots == 0:
                    assert ks == 1


@pytest.mark.parametrize("shape", ATTN_SHAPES + [(1, 17, 64, 1, 0), (4, 2, 128, 0, 0), (2, 1, 64, 1, 1)])
def test_ranges_of_a_single_row_that_folds_them_itself(rules, shape):
    """They cover the context, fit the scratch and the device, differ from the ranges the output projection folds only where those would
    be long, and change as rarely as those do."""
    G, Hkv, hd, kv_f32, _ = shape
    base, plans = 32 * 1024 // (hd * (4 if kv_f32 else 2)), []
    for ctx in list(range(1, 5000)) + list(range(5000, 33000, 61)):
        out = (C.c_int * 3)()
        rules.attention_plan_many(*shape, ctx, out)
        wide, ns, chunk = out
        plans.append(tuple(out))
        assert ns * chunk >= ctx and chunk >= 1
        if plan(rules, *shape, ctx, 1) == tuple(out):
            continue
        assert wide and -(-ctx // base) > 12 and chunk % 16 == 0 and chunk >= base
        assert plan(rules, *shape, ctx, 1)[1] < ns <= min(64, 256 // Hkv)
        assert (ns - 1) * chunk < ctx + 3 * base        # at most three empty ranges
    if plans[0][0]:
        assert len(set(plans[600:4091])) <= 36

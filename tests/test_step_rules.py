"""CPU: who owns what in a single-row step that is one launch (csrc/ssd_rules.h): every unit of every stage has one owner, no
wave more than its registers hold, and the hand-over words of the stages do not overlap."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_14612_amd", "csrc")

WRAPPERS = r"""
#include "ssd_rules.h"
using namespace ssdk;
static int layers = 4;
extern "C" {
void set_layers(int n) { layers = n; }
int blocks(const int* s, int cus) { return step_blocks(StepShape{s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[8], s[9], layers}, cus); }
int begin(int n, int b, int nb) { return step_begin(n, b, nb); }
void mail(const int* s, long* o) {
    const StepMail m = step_mail(StepShape{s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[8], s[9], layers});
    o[0] = m.x; o[1] = m.qkv; o[2] = m.part; o[3] = m.act; o[4] = m.total;
}
void rmail(const int* s, long* o) {
    const RowsMail m = rows_mail(StepShape{s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[8], s[9], layers});
    o[0] = m.x; o[1] = m.qkv; o[2] = m.att; o[3] = m.act; o[4] = m.total;
}
int rows_fit(const int* s, int M, int ctx, int nb, int max_rows) { return rows_step_fits(StepShape{s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[8], s[9], layers}, M, ctx, nb, max_rows); }
int rows_of(int M) { return rows_step_rows(M); }
int tries(int resets, int bad, int seqs_behind) {   // launches that give up in `resets` sequences whose first `bad` tries fail
    StepBackoff b;
    int gave_up = 0, first_good = -1;
    for (int r = 0; r < resets; r++) {
        if (b.on()) {
            if (gave_up < bad) { b.gave_up(); gave_up++; }
            else { b.ran = true; if (first_good < 0) first_good = r; }
        }
        b.reset();
        if (first_good >= 0 && r - first_good + 1 == seqs_behind) return b.fails;
    }
    return seqs_behind ? -1 : gave_up;
}
int limits(int i) { const int v[] = {ST_WAVES, ST_GU, ST_CD, ST_CF, AW_MAX_RANGES, ST_WAIT_WORDS, RS_ROWS}; return v[i]; }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("step_rules")
    src, lib = str(d / "rules.cpp"), str(d / "librules.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, "-o", lib, src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return C.CDLL(lib)


# d, dq, dkv, f, V, hd, H, Hkv, weight type, cache type (0 fp32, 1 bf16, 2 fp16)
SHAPES = [
    (256, 256, 256, 688, 1024, 64, 4, 4, 0, 0), (512, 512, 512, 1536, 16, 64, 8, 8, 0, 0), (1024, 1024, 1024, 2816, 32000, 64, 16, 16, 1, 0),
    (1024, 1024, 256, 3072, 4112, 128, 8, 2, 1, 1), (64, 64, 64, 48, 272, 64, 1, 1, 2, 2), (528, 512, 64, 1040, 48, 64, 8, 1, 2, 0),
    (16, 1024, 1024, 16, 16, 64, 16, 16, 1, 0), (1024, 64, 64, 16, 128256, 64, 1, 1, 1, 0),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cus", [256, 255, 200, 64])
def test_every_unit_has_one_owner_within_the_limits(rules, shape, cus):
    s = (C.c_int * 10)(*shape)
    nb = rules.blocks(s, cus)
    d, dq, dkv, f, V, hd, H, Hkv, wt, kt = shape
    waves, gu, cd, cf, ranges, ctrl = (rules.limits(i) for i in range(6))
    if nb == 0:
        assert cus < 256 or d < 256, "a full device takes shapes of at least 256 rows"
        return
    assert nb <= min(cus, d)
    chunk = 64 * (4 if wt == 0 else 8)
    assert d <= cd * chunk and dq <= cd * chunk and f <= cf * chunk
    for n, most in ((d, waves), ((dq + 2 * dkv) // 2, waves), (f, gu * waves), (V // 2, None)):
        edges = [rules.begin(n, b, nb) for b in range(nb + 1)]
        assert edges[0] == 0 and edges[-1] == n and all(a <= b for a, b in zip(edges, edges[1:]))
        if most is not None:
            assert max(b - a for a, b in zip(edges, edges[1:])) <= most
    # every block owns a row of the residual stream
    assert all(rules.begin(d, b, nb) < rules.begin(d, b + 1, nb) for b in range(nb))
    o = (C.c_long * 5)()
    rules.mail(s, o)
    sizes = (2 * d, dq + 2 * dkv, H * ranges * (hd + 2), f)
    assert o[0] >= ctrl and all(o[i] + sizes[i] <= o[i + 1] for i in range(4))
    assert all(v % 2 == 0 for v in o), "word pairs are read by 16-byte loads"
    rows = rules.limits(6)
    rules.rmail(s, o)
    sizes = (2 * rows * d, rows * (dq + 2 * dkv), rows * dq, rows * f)
    assert o[0] == 0 and all(o[i] + sizes[i] <= o[i + 1] for i in range(4)) and all(v % 2 == 0 for v in o[:4])
    for M in range(rows + 2):   # a block per head and row; no row count beyond the layout
        assert rules.rows_fit(s, M, 100, nb, rows) == int(2 <= M <= rows and H * M <= nb)
        # .. and none whose kernel would not be resident
        for most in (0, 3, 5, rows):
            assert rules.rows_fit(s, M, 100, nb, most) == int(2 <= M <= most and H * M <= nb)
    assert [rules.rows_of(M) for M in range(2, rows + 1)] == [3, 3, 5, 5] + [rows] * (rows - 5)


# where six to eight rows are faster with a launch per matrix: measured at these shapes on both sides of every edge
@pytest.mark.parametrize("shape,wt,kt,slow", [
    ((1024, 1024, 1024, 2816, 32000, 64, 16, 16), 2, 2, True), ((1024, 1024, 1024, 2816, 32000, 64, 16, 16), 1, 1, False),
    ((1024, 1024, 1024, 2816, 32000, 64, 16, 16), 2, 0, False), ((256, 256, 256, 688, 1024, 64, 4, 4), 2, 2, False),
    ((512, 512, 512, 2560, 1024, 64, 8, 8), 1, 1, True), ((512, 512, 512, 1984, 1024, 64, 8, 8), 1, 1, False),
    ((768, 768, 768, 3072, 1024, 64, 12, 12), 1, 1, True), ((512, 512, 512, 3072, 1024, 64, 8, 8), 1, 0, False),
    ((1024, 1024, 1024, 2816, 32000, 128, 8, 8), 2, 2, False), ((512, 512, 512, 1536, 1024, 64, 8, 8), 0, 0, False)])
def test_six_to_eight_rows_over_short_contexts(rules, shape, wt, kt, slow):
    s = (C.c_int * 10)(*shape, wt, kt)
    for M in range(2, 10):
        for ctx in (10, 96, 97, 200):
            assert rules.rows_fit(s, M, ctx, 256, 9) == int(not (slow and M in (6, 7, 8) and ctx <= 96)), (M, ctx)


# fewer blocks than CUs: an LM head that is large for the width and depth streams through too few of them
@pytest.mark.parametrize("d,V,layers,fits", [(64, 32000, 1, False), (64, 32000, 4, True), (64, 128256, 4, False), (64, 128256, 12, True),
                                             (128, 32000, 1, True), (128, 128256, 1, False), (128, 128256, 4, True), (240, 128256, 2, True),
                                             (256, 128256, 1, True), (1024, 256000, 1, True)])
def test_narrow_models_with_large_vocabularies(rules, d, V, layers, fits):
    s = (C.c_int * 10)(d, 64, 64, 176, V, 64, 1, 1, 1, 0)
    try:
        rules.set_layers(layers)
        assert rules.blocks(s, 256) == (min(d, 256) if fits else 0)
        if fits:
            assert rules.blocks(s, min(d, 256)) == min(d, 256)      # what a launch is checked with
    finally:
        rules.set_layers(4)


def test_a_launch_that_keeps_giving_up_is_tried_ever_more_rarely(rules):
    assert rules.tries(1, 10 ** 6, 0) == 1 and rules.tries(2, 10 ** 6, 0) == 2      # tried again behind the first reset
    assert rules.tries(1000, 10 ** 6, 0) <= 10
    assert rules.tries(20000, 10 ** 6, 0) <= 10 + 20000 // 1023 + 1                 # never given up for good
    for bad in (1, 2, 5):                                                           # and forgotten where it goes well again
        assert rules.tries(10 ** 5, bad, 15) == bad and rules.tries(10 ** 5, bad, 16) == bad - 1
        assert rules.tries(10 ** 5, bad, 16 * bad) == 0 == rules.tries(10 ** 5, bad, 16 * bad + 1000)


@pytest.mark.parametrize("shape", [(1040, 1024, 1024, 2816, 32000, 64, 16, 16, 1, 0), (1024, 1024, 1024, 3088, 32000, 64, 16, 16, 1, 0),
                                   (528, 512, 512, 688, 1024, 64, 8, 8, 0, 0), (1024, 1024, 1024, 2816, 32000, 64, 16, 16, 1, 2),
                                   (4096, 4096, 4096, 11008, 32000, 128, 32, 32, 1, 0)])
def test_wider_shapes_and_mixed_types_take_the_launches_per_matrix(rules, shape):
    assert rules.blocks((C.c_int * 10)(*shape), 256) == 0

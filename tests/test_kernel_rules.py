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


@pytest.mark.parametrize("vocab", [16, 1024, 128256])
def test_embedding_gathers_stay_inside_the_table(rules, vocab):
    """An id is a row, any other value reads the first or the last one: 0x7fffffff is what a row of NaN logits leaves as arg-max."""
    for tok in (0, 1, vocab - 1):
        assert rules.embedding_row(tok, vocab) == tok
    assert rules.embedding_row(0x7fffffff, vocab) == rules.embedding_row(vocab, vocab) == vocab - 1
    assert rules.embedding_row(-1, vocab) == rules.embedding_row(-0x80000000, vocab) == 0
    for kernel in ("embed_kernel", "embed_split_kernel", "step_finish_kernel"):
        assert "embed_row(" in kernel_source(kernel), kernel

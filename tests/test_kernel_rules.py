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
    return C.CDLL(lib)


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

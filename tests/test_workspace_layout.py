"""CPU: the regions of the workspace hold what the calls put into them, and the replayed sequences are few.  The host side of the library (ssd_api.cpp, whose layout
functions are not exported) is compiled into a small test library."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import paper_2604_14612_amd as ssd
from synth import ModelShape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_14612_amd", "csrc")

WRAPPERS = r"""
#include "%s/ssd_api.cpp"
extern "C" {
// distinct replayed sequences of drafts behind n0 .. n1 - 1 committed tokens
__attribute__((visibility("default"))) int t_draft_keys(const ssd_config* c, int k, int n0, int n1, int adaptive) {
    std::map<std::string, int> keys; const std::vector<uint8_t> sub(2 * c->n_layers, 0);
    for (int n = n0; n < n1; n++) keys[adaptive ? adaptive_key(make_dims(*c), sub, n, k, 0) : draft_key(make_dims(*c), sub, n, k)]++;
    return (int)keys.size();
}
// tap rows a confidence pass may take: a position's, a batch of the context window
__attribute__((visibility("default"))) int t_conf_rows(const ssd_config* c) {
    const Layout l = make_layout(*c); const int w = window_batch_rows(make_dims(*c), l.rows, l.conf_rows);
    return w > l.conf_rows ? w : l.conf_rows;
}
__attribute__((visibility("default"))) int t_fused(const ssd_config* c) { return rows_fused_supported(make_dims(*c)); }
__attribute__((visibility("default"))) size_t t_tapn_bytes(const ssd_config* c) { const Layout l = make_layout(*c); return l.hi - l.tapn; }
__attribute__((visibility("default"))) size_t t_hi_bytes(const ssd_config* c) { const Layout l = make_layout(*c); return l.lo - l.hi; }
__attribute__((visibility("default"))) size_t t_logits_bytes(const ssd_config* c) { const Layout l = make_layout(*c); return l.taps - l.logits; }
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    kernels_obj = os.path.join(CSRC, "ssd_kernels.o")
    if not os.path.exists(kernels_obj):
        from paper_2604_14612_amd.build import build
        build()
    d = tmp_path_factory.mktemp("layout")
    src, lib = str(d / "layout.cpp"), str(d / "liblayout.so")
    with open(src, "w") as f:
        f.write(WRAPPERS % CSRC)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                        "-Wl,-Bsymbolic", "-o", lib, src, kernels_obj, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    l = C.CDLL(lib)
    for n in ("t_tapn_bytes", "t_hi_bytes", "t_logits_bytes"):
        getattr(l, n).restype = C.c_size_t
    return l


# fp32, bf16 and fp16 with an FFN that is no multiple of 64 (the untiled paths) and the tiled one; shallow models, whose window
# batch is longer than the rows of a position, and deep ones
@pytest.mark.parametrize("dtype,d_ffn", [("fp32", 704), ("bf16", 720), ("fp16", 720), ("bf16", 704)])
@pytest.mark.parametrize("layers", [1, 2, 8, 40])
def test_a_confidence_pass_fits_its_buffers(host, layers, dtype, d_ffn):
    """Normalised rows, logits and the reduction's records (24 bytes per row and slice of the vocabulary, at most 16 slices)."""
    shape = ModelShape(layers, 256, 4, 4, d_ffn, 16384, dtype=dtype)
    cfg = ssd.make_config(shape, 64, 4, conf_window=100)
    p = C.byref(cfg)
    rows = host.t_conf_rows(p)
    assert rows >= 2 * shape.n_layers
    fused = bool(host.t_fused(p))
    buf = host.t_hi_bytes(p) if fused else host.t_tapn_bytes(p)
    assert buf >= rows * shape.d_model * (2 if fused else 4)
    records = min(rows, 256) * 24 * min(16, shape.vocab // 1024, shape.d_model * (2 if fused else 4) // 24)
    assert buf >= records
    assert host.t_logits_bytes(p) >= rows * shape.vocab * 4


def test_drafts_of_a_long_generation_replay_few_sequences(host):
    """The keys of the captured sequences name the skip mask, k and the attention plan of the draft's last step only."""
    shape = ModelShape(2, 4096, 32, 32, 11008, 32000, dtype="bf16")
    p = C.byref(ssd.make_config(shape, 8192, 8))
    for k in (1, 4, 8):
        for adaptive in (0, 1):
            assert host.t_draft_keys(p, k, 600, 4087, adaptive) <= 34

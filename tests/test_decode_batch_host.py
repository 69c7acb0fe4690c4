"""CPU: the host side of ssd_decode_many (steps that are waited for together) where a step of a batch fails or gives up.

ssd_api.cpp is compiled against stand-ins for the launches of a step and for the runtime: a step's successor is a fixed function of its
token and position, it commits what step_finish_kernel commits, and the n-th one can be made to fail or to give up.  What is enqueued
runs when the host waits, or step by step while it polls."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2604_14612_amd as ssd
from paper_2604_14612_amd.binding import SYMBOLS, ssd_stats, ssd_weights
from synth import ModelShape

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_14612_amd", "csrc")

STANDINS = r"""
#include "%(csrc)s/ssd_kernels.h"
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <thread>
#include <vector>
using namespace ssdk;
namespace sim {
int V = 1024, steps_left = -1, fail_sync = 0, syncs = 0, dropped_in_flight = 0, short_plans = 0, blocks = 0, give_up_at = -1, step = 0, captures = 0, most_steps = 0, steps_enqueued = 0, step_ends = 0;
struct Launch { std::function<void()> f; bool step; };   // step: the last one of a step
using Sequence = std::vector<Launch>;
Sequence* rec = nullptr;            // of the sequence being captured
std::deque<Launch> stream;
void enqueue(const Launch& l)
{
    stream.push_back(l);
    if (l.step) { steps_enqueued++; if (steps_enqueued > most_steps) most_steps = steps_enqueued; }
}
void run_one() { const Launch l = stream.front(); stream.pop_front(); if (l.step) { steps_enqueued--; step_ends++; } l.f(); }
void drain() { while (!stream.empty()) run_one(); }
template <typename F> hipError_t run(F f, bool ends_step = false) { if (rec) rec->push_back({f, ends_step}); else enqueue({f, ends_step}); return hipSuccess; }
int next(int tok, int pos) { return (int)(((long)tok * 31 + pos * 7 + 3) %% V); }
void finish(float tok, const StepOut& o, bool ok)
{
    const int t = next((int)tok, o.pos_dev ? *o.pos_dev : 0);
    *o.tok_out = *o.tok_host = t;
    if (o.step_ctrl && !ok) *o.step_err_host = 1;
    if (o.pos_dev && ok) { const int p = *o.pos_dev; if (o.tok_log) o.tok_log[p] = t; *o.pos_dev = p + 1; *o.tok0 = t; }
    if (o.x_next) o.x_next[0] = (float)t;
}
bool counted_out() { return steps_left >= 0 && steps_left-- == 0; }
}
#define SIM static inline hipError_t
SIM sim_embed_rows(const Dims&, const void*, Tokens t, int, float* x, hipStream_t, const float* = nullptr, const int* = nullptr, int = 0, float* = nullptr)
{ return sim::run([=] { x[0] = (float)(t.first ? t.first[0] : t.ids[0]); }); }
SIM sim_rows_plain(const Dims&, const RowsPlain&, hipStream_t) { return hipSuccess; }
SIM sim_gemv_qkv(const Dims&, const void*, const void*, const void*, const float*, const float*, const float*, const int*, int, float*, void*, void*, hipStream_t) { return hipSuccess; }
SIM sim_gemv_resid(const Dims&, const void*, int, int, const float*, float*, float*, hipStream_t) { return hipSuccess; }
SIM sim_gemv_swiglu(const Dims&, const void*, const void*, const float*, const float*, float*, hipStream_t) { return hipSuccess; }
SIM sim_attention(const Dims&, const float*, int, const void*, const void*, const int* pos, int off, int hint, int M, float*, float*, uint16_t*, uint16_t*, hipStream_t, int* fold = nullptr, unsigned* = nullptr)
{
    if (fold) *fold = 0;
    return sim::rec ? hipSuccess : sim::run([=] { sim::short_plans += *pos + off + M > hint + off + M; });   // (a replayed plan serves several positions)
}
SIM sim_gemv_lmhead_argmax(const Dims&, const void*, const float*, const float* x, float*, float, float*, const StepOut& o, hipStream_t)
{
    if (sim::counted_out()) return hipErrorOutOfMemory;
    return sim::run([=] { sim::finish(x[0], o, true); }, true);
}
SIM sim_step_fused(const Dims&, const StepLaunch& a, const StepOut& o, hipStream_t)
{
    if (sim::counted_out()) return hipErrorOutOfMemory;
    return sim::run([=] { if (sim::step++ == sim::give_up_at) o.step_ctrl[1] = 1; sim::finish(a.x[0], o, o.step_ctrl[1] == 0); }, true);
}
SIM sim_vocab_reduce(const float*, int M, int, float, float, int32_t* out, int32_t* host, int32_t*, float*, float*, hipStream_t)
{ return sim::run([=] { for (int r = 0; r < M; r++) out[r] = host[r] = 5; }); }
SIM sim_set_state(int32_t* tok, int32_t t, int* pos, int p, hipStream_t) { return sim::run([=] { *tok = t; *pos = p; }); }
SIM sim_advance_state(int* pos, int n, int32_t* tok, const int32_t* src, hipStream_t) { return sim::run([=] { *pos += n; if (src) *tok = *src; }); }
SIM sim_copy_f32(const float*, float*, size_t, hipStream_t) { return hipSuccess; }
SIM sim_step_device_blocks(const Dims&, int, int* b, int* m) { *b = sim::blocks; *m = 0; return hipSuccess; }
SIM sim_static(int, void** p) { *p = nullptr; return hipSuccess; }
SIM sim_malloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
SIM sim_free(void* p) { free(p); return hipSuccess; }
SIM sim_device(int* d) { *d = 0; return hipSuccess; }
SIM sim_copy(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { sim::drain(); memcpy(d, s, n); return hipSuccess; }
SIM sim_fill(void* d, int v, size_t n, hipStream_t) { sim::drain(); memset(d, v, n); return hipSuccess; }
SIM sim_sync(hipStream_t) { sim::syncs++; sim::drain(); return sim::fail_sync ? hipErrorUnknown : hipSuccess; }
SIM sim_query(hipStream_t) { return sim::stream.empty() ? hipSuccess : hipErrorNotReady; }
namespace std { namespace this_thread { inline void sim_yield() { for (const int was = sim::step_ends; !sim::stream.empty() && sim::step_ends == was;) sim::run_one(); } } }
SIM sim_begin(hipStream_t, hipStreamCaptureMode) { sim::rec = new sim::Sequence; return hipSuccess; }
SIM sim_end(hipStream_t, hipGraph_t* g) { *g = (hipGraph_t)sim::rec; sim::rec = nullptr; sim::captures++; return hipSuccess; }
SIM sim_inst(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) { *e = (hipGraphExec_t) new sim::Sequence(*(sim::Sequence*)g); return hipSuccess; }
SIM sim_gdel(hipGraph_t g) { delete (sim::Sequence*)g; return hipSuccess; }
SIM sim_edel(hipGraphExec_t e) { sim::dropped_in_flight += !sim::stream.empty(); delete (sim::Sequence*)e; return hipSuccess; }
SIM sim_launch(hipGraphExec_t e, hipStream_t) { for (auto& l : *(sim::Sequence*)e) sim::enqueue(l); return hipSuccess; }
#define embed_rows sim_embed_rows
#define rows_plain sim_rows_plain
#define gemv_qkv sim_gemv_qkv
#define gemv_resid sim_gemv_resid
#define gemv_swiglu sim_gemv_swiglu
#define attention sim_attention
#define gemv_lmhead_argmax sim_gemv_lmhead_argmax
#define step_fused sim_step_fused
#define vocab_reduce sim_vocab_reduce
#define set_state sim_set_state
#define advance_state sim_advance_state
#define copy_f32 sim_copy_f32
#define step_device_blocks sim_step_device_blocks
#define static_scratch_for_device sim_static
#define hipHostMalloc sim_malloc
#define hipHostFree sim_free
#define hipGetDevice sim_device
#define hipMemcpyAsync sim_copy
#define hipMemsetAsync sim_fill
#define hipStreamSynchronize sim_sync
#define hipStreamQuery sim_query
#define yield sim_yield
#define hipStreamBeginCapture sim_begin
#define hipStreamEndCapture sim_end
#define hipGraphInstantiate sim_inst
#define hipGraphDestroy sim_gdel
#define hipGraphExecDestroy sim_edel
#define hipGraphLaunch sim_launch
#include "%(csrc)s/ssd_api.cpp"
extern "C" {
#define T_API __attribute__((visibility("default")))
T_API int* t_sim(int i) { int* v[] = {&sim::steps_left, &sim::fail_sync, &sim::syncs, &sim::dropped_in_flight, &sim::short_plans, &sim::blocks, &sim::give_up_at, &sim::step, &sim::captures, &sim::most_steps}; return v[i]; }
T_API int t_next(int tok, int pos) { return sim::next(tok, pos); }
T_API void t_fill_cache(ssd_ctx* c, int n) { for (int i = (int)c->graphs.size(); i < n; i++) c->graphs["filler " + std::to_string(i)] = nullptr; }
T_API void t_other_calls(int n) { calls_in_flight[0] += n; calls_begun[0] += n > 0; }
T_API int t_cached(ssd_ctx* c) { return (int)c->graphs.size(); }
}
"""
NAMES = ("steps_left", "fail_sync", "syncs", "dropped_in_flight", "short_plans", "blocks", "give_up_at", "step", "captures", "most_steps")
SHAPE = ModelShape(2, 256, 4, 4, 688, 1024, dtype="fp32")
PROMPT = [1, 2, 3]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    kernels_obj = os.path.join(CSRC, "ssd_kernels.o")
    if not os.path.exists(kernels_obj):
        from paper_2604_14612_amd.build import build
        build()
    d = tmp_path_factory.mktemp("batch")
    src, lib = str(d / "batch.cpp"), str(d / "libbatch.so")
    with open(src, "w") as f:
        f.write(STANDINS % {"csrc": CSRC})
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                        "-Wl,-Bsymbolic", "-o", lib, src, kernels_obj, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    l = C.CDLL(lib)
    for name in ("ssd_create", "ssd_workspace_bytes", "ssd_set_workspace", "ssd_load_weights", "ssd_reset", "ssd_destroy", "ssd_prefill", "ssd_decode",
                 "ssd_decode_many", "ssd_get_stats", "ssd_get_one_launch", "ssd_set_one_launch", "ssd_last_error"):
        getattr(l, name).restype, getattr(l, name).argtypes = SYMBOLS[name]
    l.t_sim.restype = C.POINTER(C.c_int)
    l.t_fill_cache.argtypes = [C.c_void_p, C.c_int]
    l.t_cached.argtypes = [C.c_void_p]
    return l


class Sim:
    """A context on the stand-ins; its stream is no null stream where sequences are to be replayed."""

    def __init__(self, l, max_seq=400, replay=False, blocks=0):
        self.l = l
        for n in NAMES:
            self[n] = -1 if n in ("steps_left", "give_up_at") else 0
        self["blocks"] = blocks
        cfg, self.h = ssd.make_config(SHAPE, max_seq, 4), C.c_void_p()
        assert l.ssd_create(C.byref(cfg), C.c_void_p(1 if replay else 0), C.byref(self.h)) == 0
        n = l.ssd_workspace_bytes(C.byref(cfg))
        self.ws = np.zeros(n + 256, np.uint8)
        assert l.ssd_set_workspace(self.h, C.c_void_p(-(-self.ws.ctypes.data // 256) * 256), n) == 0
        layers = C.cast((C.c_void_p * 2)(4096, 4096), C.POINTER(C.c_void_p))
        assert l.ssd_load_weights(self.h, C.byref(ssd_weights(4096, 4096, 4096, *[layers] * 9))) == 0
        self.prefill()

    def __getitem__(self, name):
        return self.l.t_sim(NAMES.index(name))[0]

    def __setitem__(self, name, v):
        self.l.t_sim(NAMES.index(name))[0] = v

    def prefill(self):
        out = np.zeros(1, np.int32)
        assert self.l.ssd_prefill(self.h, (C.c_int32 * 3)(*PROMPT), 3, out.ctypes.data) == 0
        self.want = [int(out[0])]
        return self.want[0]

    def expect(self, n):
        """The next n tokens of the sequence."""
        for _ in range(n):
            self.want.append(self.l.t_next(self.want[-1], len(PROMPT) + len(self.want) - 1))
        return self.want[len(self.want) - n:]

    def many(self, count):
        out = np.full(count, -1, np.int32)
        return self.l.ssd_decode_many(self.h, count, out.ctypes.data), out.tolist()

    def decode(self):
        out = np.zeros(1, np.int32)
        return self.l.ssd_decode(self.h, out.ctypes.data), int(out[0])

    def stats(self):
        st = ssd_stats()
        assert self.l.ssd_get_stats(self.h, C.byref(st)) == 0
        return st

    def one_launch(self):
        v = np.zeros(3, np.int64)
        assert self.l.ssd_get_one_launch(self.h, v[:1].ctypes.data, v[1:2].ctypes.data, v[2:].ctypes.data) == 0
        return v.tolist()

    def close(self):
        self.l.ssd_destroy(self.h)


@pytest.fixture
def sim(host):
    made = []

    def make(**kw):
        made.append(Sim(host, **kw))
        return made[-1]
    yield make
    for s in made:
        s.close()


@pytest.mark.parametrize("replay", [False, True])
@pytest.mark.parametrize("blocks", [0, 256])
def test_the_stand_ins_decode_a_sequence(sim, replay, blocks):
    s = sim(replay=replay, blocks=blocks)
    for n in (1, 31, 70):
        assert s.many(n) == (0, s.expect(n))
    assert s.decode() == (0, s.expect(1)[0])
    assert s.stats().n_tokens == 3 + len(s.want) and s["short_plans"] == 0
    assert s.one_launch() == [103 if blocks else 0, 0, 0]
    assert (s["captures"] > 0) == (replay and not blocks)


@pytest.mark.parametrize("blocks", [0, 256])
@pytest.mark.parametrize("good", [0, 1, 20, 31, 40])
def test_a_step_of_a_batch_that_fails(sim, blocks, good):
    """The steps in front of it have committed on the device: they count, and the sequence goes on behind them."""
    s = sim(blocks=blocks)
    s["steps_left"] = good
    rc, got = s.many(64)
    assert rc == ssd.SSD_EHIP and b"memory" in s.l.ssd_last_error(s.h)
    assert got[:good] == s.expect(good) and got[good:] == [-1] * (64 - good)
    st = s.stats()
    assert st.n_tokens == 4 + good and st.decode_steps == good and st.committed == 1 + good
    assert s.decode() == (0, s.expect(1)[0])
    assert s.many(40) == (0, s.expect(40))
    assert s["short_plans"] == 0 and s.stats().n_tokens == 3 + len(s.want)


def test_a_device_that_no_longer_answers(sim):
    """Nobody knows what was committed: the sequence is over, the context goes on with a prompt."""
    s = sim()
    s["fail_sync"] = 1
    assert s.many(8)[0] == ssd.SSD_EHIP
    s["fail_sync"] = 0
    assert s.decode()[0] == ssd.SSD_ESTATE and s.many(2)[0] == ssd.SSD_ESTATE and s.stats().n_tokens == 0
    s.prefill()
    assert s.many(8) == (0, s.expect(8))


@pytest.mark.parametrize("at", [0, 1, 17, 31, 32, 39])
def test_a_step_that_gives_up_inside_a_batch(sim, at):
    """Those in front of it stay, those behind it commit nothing and are done again by the launches per matrix."""
    s = sim(blocks=256)
    s["give_up_at"] = at
    assert s.many(40) == (0, s.expect(40))
    assert s.one_launch() == [at, 0, 1] and s.stats().decode_steps == 40 and s.stats().n_tokens == 44


def test_a_full_cache_of_sequences_costs_no_waits(sim):
    """Sequences are dropped, behind a wait, where a new one finds the cache full, and nowhere else."""
    s = sim(replay=True)
    assert s.many(33) == (0, s.expect(33))
    s.l.t_fill_cache(s.h, 256)
    for _ in range(3):
        before = s["syncs"]
        assert s.many(4) == (0, s.expect(4)) and s["syncs"] == before + 1
    assert s.l.t_cached(s.h) == 256
    assert s.many(300) == (0, s.expect(300)) and s.l.t_cached(s.h) < 256     # plans that were not seen yet
    assert s["dropped_in_flight"] == 0
    narrow = sim(replay=True, blocks=256)
    narrow.l.t_fill_cache(narrow.h, 256)
    before = narrow["syncs"]
    assert narrow.many(32) == (0, narrow.expect(32)) and narrow["syncs"] == before + 1


@pytest.mark.parametrize("replay", [False, True])
@pytest.mark.parametrize("blocks", [0, 256])
def test_a_batch_leaves_the_device_to_others(sim, replay, blocks):
    """Two steps are on the stream at most; while another context's call has work on the device every step is waited for."""
    s = sim(replay=replay, blocks=blocks)
    before = s["syncs"]
    assert s.many(64) == (0, s.expect(64))
    assert s["most_steps"] == 2 and s["syncs"] == before + 2
    s["most_steps"] = 0
    s.l.t_other_calls(1)
    try:
        before = s["syncs"]
        assert s.many(40) == (0, s.expect(40))
        assert s["most_steps"] == 1 and s["syncs"] == before + 40
    finally:
        s.l.t_other_calls(-1)
    before = s["syncs"]
    assert s.many(32) == (0, s.expect(32)) and s["syncs"] == before + 1


def test_steps_in_one_launch_and_the_cache_of_sequences(sim):
    """They are never captured, so they leave nothing there, and a new bound of their waits takes nothing out."""
    s = sim(replay=True, blocks=256)
    assert s.many(40) == (0, s.expect(40)) and s.decode() == (0, s.expect(1)[0])
    assert s.l.t_cached(s.h) == 0
    assert s.l.ssd_set_one_launch(s.h, 0, 0) == 0
    assert s.many(40) == (0, s.expect(40))
    cached = s.l.t_cached(s.h)
    assert cached > 0
    for bound in (-1, 1000, 0):
        assert s.l.ssd_set_one_launch(s.h, 1, bound) == 0 and s.l.t_cached(s.h) == cached
    before = s.one_launch()[0]
    assert s.many(3) == (0, s.expect(3)) and s.decode() == (0, s.expect(1)[0])
    assert s.l.t_cached(s.h) == cached and s.one_launch()[0] == before + 4


@pytest.mark.parametrize("n_new", [0, 1, 2, 33, 34, 100])
def test_a_request_can_be_interrupted_between_batches(n_new):
    """Python sees a signal when a call has returned: no call of a request makes more steps than are waited for together."""
    class Steps:
        def __init__(self):
            self.made = []

        def ssd_prefill(self, prompt):
            return 100

        def ssd_decode_many(self, count):
            self.made.append(count)
            return [101 + i for i in range(sum(self.made) - count, sum(self.made))]
    s = Steps()
    assert ssd.generate_vanilla(s, PROMPT, n_new) == list(range(100, 100 + n_new))
    assert sum(s.made) == max(n_new - 1, 0) and all(1 <= m <= 32 for m in s.made) and len(s.made) == -(-max(n_new - 1, 0) // 32)

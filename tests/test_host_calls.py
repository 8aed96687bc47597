"""The library's host side on the CPU: llma_api.hip and llma_trigger.hip compiled for the host alone and linked against tests/host_stub.cpp,
where a stream is a queue that runs when it is waited for and every launcher notes its arguments.  What a GPU cannot
show reliably: what is still in flight when a call returns, and what the host had told the device by then."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_2304_04487_amd as llma
from paper_2304_04487_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("host")
    objs = []
    for src in (os.path.join(build.CSRC, "llma_api.hip"), os.path.join(build.CSRC, "llma_trigger.hip"), os.path.join(HERE, "host_stub.cpp")):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        run([build._hipcc(), "-std=c++17", "-O1", "-fPIC", "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-Wno-unused-result",
             "-I", build.CSRC, "-c", src, "-o", objs[-1]])
    out = tmp / "libhost.so"
    run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", str(out), *objs])     # (its own HIP calls, whatever else is loaded)
    lib = ctypes.CDLL(str(out))
    lib.llma_last_error.restype = ctypes.c_char_p
    return lib


def i32(*values):
    return (ctypes.c_int32 * len(values))(*values)


class Ctx:
    """a context of zero weights on the stubbed runtime"""

    def __init__(self, lib, dtype, n_layers=3, max_batch=2, max_k=4, max_seq=128):
        self.lib, self.L = lib, n_layers
        bf16 = dtype == "bf16"
        d, F, V = 128, 256, 64
        cfg = llma.ModelCfgC(n_layers, d, 2, 64, F, V, max_seq, max_batch, max_k, llma.LLMA_DTYPE_BF16 if bf16 else llma.LLMA_DTYPE_F32, 1, 1e-6, 1e4)
        self.keep = np.zeros(2 * F * d + 3 * d * d + 2 * V * d, np.float32)
        p = self.keep.ctypes.data
        per = (ctypes.c_void_p * n_layers)(*[p] * n_layers)
        w = llma.WeightsC(p, p, p, per, per, per, per, per, per)
        self.h = ctypes.c_void_p()
        assert lib.llma_create(ctypes.byref(cfg), ctypes.byref(w), None, ctypes.byref(self.h)) == 0, lib.llma_last_error(None)
        self.notes()

    def notes(self):
        """(prompt passes' start lengths, rows of the decoding GEMMs, their split flags) since the last look"""
        out = []
        for f in (self.lib.stub_prompt_T, self.lib.stub_gemm_rows, self.lib.stub_gemm_split):
            a = (ctypes.c_int32 * 4096)()
            out.append(list(a[:f(a, 4096)]))
        return out

    def prefill(self, n, seq=0):
        assert self.lib.llma_prefill(self.h, seq, i32(*[1] * n), n) == 0

    def verify(self, drafts, seq=0):
        return self.lib.llma_verify_step(self.h, seq, i32(*drafts), len(drafts), None, None, None)

    def generate(self, max_new, prompt=8, k=2):
        self.out, n_out = np.full(max_new, -1, np.int32), ctypes.c_int32()
        offs = i32(0, 0)
        return self.lib.llma_generate(self.h, 0, i32(*[1] * prompt), prompt, None, offs, 0, 1, k, max_new,
                                      self.out.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), ctypes.byref(n_out), None, None)

    def generate_batch(self, lens, max_new, k):
        n, total = len(lens), sum(lens)
        out, n_out = (ctypes.c_int32 * (n * max_new))(), (ctypes.c_int32 * n)()
        offs = i32(*[sum(lens[:b]) for b in range(n + 1)])
        return self.lib.llma_generate_batch(self.h, n, i32(*range(n)), i32(*[1] * total), offs, None, None, None, 1, k, max_new, out, n_out, None, None)

    def state(self, seq=0):
        t, p = ctypes.c_int32(), ctypes.c_int32()
        assert self.lib.llma_get_state(self.h, seq, ctypes.byref(t), ctypes.byref(p)) == 0
        return t.value, p.value


@pytest.fixture
def ctx(lib, request, monkeypatch):
    monkeypatch.setenv("LLMA_NO_AUTOTUNE", "1")
    c = Ctx(lib, request.param)
    yield c
    lib.stub_fail_last_error(-1)
    lib.stub_fail_event_record(-1)
    lib.llma_destroy(c.h)


both_types = pytest.mark.parametrize("ctx", ["fp32", "bf16"], indirect=True)


def test_only_contexts_whose_prompts_can_share_passes_hold_their_rows(lib, monkeypatch):
    """prompts share passes where a step can have more than 48 rows; other contexts need scratch for one sequence's prompt"""
    monkeypatch.setenv("LLMA_NO_AUTOTUNE", "1")
    lib.llma_device_bytes.restype = ctypes.c_int64
    held = []
    for max_batch in (8, 9, 10):                # 40, 45 and 50 rows
        c = Ctx(lib, "bf16", max_batch=max_batch, max_k=4)
        held.append(lib.llma_device_bytes(c.h))
        lib.llma_destroy(c.h)
    slot = 3 * 2 * 128 * 128 * 3 + 2 * 48 * 66 * 4 + 1000       # a slot's cache, attention partials and words
    assert held[1] - held[0] <= slot and held[2] - held[1] > slot


@both_types
def test_calls_run_on_the_stub(ctx):
    ctx.prefill(20)
    assert ctx.state() == (19, 1)
    assert ctx.verify([2, 3]) == 0 and ctx.state() == (20, 7)
    assert ctx.generate(9) == 0 and ctx.out.tolist() == [7] * 9
    assert ctx.state() == (7 + 9, 7)


@both_types
def test_failed_step_leaves_nothing_in_flight(ctx):
    """launches of a step that failed half way read the host's words in pinned memory, which the next call rewrites: a
    step of other slots and fewer rows would then write K / V at positions the failed step's row count runs past"""
    ctx.prefill(20)
    ctx.lib.stub_fail_last_error(0)
    assert ctx.verify([2, 3, 4]) == llma.LLMA_E_HIP
    assert ctx.lib.stub_pending() == 0
    ctx.prefill(30, seq=1)
    assert ctx.verify([], seq=1) == 0 and ctx.state(1) == (30, 7) and ctx.state(0) == (19, 1)


@both_types
@pytest.mark.parametrize("record", [0, 1, 4])
def test_failed_generation_leaves_nothing_in_flight(ctx, record):
    """the step that runs ahead writes output counts the next generation clears and waits on"""
    ctx.lib.stub_fail_event_record(record)
    assert ctx.generate(9) == llma.LLMA_E_HIP
    assert ctx.lib.stub_pending() == 0
    assert ctx.generate(5) == 0 and ctx.out.tolist() == [7] * 5


@pytest.mark.parametrize("ctx", ["bf16"], indirect=True)
def test_kernel_timing_counts_steps_only(ctx):
    """prompt passes are not bracketed, whatever GEMM they use"""
    def launches():
        n, ms = ctypes.c_int64(), ctypes.c_double()
        assert ctx.lib.llma_get_kernel_timing(ctx.h, ctypes.byref(n), ctypes.byref(ms)) == 0
        return n.value
    assert ctx.lib.llma_set_option(ctx.h, llma.LLMA_OPT_KERNEL_TIMING, 1) == 0
    for n in (2, 20, 49, 50):
        ctx.prefill(n, seq=1)
        assert ctx.lib.llma_reset(ctx.h, 1) == 0
    assert launches() == 0
    ctx.prefill(20)
    assert ctx.verify([2, 3]) == 0 and launches() == ctx.L


@pytest.mark.parametrize("ctx", ["bf16"], indirect=True)
def test_prompt_passes_keep_both_activation_planes(ctx):
    """LLMA_OPT_ACT_SPLIT = 0 rounds the activations of decoding steps of up to 48 rows; every prompt pass and every
    larger step feeds hi + lo"""
    ctx.prefill(20)
    ctx.notes()
    assert ctx.lib.llma_set_option(ctx.h, llma.LLMA_OPT_ACT_SPLIT, 0) == 0
    ctx.prefill(20, seq=1)
    _, rows, split = ctx.notes()
    assert rows == [19] * (4 * ctx.L) and split == [1] * (4 * ctx.L)
    assert ctx.verify([2]) == 0
    _, rows, split = ctx.notes()
    assert rows == [2] * (4 * ctx.L + 1) and split == [0] * (4 * ctx.L + 1)


@both_types
def test_state_calls_reach_the_next_prompt(ctx):
    """reset, truncate and set_pending change the host's copy only; a prompt brings the device's up to date before it starts"""
    ctx.prefill(20)
    ctx.notes()
    assert ctx.lib.llma_truncate(ctx.h, 0, 11) == 0 and ctx.lib.llma_set_pending(ctx.h, 0, 5) == 0
    ctx.prefill(10)
    assert ctx.notes()[0] == [11] and ctx.state() == (20, 1)
    assert ctx.verify([1]) == 0 and ctx.state() == (21, 7)
    assert ctx.lib.llma_reset(ctx.h, 0) == 0
    ctx.prefill(4)
    assert ctx.notes()[0] == [0] and ctx.state() == (3, 1)


@pytest.mark.parametrize("ctx", ["bf16"], indirect=True)
def test_many_shapes_do_not_end_the_replay_of_steps(ctx, monkeypatch):
    """prompts, shared prompt passes above all, have a shape of their own nearly every time: steps are replayed from their
    graphs whatever has been seen in between, those captured before and new ones, and the graphs held stay bounded"""
    lib = ctx.lib
    wide = Ctx(lib, "bf16", max_batch=16, max_k=4)
    lib.stub_capture(1)
    try:
        def replayed(k):
            for _ in range(2):                      # seen, captured
                assert wide.verify([2] * k) == 0
                assert lib.llma_truncate(wide.h, 0, 19) == 0
            before = lib.stub_graph_launches()
            assert wide.verify([2] * k) == 0 and lib.llma_truncate(wide.h, 0, 19) == 0
            return lib.stub_graph_launches() - before

        wide.prefill(20)
        assert replayed(2) == 1
        rng = np.random.RandomState(4)
        for i in range(400):
            lens = rng.randint(2, 60, 10 + i % 7).tolist()
            for _ in range(1 + (i % 3 == 0) * 2):   # (some often enough to be captured)
                assert wide.generate_batch(lens, 2, 4) == 0
        assert lib.llma_reset(wide.h, 0) == 0
        wide.prefill(20)
        assert replayed(2) == 1 and replayed(3) == 1
        assert 0 < lib.stub_graphs_alive() <= 256
    finally:
        lib.stub_capture(0)
        lib.llma_destroy(wide.h)
    assert lib.stub_graphs_alive() == 0


@both_types
def test_input_lists_beyond_2_gib_get_memory_of_their_size(ctx):
    """prompts, references and document lists of a generation share one allocation: its size does not wrap around (the list is all zeros, so the host
    holds no memory for it either; nothing of this size is given to it here)"""
    lib, words = ctx.lib, 1_450_000_000
    ref = np.zeros(words, np.int32)
    lib.stub_refused.restype = ctypes.c_ulong
    out, n_out = np.zeros(4, np.int32), ctypes.c_int32()
    p = [a.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)) for a in (ref, out)]
    lib.stub_alloc_limit(ctypes.c_long(1 << 32))
    try:
        rc = lib.llma_generate(ctx.h, 0, i32(1, 2), 2, p[0], i32(0, words), 1, 1, 2, 4, p[1], ctypes.byref(n_out), None, None)
    finally:
        lib.stub_alloc_limit(ctypes.c_long(-1))
    assert rc == llma.LLMA_E_NOMEM
    assert 4 * words <= lib.stub_refused() <= 8 * words
    assert ctx.generate(9) == 0 and ctx.out.tolist() == [7] * 9


@pytest.mark.parametrize("max_new", [3212, 3213, 16320, 16321, 40000])
def test_long_results_come_as_they_are(lib, monkeypatch, max_new):
    """results of more than the 16384 words that pass through pinned memory go straight to the caller: the tokens, and of the trace
    the steps that were taken"""
    monkeypatch.setenv("LLMA_NO_AUTOTUNE", "1")
    lib.stub_fetched.restype = ctypes.c_long
    c = Ctx(lib, "fp32", n_layers=1, max_seq=max_new + 16)
    try:
        offs, n_out, steps = i32(0, 0), ctypes.c_int32(), ctypes.c_int32()
        for with_trace in (False, True):
            out, trace = np.full(max_new, -1, np.int32), np.full((max_new, 4), -2, np.int32)
            p = [a.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)) for a in (out, trace)]
            lib.stub_fetched()
            assert lib.llma_generate(c.h, 0, i32(*[1] * 8), 8, None, offs, 0, 1, 2, max_new, p[0], ctypes.byref(n_out), p[1] if with_trace else None, ctypes.byref(steps)) == 0
            words = max_new + 4 * steps.value * with_trace
            assert (out == 7).all() and n_out.value == steps.value == max_new and c.state() == (7 + max_new, 7)
            assert (trace == ([1, 1, -1, -1] if with_trace else -2)).all()
            if (max_new + 64) * (5 if with_trace else 1) > 16384:
                assert lib.stub_fetched() <= 4 * words + 128            # (and the slots' words)
    finally:
        lib.llma_destroy(c.h)


def checksum(a):
    h = 1
    for v in a.tolist():
        h = (h * 31 + v) & 0xffffffff
    return h & 0x7fffffff


def find_trigger(lib, seed, y_len, ref_len):
    rng = np.random.RandomState(seed)
    y, ref = rng.randint(0, 32000, y_len).astype(np.int32), rng.randint(0, 32000, ref_len).astype(np.int32)
    offs = np.array([0, ref_len // 3, ref_len], np.int32)
    doc, pos = ctypes.c_int32(), ctypes.c_int32()
    p = [a.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)) for a in (y, ref, offs)]
    assert lib.llma_find_trigger(p[0], y_len, p[1], p[2], 2, 1, ctypes.byref(doc), ctypes.byref(pos)) == 1, lib.llma_last_error(None)
    assert lib.stub_pending() == 0
    assert (doc.value, pos.value) == (checksum(ref), checksum(y) ^ checksum(offs)), (y_len, ref_len)


def test_large_lookups_pin_no_more_than_a_thread_keeps(lib):
    """a list longer than the kept buffers passes through them in pieces; pinned memory of its size costs more than it saves"""
    lib.stub_pinned.restype = ctypes.c_long
    find_trigger(lib, 1, 40, 1000)
    for i, (y_len, ref_len) in enumerate([(3, 262100), (131069, 131070), (131070, 262140), (262144, 5), (1, 700001), (20, 500)]):
        find_trigger(lib, 2 + i, y_len, ref_len)
    assert lib.stub_pinned() <= 3 * (1 << 20)


@pytest.mark.parametrize("reused", [0, 1])
def test_kept_buffers_do_not_outlive_a_device_reset(lib, reused):
    """the caller may reset the device between two lookups: what the thread kept is gone, its addresses may be others'"""
    find_trigger(lib, 11, 40, 1000)
    lib.stub_device_reset(reused)
    find_trigger(lib, 12, 40, 1000)
    find_trigger(lib, 13, 40, 300000)
    assert lib.stub_stale_uses() == 0

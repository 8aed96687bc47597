"""The trigger's scan in spans of 4096 positions: sizes at the edges of a span, matches across one, several spans per
sequence of a generation.  Against the oracle, exact."""
import numpy as np
import pytest

import synth
from oracle import OracleModel, CachedLLM, greedy_decode, llma_decode, match_ngrams, docs_from_flat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def llma():
    import paper_2304_04487_amd as m
    m.load_library()
    return m


def both(llma, y, ref, offs, n):
    """host-list form and device form of the call"""
    import torch
    host = llma.llma_find_trigger(y, ref, offs, n)
    dev = [torch.tensor(np.asarray(a, np.int32), device="cuda") for a in (y, ref, offs)]
    res = torch.full((3,), 77, dtype=torch.int32, device="cuda")
    llma.llma_find_trigger_static(*dev, n, res)
    r = res.cpu().tolist()
    return host, (bool(r[0]), r[1], r[2])


@pytest.mark.parametrize("length", [1, 2, 4095, 4096, 4097, 8191, 8193, 20000])
def test_span_edges(llma, length):
    """the tail of y is planted so that the copied token falls on the first / last position of a span"""
    rng = np.random.RandomState(length)
    y = rng.randint(0, 1000, 200)
    for at in sorted({1, 2, 4095, 4096, 4097, 8191, 8192, length - 1} & set(range(1, length))):
        for tail in (1, 3, 130):                                # 130 tokens: more than one 64-token step of a wave
            ref = rng.randint(1000, 2000, length)
            t = min(tail, at)
            ref[at - t:at] = y[len(y) - t:]
            for offs in ([0, length], [0, 0, at - min(t, 2), length, length]):
                for n in (1, 2):
                    want = match_ngrams(y.tolist(), docs_from_flat(ref, offs), n)
                    assert both(llma, y, ref, offs, n) == (want, want), (length, at, tail, offs, n)


def test_many_candidates(llma):
    """two symbols: nearly every position survives the one-token test; ties between spans go to the smallest position"""
    rng = np.random.RandomState(3)
    for length in (5000, 9000):
        ref = rng.randint(0, 2, length)
        y = np.concatenate([rng.randint(0, 2, 40), ref[4000:4100]])
        offs = [0, 1234, 4090, 4090, length]
        for n in (1, 3):
            want = match_ngrams(y.tolist(), docs_from_flat(ref, offs), n)
            assert both(llma, y, ref, offs, n) == (want, want)
    ref = np.full(9000, 7)
    want = match_ngrams([7] * 90, [ref.tolist()], 2)
    assert both(llma, [7] * 90, ref, [0, 9000], 2) == (want, want)


@pytest.mark.parametrize("bad", [[1, 5000, 9000], [0, 9000, 5000], [0, 5000, 8999], [0, -4, 9000], [0, 9000, -1, 9000]])
def test_bad_device_list_over_several_spans(llma, bad):
    import torch
    ref = torch.zeros(9000, dtype=torch.int32, device="cuda")
    y = torch.zeros(50, dtype=torch.int32, device="cuda")
    res = torch.zeros(3, dtype=torch.int32, device="cuda")
    llma.llma_find_trigger_static(y, ref, torch.tensor(bad, dtype=torch.int32, device="cuda"), 1, res)
    assert res.cpu().tolist() == [-1, -1, -1]


def test_generate_with_references_of_several_spans(llma):
    wl = synth.WORKLOADS["tiny"]
    w = synth.make_weights(wl.model, wl.seed)
    om = OracleModel(wl.model, w)
    prompt = synth.make_prompt(wl)
    y = greedy_decode(CachedLLM(om, prompt, 160), wl.max_new)
    refs = []
    for i, (before, after) in enumerate([(4090, 10), (9000, 0), (3, 0)]):
        noise = synth.uniform_tokens(5, 20 + i, before + after, wl.model.vocab)
        refs.append((np.concatenate([noise[:before], np.array(y, np.int32), noise[before:]]), np.array([0, 2, before + after + len(y)], np.int32)))
    want = [llma_decode(CachedLLM(om, prompt, 160), docs_from_flat(*r), wl.n, wl.k, wl.max_new) for r in refs]
    ctx = llma.Context(wl.model, w, max_seq=160, max_batch=3, max_k=8)
    for b, r in enumerate(refs):
        toks, trace = ctx.generate(prompt, *r, wl.n, wl.k, wl.max_new, seq=b)
        assert toks.tolist() == want[b][0] and trace == want[b][1]
    got = ctx.generate_batch([prompt] * 3, refs, wl.n, wl.k, wl.max_new)
    assert [g[0].tolist() for g in got] == [t for t, _ in want] and [g[1] for g in got] == [t for _, t in want]
    ctx.close()


def skewed(rng, length, share, last):
    ref = rng.randint(1000, 2000, length)
    ref[rng.rand(length) < share] = last
    return ref


@pytest.mark.parametrize("length", [48, 1472, 4096, 9000])
@pytest.mark.parametrize("share", [0.02, 0.3, 0.97])
def test_frequent_last_token(llma, length, share):
    """the last token of y makes up a good part of the reference: few, hundreds or nearly all positions survive the
    one-token test, matches of 1 .. 300 tokens among them"""
    rng = np.random.RandomState(length + int(100 * share))
    for y_len in (1, 7, 8, 9, 300):
        y = np.append(rng.randint(1000, 2000, y_len - 1), 13)
        ref = skewed(rng, length, share, 13)
        for tail in (2, 8, 9, 24, 25, 299):                     # (the copies of a tail: two, the later one a token longer)
            for at, t in ((length // 3, tail), (length - 1, tail + 1)):
                t = min(t, at, y_len)
                ref[at - t:at] = y[y_len - t:]
        for offs in ([0, length], [0, 0, length // 3 - 1, length // 3 + 5, length]):
            for n in (1, 2, 9):
                want = match_ngrams(y.tolist(), docs_from_flat(ref, offs), n)
                assert both(llma, y, ref, offs, n) == (want, want), (y_len, offs, n)


@pytest.mark.parametrize("period,noise", [(1, 0.0), (1, 0.01), (2, 0.0), (16, 0.0), (16, 0.01), (50, 0.002)])
def test_repetitive_references(llma, period, noise):
    """periodic texts with a few changed tokens: many long agreements of different lengths, ties go to the smallest position"""
    rng = np.random.RandomState(period)
    text = np.arange(9000) % period
    hit = rng.rand(9000) < noise
    text[hit] = rng.randint(0, max(period, 2), int(hit.sum()))
    for length, y_len in ((4096, 600), (9000, 90)):
        ref = text[:length]
        for y in (text[:y_len], np.arange(y_len) % period):
            for offs in ([0, length], [0, 777, 4090, length]):
                want = match_ngrams(y.tolist(), docs_from_flat(ref, offs), 2)
                assert both(llma, y, ref, offs, 2) == (want, want), (length, y_len, offs)


def test_frequent_tokens_cost_no_serial_chain(llma):
    """2048 of 4096 positions survive the one-token test: less than six times the call without any (followed one after
    the other they cost 50 times, side by side twice as much)"""
    import torch
    rng = np.random.RandomState(1)
    y = np.append(rng.randint(1000, 2000, 255), 13)
    res = torch.zeros(3, dtype=torch.int32, device="cuda")
    us = {}
    for share in (0.0, 0.5):
        a = [torch.tensor(np.asarray(x, np.int32), device="cuda") for x in (y, skewed(rng, 4096, share, 13), [0, 1500, 4096])]
        best = 1e9
        for _ in range(6):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(50):
                llma.llma_find_trigger_static(*a, 2, res)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1) * 20)
        us[share] = best
    assert us[0.5] < 6 * us[0.0], us


def test_generate_with_frequent_tokens(llma):
    """references made of the generation's own tokens: every step's last token occurs about a hundred times in them"""
    wl = synth.WORKLOADS["tiny"]
    w = synth.make_weights(wl.model, wl.seed)
    om = OracleModel(wl.model, w)
    prompt = synth.make_prompt(wl)
    y = greedy_decode(CachedLLM(om, prompt, 160), wl.max_new)
    rng = np.random.RandomState(9)
    refs = [(rng.choice(y, size).astype(np.int32), np.array([0, size // 3, size], np.int32)) for size in (3000, 4096, 9000)]
    want = [llma_decode(CachedLLM(om, prompt, 160), docs_from_flat(*r), 1, 8, wl.max_new) for r in refs]
    ctx = llma.Context(wl.model, w, max_seq=160, max_batch=3, max_k=8)
    for b, r in enumerate(refs):
        toks, trace = ctx.generate(prompt, *r, 1, 8, wl.max_new, seq=b)
        assert toks.tolist() == want[b][0] and trace == want[b][1]
    got = ctx.generate_batch([prompt] * 3, refs, 1, 8, wl.max_new)
    assert [g[0].tolist() for g in got] == [t for t, _ in want] and [g[1] for g in got] == [t for _, t in want]
    ctx.close()

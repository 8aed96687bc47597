"""Generations whose inputs or results are around the 16384 words that pass through a context's pinned memory (longer ones come and go straight
from and to the caller's), one sequence and several with ragged references: tokens of the plain decoding, traces of Algorithm 2 on
them; and the sequence state that the next call starts from."""
import numpy as np
import pytest

import synth
from oracle import docs_from_flat, infer_decoding_sequence

pytestmark = pytest.mark.gpu

CFG = synth.ModelCfg("inputs", 1, 64, 2, 32, 64, 300, "fp32")


@pytest.fixture(scope="module")
def ctx():
    import paper_2304_04487_amd as llma
    c = llma.Context(CFG, synth.make_weights(CFG, 3), max_seq=3500, max_batch=3, max_k=4)
    c.enable_logits_dump(15)
    yield c
    c.close()


def reference(y, length, docs, seed):
    """noise with pieces of y in it, the last one at the reference's end"""
    ref = synth.uniform_tokens(seed, 1, length, CFG.vocab).astype(np.int32)
    for i, at in enumerate(range(5, length - 12, max(13, length // 40))):
        ref[at:at + 10] = y[(3 * i) % (len(y) - 10):][:10]
    ref[-10:] = y[5:15]
    return ref, np.linspace(0, length, docs + 1).astype(np.int32)


def plain(ctx, prompt, n):
    return ctx.generate(prompt, None, None, 1, 0, n)[0].tolist()


@pytest.mark.parametrize("ref_len", [100, 16340, 16341, 16342, 16360, 16384, 40000])
def test_inputs_of_one_sequence(ctx, ref_len):
    prompt = synth.uniform_tokens(5, 1, 40, CFG.vocab).astype(np.int32)       # (40 + ref_len, rounded up to fours, + 4 words of input)
    y = plain(ctx, prompt, 48)
    ref, offs = reference(y, ref_len, 3, 7)
    tokens, trace = ctx.generate(prompt, ref, offs, 2, 4, 48)
    assert tokens.tolist() == y
    assert trace == infer_decoding_sequence(y, docs_from_flat(ref, offs), 2, 4)
    assert ctx.get_state(0) == (39 + 48, y[-1])
    more = ctx.verify_step([])[2]
    assert y + more == plain(ctx, prompt, 49)


@pytest.mark.parametrize("lens", [(30, 0, 500), (6000, 10000, 200), (16000, 3, 9000)])
def test_inputs_of_several(ctx, lens):
    prompts = [synth.uniform_tokens(6, i, n, CFG.vocab).astype(np.int32) for i, n in enumerate((1, 60, 17))]
    ys = [plain(ctx, p, 40) for p in prompts]
    refs = [reference(y, n, 1 + i, 8 + i) if n > 20 else (None if n == 0 else (np.array(y[:n], np.int32), np.array([0, n], np.int32))) for i, (y, n) in enumerate(zip(ys, lens))]
    slots = [2, 0, 1]
    for (tokens, trace), y, r, p, s in zip(ctx.generate_batch(prompts, refs, 1, 4, 40, seqs=slots), ys, refs, prompts, slots):
        assert tokens.tolist() == y
        assert trace == infer_decoding_sequence(y, docs_from_flat(*r) if r else [], 1, 4)
        assert ctx.get_state(s) == (len(p) - 1 + 40, y[-1])


@pytest.mark.parametrize("max_new", [3212, 3213, 3300])
def test_results(ctx, max_new):
    prompt = synth.uniform_tokens(5, 2, 9, CFG.vocab).astype(np.int32)        # (5 (max_new + 64) words of results: 16380 .. 16820)
    y = plain(ctx, prompt, max_new)
    ref, offs = reference(y, 90, 2, 9)
    tokens, trace = ctx.generate(prompt, ref, offs, 1, 4, max_new)
    assert tokens.tolist() == y
    assert trace == infer_decoding_sequence(y, docs_from_flat(ref, offs), 1, 4)

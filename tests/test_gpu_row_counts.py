"""Prompt passes and batched steps over the row counts at which the GEMMs change their form (48 / 49 rows: tile-K to
panel; a K split or none; row tiles and weight tiles per workgroup), on a shape whose k-steps fill no whole turn of
the panel kernel's weight ring (36 and 89 k-steps) and whose last feature blocks are ragged.  Logits against the oracle
in float64 within the project's bf16 tolerance, tokens exact."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

CFG = synth.ModelCfg("rows", 2, 1152, 9, 128, 2848, 1040, "bf16")
ATOL, RTOL = 1e-2, 2e-2                     # measured here: below 1e-3 absolute


@pytest.fixture(scope="module")
def setup():
    import paper_2304_04487_amd as llma
    w = synth.make_weights(CFG, 31, gain_jitter=0.2)
    return llma, w, OracleModel(CFG, w)


@pytest.mark.parametrize("length", [2, 17, 18, 33, 49, 50, 65, 66, 81, 97, 145, 161, 162, 200, 321, 640])
def test_prompt_lengths(setup, length):
    llma, w, om = setup
    ctx = llma.Context(CFG, w, max_seq=700, max_batch=1, max_k=4)
    ctx.enable_logits_dump(5)
    prompt = synth.uniform_tokens(7, length, length, CFG.vocab)
    drafts = synth.uniform_tokens(8, length, 4, CFG.vocab).tolist()
    want = om.forward(np.concatenate([prompt, drafts]), om.new_cache(700), 0)[-5:]
    for _ in range(3):                      # eager, captured, replayed
        ctx.reset()
        ctx.prefill(prompt)
        ctx.verify_step(drafts)
        got = ctx.logits(5)
        assert np.all(np.abs(got - want) <= ATOL + RTOL * np.abs(want)), float(np.abs(got - want).max())
    ctx.close()


@pytest.mark.parametrize("seqs,k", [(2, 23), (7, 6), (4, 15), (13, 4), (11, 8), (16, 8), (5, 32)])
def test_step_rows(setup, seqs, k):
    """48, 49, 64, 65, 99, 144 and 165 rows"""
    llma, w, om = setup
    ctx = llma.Context(CFG, w, max_seq=160, max_batch=seqs, max_k=k)
    ctx.enable_logits_dump(seqs * (k + 1))
    prompts = [synth.uniform_tokens(9, 10 * seqs + b, 20 + 3 * b, CFG.vocab) for b in range(seqs)]
    drafts = np.stack([synth.uniform_tokens(10, 10 * seqs + b, k, CFG.vocab) for b in range(seqs)])
    want = np.concatenate([om.forward(np.concatenate([p, d]), om.new_cache(160), 0)[-(k + 1):] for p, d in zip(prompts, drafts)])
    for b, p in enumerate(prompts):
        ctx.prefill(p, seq=b)
    for _ in range(3):
        for b, p in enumerate(prompts):
            ctx.truncate(len(p) - 1, seq=b)
            ctx.set_pending(p[-1], seq=b)
        ctx.verify_step_batch(list(range(seqs)), drafts)
        got = ctx.logits(seqs * (k + 1))
        assert np.all(np.abs(got - want) <= ATOL + RTOL * np.abs(want)), float(np.abs(got - want).max())
    ctx.close()


@pytest.mark.parametrize("d,heads,dh,ffn,vocab", [(128, 4, 32, 258, 300), (192, 3, 64, 511, 97), (256, 2, 128, 1028, 512), (640, 5, 128, 516, 64)])
def test_fp32_shapes(d, heads, dh, ffn, vocab):
    """FFN widths that are no multiple of 4, several head widths, more and fewer elements than a pass of 512; 1, 8, 9 and 10 rows"""
    import paper_2304_04487_amd as llma
    cfg = synth.ModelCfg("f32", 2, d, heads, dh, ffn, vocab, "fp32")
    w = synth.make_weights(cfg, 41, gain_jitter=0.2)
    om = OracleModel(cfg, w)
    ctx = llma.Context(cfg, w, max_seq=200, max_batch=2, max_k=9)
    ctx.enable_logits_dump(20)
    prompt = synth.uniform_tokens(3, d, 120, vocab)
    for k in (0, 7, 8, 9):
        drafts = synth.uniform_tokens(4, k, k, vocab)
        want = om.forward(np.concatenate([prompt, drafts]), om.new_cache(200), 0)[-(k + 1):]
        for b in range(2):
            ctx.reset(b)
            ctx.prefill(prompt, seq=b)
        ctx.verify_step(drafts)
        assert np.abs(ctx.logits(k + 1) - want).max() <= 1e-4
        ctx.reset(0)
        ctx.prefill(prompt)
        ctx.verify_step_batch([1, 0], np.stack([drafts, drafts]))
        assert np.abs(ctx.logits(2 * (k + 1)) - np.concatenate([want, want])).max() <= 1e-4
    ctx.close()


def test_activation_planes_beyond_4_gib():
    """2112 rows of an FFN 2^20 wide: each plane of the down projection's input holds 4.4 GB.  The matrices repeat 4096
    hidden features 256 times, with the down projection scaled by 2^-8, so the model equals a small one for the oracle."""
    import paper_2304_04487_amd as llma
    small = synth.ModelCfg("narrow", 1, 128, 2, 64, 4096, 512, "bf16")
    w = synth.make_weights(small, 51, gain_jitter=0.2)
    om = OracleModel(small, w)
    lay = w["layers"][0]
    wd = synth.f32_to_bf16(synth.bf16_to_f32(lay["wd"]) / 256.0)
    wide = synth.ModelCfg("wide", 1, 128, 2, 64, 4096 * 256, 512, "bf16")
    layer = dict(lay, wgu=np.concatenate([np.tile(lay["wgu"][:4096], (256, 1)), np.tile(lay["wgu"][4096:], (256, 1))]), wd=np.tile(wd, (1, 256)))
    seqs, k = 64, 32
    ctx = llma.Context(wide, dict(w, layers=[layer]), max_seq=64, max_batch=seqs, max_k=k)
    ctx.enable_logits_dump(seqs * (k + 1))
    prompts = [synth.uniform_tokens(5, b, 3, 512) for b in range(seqs)]
    drafts = np.stack([synth.uniform_tokens(6, b, k, 512) for b in range(seqs)])
    want = np.concatenate([om.forward(np.concatenate([p, d]), om.new_cache(64), 0)[-(k + 1):] for p, d in zip(prompts, drafts)])
    for b, p in enumerate(prompts):
        ctx.prefill(p, seq=b)
    ctx.verify_step_batch(list(range(seqs)), drafts)
    got = ctx.logits(seqs * (k + 1))
    assert np.all(np.abs(got - want) <= ATOL + RTOL * np.abs(want)), float(np.abs(got - want).max())
    ctx.close()

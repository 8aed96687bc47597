"""Matrices of a few feature tiles and passes of many rows: the split-K launch has fewer waves than groups of four rows, whose rstd
they compute for the finishing kernel (tests/test_panel_cut.py counts them).  Logits against the oracle in float64."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

ATOL = 7e-4          # four times the largest error measured below (1.7e-4); rows scaled by another norm's rstd: 0.13 and more


def model(d_ffn, vocab):
    cfg = synth.ModelCfg("narrow", 2, 1024, 8, 128, d_ffn, vocab, "bf16")
    w = synth.make_weights(cfg, 61, gain_jitter=0.2)
    return cfg, w, OracleModel(cfg, w)


def test_lm_head_of_a_step():
    """648 rows of 72 sequences, 8 tiles of the vocabulary"""
    import paper_2304_04487_amd as llma
    cfg, w, om = model(2848, 128)
    seqs, k = 72, 8
    ctx = llma.Context(cfg, w, max_seq=40, max_batch=seqs, max_k=k)
    ctx.enable_logits_dump(seqs * (k + 1))
    prompts = [synth.uniform_tokens(5, b, 2 + b % 20, cfg.vocab) for b in range(seqs)]
    drafts = np.stack([synth.uniform_tokens(6, b, k, cfg.vocab) for b in range(seqs)])
    want = np.concatenate([om.forward(np.concatenate([p, d]), om.new_cache(40), 0)[-(k + 1):] for p, d in zip(prompts, drafts)])
    for b, p in enumerate(prompts):
        ctx.prefill(p, seq=b)
    ctx.verify_step_batch(list(range(seqs)), drafts)
    err = np.abs(ctx.logits(seqs * (k + 1)) - want).max(axis=1)
    ctx.close()
    assert float(err.max()) <= ATOL, (float(err.max()), int(err.argmax()))


@pytest.mark.parametrize("d_ffn,rows", [(128, 1664), (64, 643)])
def test_gate_up_of_a_prompt(d_ffn, rows):
    import paper_2304_04487_amd as llma
    cfg, w, om = model(d_ffn, 528)
    ctx = llma.Context(cfg, w, max_seq=rows + 8, max_batch=1, max_k=4)
    ctx.enable_logits_dump(5)
    prompt = synth.uniform_tokens(7, rows, rows + 1, cfg.vocab)
    draft = synth.uniform_tokens(8, rows, 4, cfg.vocab)
    want = om.forward(np.concatenate([prompt, draft]), om.new_cache(rows + 8), 0)[-5:]
    ctx.prefill(prompt)
    ctx.verify_step(draft)
    err = float(np.abs(ctx.logits(5) - want).max())
    ctx.close()
    assert err <= ATOL, err

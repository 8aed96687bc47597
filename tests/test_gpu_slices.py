"""Steps and short prompt passes of 17 .. 48 rows whose down projection (and O projection, QKV, LM head) runs in K slices over
several workgroups: the same bits as one-row steps give, for K slices of unequal length, groups of slices, ragged feature blocks, one to three row
tiles and several sequences; and the oracle's logits (float64) within the bound of tests/test_gpu_row_counts.py."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

# k-steps: 325 (slices of 40 and 41) in the down projection, 36 (4 and 5) in O; 72 feature tiles.  `wide`: O takes slices from 38 rows on too.
# LM head: 16 slices in two groups (1601 tiles, slices of two k-steps) and in four (1089 tiles, slices of four).  QKV: 960 tiles from 33 rows on
CFGS = [synth.ModelCfg("deep-ffn", 1, 1152, 9, 128, 10400, 1040, "bf16"), synth.ModelCfg("wide", 1, 4672, 73, 64, 10304, 528, "bf16"),
        synth.ModelCfg("head-2", 1, 1024, 8, 128, 512, 25616, "bf16"), synth.ModelCfg("head-4", 1, 2048, 16, 128, 512, 17424, "bf16"),
        synth.ModelCfg("qkv", 1, 5120, 40, 128, 512, 528, "bf16")]
ATOL = 1e-3


@pytest.fixture(scope="module", params=CFGS, ids=lambda c: c.name)
def setup(request):
    import paper_2304_04487_amd as llma
    cfg = request.param
    w = synth.make_weights(cfg, 77, gain_jitter=0.2)
    ctx = llma.Context(cfg, w, max_seq=160, max_batch=2, max_k=32)
    ctx.enable_logits_dump(66)
    yield cfg, ctx, OracleModel(cfg, w)
    ctx.close()


def one_row_logits(ctx, prompt, tokens, seq=0):
    """logits after prompt and after each of the tokens, one row at a time from the first prompt token on"""
    out = []
    ctx.reset(seq=seq)
    ctx.set_pending(int(prompt[0]), seq=seq)
    for t in list(prompt[1:]) + list(tokens):
        ctx.verify_step([], seq=seq)
        out.append(ctx.logits(1)[0].copy())
        ctx.set_pending(int(t), seq=seq)
    ctx.verify_step([], seq=seq)
    out.append(ctx.logits(1)[0].copy())
    return np.stack(out[len(prompt) - 1:])


def test_rows_are_those_of_one_row_steps(setup):
    cfg, ctx, om = setup
    toks = synth.uniform_tokens(5, 1, 80, cfg.vocab)
    want = one_row_logits(ctx, toks[:40], toks[40:73])
    exact = om.forward(toks[:73], om.new_cache(80), 0)[39:]
    assert float(np.abs(want - exact).max()) <= ATOL
    for k in (15, 16, 17, 24, 31, 32):
        for _ in range(3):                      # eager, captured, replayed
            ctx.reset()
            ctx.prefill(toks[:40])              # (a pass of 39 rows)
            ctx.verify_step(toks[40:40 + k])
            assert np.array_equal(ctx.logits(k + 1), want[:k + 1]), k


def test_two_sequences(setup):
    cfg, ctx, om = setup
    toks = synth.uniform_tokens(6, 2, 80, cfg.vocab)
    a, b = toks[:34], toks[5:28]
    wa, wb = one_row_logits(ctx, a, toks[40:63]), one_row_logits(ctx, b, toks[50:73])
    for k in (8, 16, 19, 23):                   # 18, 34, 40 and 48 rows
        for s, p in ((0, a), (1, b)):
            ctx.reset(seq=s)
            ctx.prefill(p, seq=s)
        ctx.verify_step_batch([0, 1], np.stack([toks[40:40 + k], toks[50:50 + k]]))
        got = ctx.logits(2 * (k + 1))
        assert np.array_equal(got[:k + 1], wa[:k + 1]) and np.array_equal(got[k + 1:], wb[:k + 1]), k

"""The vocabulary arg max and the accept decision over row counts and numbers of partials at the edges of the kernel's trips: partials
read four and one at a time, one trip and two, ties at distant tokens (the lowest id wins), rows without a comparable logit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# partials: a token each (fp32), 16 tokens each (bf16)
CASES = [("fp32", v) for v in (512, 515, 516, 1301, 2048, 2052)] + [("bf16", 16 * n) for n in (67, 132, 512, 516, 1027, 2052)]
K = 16


def make(dtype, vocab, head):
    import paper_2304_04487_amd as llma
    cfg = synth.ModelCfg("argmax", 1, 64, 2 if dtype == "fp32" else 1, 32 if dtype == "fp32" else 64, 64, vocab, dtype)
    w = synth.make_weights(cfg, 11)
    w["lm_head"] = head(w["lm_head"])
    ctx = llma.Context(cfg, w, max_seq=96, max_batch=1, max_k=K)
    ctx.enable_logits_dump(K + 1)
    return cfg, ctx


@pytest.mark.parametrize("dtype,vocab", CASES)
def test_lowest_of_equal_maxima_and_accepted_prefix(dtype, vocab):
    period = vocab // 3                     # every logit occurs at least three times
    cfg, ctx = make(dtype, vocab, lambda h: h[np.arange(vocab) % period].copy())
    prompt = synth.uniform_tokens(3, 1, 20, vocab)
    drafts = synth.uniform_tokens(3, 2, K, vocab).astype(np.int32)
    for _ in range(5):
        ctx.reset()
        ctx.prefill(prompt)
        acc, nxt, emitted = ctx.verify_step(drafts)
        logits = ctx.logits(K + 1)
        best = logits.argmax(1)             # (numpy: the first of equal values)
        assert best.max() < period
        a = 0
        while a < K and drafts[a] == best[a]:
            a += 1
        assert (acc, nxt, list(emitted)) == (a, best[a], best[:a + 1].tolist())
        drafts = best[:K].astype(np.int32)  # accepted at least one further each time
    ctx.close()


@pytest.mark.parametrize("dtype,vocab", [("fp32", 515), ("fp32", 2052), ("bf16", 16 * 67), ("bf16", 16 * 2052)])
def test_rows_without_a_comparable_logit_give_token_0(dtype, vocab):
    nan = (lambda h: np.full_like(h, np.nan)) if dtype == "fp32" else (lambda h: np.full_like(h, 0x7FC0))
    cfg, ctx = make(dtype, vocab, nan)
    ctx.prefill(synth.uniform_tokens(3, 1, 20, vocab))
    acc, nxt, emitted = ctx.verify_step([0, 0, 5])
    assert np.isnan(ctx.logits(4)).all()
    assert (acc, nxt, list(emitted)) == (2, 0, [0, 0, 0])
    ctx.close()


@pytest.mark.parametrize("vocab,first", [(515, 0), (515, 7), (515, 514), (2052, 3), (2052, 700), (2052, 2051)])
def test_minus_infinity_beside_nan(vocab, first):
    """the largest comparable logit is the arg max also where it is minus infinity: the first one of them, behind tokens whose logit is NaN"""
    def head(value):
        def make_head(h):
            h = np.zeros_like(h)
            h[:first, 0] = np.nan
            h[first:, 0] = value
            return h
        return make_head
    prompt = synth.uniform_tokens(3, 1, 20, vocab)
    for value in (1.0, None):
        if value is None:
            value = -np.inf * sign              # the logits' sign is that of the row's first feature
        cfg, ctx = make("fp32", vocab, head(value))
        ctx.prefill(prompt)
        acc, nxt, emitted = ctx.verify_step([])
        logits = ctx.logits(1)[0]
        assert np.isnan(logits[:first]).all()
        sign = np.sign(logits[first])
        assert sign != 0
        ctx.close()
    assert (logits[first:] == -np.inf).all()
    assert (acc, nxt, list(emitted)) == (0, first, [first])

"""Long prompt passes whose gate/up and QKV products go through blocks of 16 and 12 row tiles (256 compute units), with one or
fifteen rows in the last tile and eleven tiles in the last block, against the oracle's logits (float64) of the row after the prompt, which attends
over the K and V of every row in both layers; and every product in either height and in the panel GEMM, whose sums are the same bits."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

CFG = synth.ModelCfg("blocks", 2, 2048, 16, 128, 8192, 256, "bf16")
# gate/up (64 feature blocks): blocks of 16 row tiles at 2033 and 2047 rows.  QKV (24): of 12 at 1889 and 1905
ROWS = [2047, 2033, 1905, 1889]
# largest error over these lengths (2.1e-4), times four
ATOL = 8.4e-4


def test_long_prompts():
    import paper_2304_04487_amd as llma
    w = synth.make_weights(CFG, 31, gain_jitter=0.2)
    om = OracleModel(CFG, w)
    toks = synth.uniform_tokens(8, 1, 2100, CFG.vocab)
    cache = om.new_cache(2048)
    want = om.forward(toks[:2048], cache, 0)
    ctx = llma.Context(CFG, w, max_seq=2112, max_batch=1, max_k=8)
    ctx.enable_logits_dump(9)
    for rows in ROWS:
        ctx.reset()
        ctx.prefill(toks[:rows + 1])
        ctx.verify_step([])
        err = float(np.abs(ctx.logits(1)[0] - want[rows]).max())
        assert err <= ATOL, rows
    ctx.close()


RAGGED = synth.ModelCfg("ragged", 2, 2112, 33, 64, 2112, 256, "bf16")


@pytest.mark.parametrize("cfg,lengths", [(CFG, (2047, 1905)), (RAGGED, (2047, 1905, 1889, 1500))], ids=["whole", "ragged"])
def test_forms_have_the_same_bits(cfg, lengths, monkeypatch):
    """QKV, O, gate/up and down of unsplit passes, forced into the panel GEMM, into blocks of 12 and of 16 row tiles, and as the rule has them:
    the steps on top of the caches they leave, at several lengths, have the same logits.  The second model has a quarter or half
    of a feature block left over in every matrix; lengths leave 1, 12 and 15 rows in the last tile and 7 .. 16 tiles in the last block."""
    import paper_2304_04487_amd as llma
    w = synth.make_weights(cfg, 33, gain_jitter=0.2)
    toks = synth.uniform_tokens(8, 3, 2100, cfg.vocab)
    seen = {}
    for form in ("0", "12", "16", None):
        monkeypatch.delenv("LLMA_BLOCK_ROWS", raising=False)
        if form is not None:
            monkeypatch.setenv("LLMA_BLOCK_ROWS", form)
        ctx = llma.Context(cfg, w, max_seq=2112, max_batch=1, max_k=8)
        ctx.enable_logits_dump(9)
        for rows in lengths:
            ctx.reset()
            ctx.prefill(toks[:rows + 1])
            for past in (rows, rows - 7, rows - 200, 1000, 300, 20, 1):
                ctx.truncate(past)
                ctx.set_pending(int(toks[past]))
                ctx.verify_step([])
                got = ctx.logits(1)[0].copy()
                assert np.isfinite(got).all()
                assert np.array_equal(got, seen.setdefault((rows, past), got)), (form, rows, past)
        ctx.close()

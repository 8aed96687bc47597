"""The rows' sums of squares behind rstd, a sixteenth of a row's tiles per lane: 3 .. 18 tiles to add, which are requested by fours, eights, twelves and
sixteens, sixteenths with fewer and with none; in the decoding GEMM at one, two and three row tiles and for the panel GEMM: the oracle's logits (float64)."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

# model width -> tiles per sixteenth (of the last sixteenths): 3 (0), 4, 5 (3, 0), 8, 10 (8), 13 (1), 18 (6, 0)
WIDTHS = [576, 1024, 1088, 2048, 2368, 3136, 4416]
# largest errors: 7.2e-5 at d 576 .. 4.1e-4 at 4416, 0.9e-7 .. 1.3e-7 times the width; four times that
ATOL_PER_FEATURE = 4 * 1.3e-7


@pytest.mark.parametrize("d", WIDTHS)
def test_steps_and_prompts(d):
    import paper_2304_04487_amd as llma
    cfg = synth.ModelCfg("sums", 1, d, d // 64, 64, 128, 128, "bf16")
    w = synth.make_weights(cfg, 51, gain_jitter=0.2)
    toks = synth.uniform_tokens(8, 4, 120, cfg.vocab)
    om = OracleModel(cfg, w)
    want = om.forward(toks, om.new_cache(120), 0)
    ctx = llma.Context(cfg, w, max_seq=128, max_batch=1, max_k=32)
    ctx.enable_logits_dump(33)
    worst = 0.0
    for past in (3, 40, 70):                                    # prompts in the decoding GEMM's one and three row tiles, and in the panel GEMM
        ctx.reset()
        ctx.prefill(toks[:past + 1])
        for k in (0, 8, 16, 32):
            ctx.truncate(past)
            ctx.set_pending(int(toks[past]))
            ctx.verify_step(toks[past + 1:past + 1 + k])
            worst = max(worst, float(np.abs(ctx.logits(k + 1) - want[past:past + k + 1]).max()))
    ctx.close()
    assert worst <= ATOL_PER_FEATURE * d

"""Prompt passes of 161 .. 192 rows whose gate/up products go through row blocks of 11 and 12 tiles (shape of 7B's feed-forward, one layer), full and
ragged last tiles, and the row counts next to them: the oracle's logits (float64) of the row after the prompt."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

CFG = synth.ModelCfg("tall", 2, 4096, 32, 128, 11008, 128, "bf16")
# largest error over these lengths (6.6e-4), times four
ATOL = 2.7e-3


def test_prompts_of_eleven_and_twelve_row_tiles():
    import paper_2304_04487_amd as llma
    w = synth.make_weights(CFG, 41, gain_jitter=0.2)
    om = OracleModel(CFG, w)
    toks = synth.uniform_tokens(8, 2, 200, CFG.vocab)
    want = om.forward(toks, om.new_cache(200), 0)
    ctx = llma.Context(CFG, w, max_seq=256, max_batch=1, max_k=8)
    ctx.enable_logits_dump(9)
    for rows in (160, 161, 175, 176, 177, 192, 193):
        ctx.reset()
        ctx.prefill(toks[:rows + 1])
        ctx.verify_step([])
        err = float(np.abs(ctx.logits(1)[0] - want[rows]).max())
        assert err <= ATOL, rows
    ctx.close()

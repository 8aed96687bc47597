"""Long prompt passes whose gate/up and QKV products go through blocks of 16 and 12 row tiles (256 compute units), with one or
fifteen rows in the last tile and eleven tiles in the last block, against the oracle's logits (float64) of the row after the prompt, which attends
over the K and V of every row in both layers."""
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

"""llma_generate_batch feeding its sequences' prompts in shared passes (steps of more than 48 rows): ragged lengths around
the row blocks of the attention and of the GEMMs, sequences without a row of their own, a sequence cut between two passes,
a last pass short enough for the decoding GEMM, slots in another order.  Logits after the generation against the oracle in
float64 within the bound of tests/test_gpu_row_counts.py (four times the error measured on this shape)."""
import numpy as np
import pytest

import synth
from oracle import OracleModel, top2_gap

pytestmark = pytest.mark.gpu

CFG = synth.ModelCfg("rows", 2, 1152, 9, 128, 2848, 1040, "bf16")
ATOL = 1e-3


@pytest.fixture(scope="module")
def setup():
    import paper_2304_04487_amd as llma
    w = synth.make_weights(CFG, 31, gain_jitter=0.2)
    return llma, w, OracleModel(CFG, w)


@pytest.mark.parametrize("lens,max_seq,k", [
    ((2, 1, 33, 34, 17, 3, 66), 200, 8),                   # one pass of 149 rows
    ((32, 33, 1, 65, 2), 120, 10),                         # blocks that end on a multiple of 32
    ((100, 30, 72), 100 + 20, 16),                         # passes of 480 rows at most: one of 199
    ((900, 41, 1100, 24, 16), 1200, 12),                   # 2048 rows and a remainder of 28 that two sequences share
    ((700, 690, 680, 90), 760, 12),                        # 2048 rows, of them 660 of the third sequence, and 108: its last 19 and the fourth's
], ids=str)
def test_shared_prompt_passes(setup, lens, max_seq, k):
    llma, w, om = setup
    B = len(lens)
    assert B * (k + 1) > 48
    ctx = llma.Context(CFG, w, max_seq=max_seq, max_batch=B + 1, max_k=k)
    ctx.enable_logits_dump(B * (k + 1))
    prompts = [synth.uniform_tokens(3, 10 * sum(lens) + b, n, CFG.vocab) for b, n in enumerate(lens)]
    slots = [(2 * b + 1) % (B + 1) if B % 2 == 0 else B - b for b in range(B)]
    wants = None
    for _ in range(3):                                      # eager, captured, replayed
        out = ctx.generate_batch(prompts, [None] * B, 1, k, 1, seqs=slots)
        first = [int(t[0]) for t, _ in out]
        if wants is None:
            wants = []
            for p, y in zip(prompts, first):
                lg = om.forward(np.append(p, y), om.new_cache(len(p) + 1), 0)[-2:]
                assert y == int(np.argmax(lg[0])) or top2_gap(lg[0]) <= 2 * ATOL
                wants.append(lg[1])
        ctx.verify_step_batch(slots, np.zeros((B, 0), np.int32))
        got = ctx.logits(B)
        for b in range(B):
            assert float(np.abs(got[b] - wants[b]).max()) <= ATOL, (lens[b], float(np.abs(got[b] - wants[b]).max()))
            assert ctx.get_state(slots[b])[0] == lens[b] + 1
    ctx.close()

"""fp32 path: row counts around the two rows of a wave and the eight of a workgroup, cache lengths around the attention's trips (128 / 64 /
32 keys at head_dim 32 / 64 / 128), a reduction length that is no multiple of the lanes' share: the oracle's logits (float64) within 1e-4
(F32_ATOL of test_gpu_parity.py), and every row the bits of a step of its own."""
import numpy as np
import pytest

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

CFGS = [synth.ModelCfg("dh32", 2, 96, 3, 32, 332, 200, "fp32"), synth.ModelCfg("dh64", 2, 128, 2, 64, 512, 200, "fp32"),
        synth.ModelCfg("dh128", 2, 256, 2, 128, 1028, 200, "fp32")]


@pytest.mark.parametrize("cfg", CFGS, ids=lambda c: c.name)
def test_rows_and_cache_lengths(cfg):
    import paper_2304_04487_amd as llma
    w = synth.make_weights(cfg, 21, gain_jitter=0.2)
    ctx = llma.Context(cfg, w, max_seq=384, max_batch=1, max_k=17)
    ctx.enable_logits_dump(18)
    toks = synth.uniform_tokens(4, 1, 380, cfg.vocab)
    want = OracleModel(cfg, w).forward(toks, OracleModel(cfg, w).new_cache(384), 0)
    for past in (1, 15, 31, 32, 33, 63, 64, 127, 128, 300):
        ctx.reset()
        ctx.prefill(toks[:past + 1])
        single = []
        for j in range(18):
            ctx.truncate(past + j)
            ctx.set_pending(int(toks[past + j]))
            ctx.verify_step([])
            single.append(ctx.logits(1)[0].copy())
        single = np.stack(single)
        assert float(np.abs(single - want[past:past + 18]).max()) <= 1e-4, past
        for k in (1, 2, 6, 7, 8, 15, 17):
            ctx.truncate(past)
            ctx.set_pending(int(toks[past]))
            ctx.verify_step(toks[past + 1:past + 1 + k])
            assert np.array_equal(ctx.logits(k + 1), single[:k + 1]), (past, k)
    ctx.close()


WIDE = synth.ModelCfg("wide", 1, 2048, 16, 128, 6002, 8000, "fp32")


def test_rows_per_wave_of_wide_models():
    """four and eight rows per wave (launches of 48 M products and more) beside two: QKV, gate/up, down (6002: no multiple of four) and LM head
    from three or four rows on, O from twelve; single waves and six of them, full and with one row; prompts of 48 and of 3 rows.  Every row
    the bits of a step of its own."""
    import paper_2304_04487_amd as llma
    w = synth.make_weights(WIDE, 23, gain_jitter=0.2)
    ctx = llma.Context(WIDE, w, max_seq=160, max_batch=1, max_k=32)
    ctx.enable_logits_dump(33)
    toks = synth.uniform_tokens(4, 2, 150, WIDE.vocab)
    om = OracleModel(WIDE, w)
    want = om.forward(toks, om.new_cache(160), 0)
    for past in (3, 48, 99):
        ctx.reset()
        ctx.prefill(toks[:past + 1])
        single = []
        for j in range(33):
            ctx.truncate(past + j)
            ctx.set_pending(int(toks[past + j]))
            ctx.verify_step([])
            single.append(ctx.logits(1)[0].copy())
        single = np.stack(single)
        assert float(np.abs(single - want[past:past + 33]).max()) <= 1e-4, past
        for k in (1, 2, 3, 4, 7, 8, 11, 15, 16, 23, 24, 31, 32):
            ctx.truncate(past)
            ctx.set_pending(int(toks[past]))
            ctx.verify_step(toks[past + 1:past + 1 + k])
            assert np.array_equal(ctx.logits(k + 1), single[:k + 1]), (past, k)
    ctx.close()

"""The attention combine over numbers of chunks at the edges of its trips (4, 8 and 16 chunks per group of lanes; two groups at head_dim
128, four at 64), steps whose rows lie on both sides of an edge, one to three row tiles: the oracle's logits (float64) on the same
imported cache, and every row the bits of a one-row step of its own."""
import numpy as np
import pytest
import torch

import synth
from oracle import OracleModel

pytestmark = pytest.mark.gpu

# activations as bf16 pairs, one layer: 1.4e-5 of the largest logit at most over these lengths; four times that
RTOL = 5.6e-5
# the prompt pass over steep scores, two layers: 2.1e-4 at most; four times that
RISING_RTOL = 8.6e-4


@pytest.mark.parametrize("dh", [64, 128])
def test_chunk_counts(dh):
    import paper_2304_04487_amd as llma
    cfg = synth.ModelCfg("combine", 1, 2 * dh, 2, dh, 64, 128, "bf16")
    w = synth.make_weights(cfg, 5, gain_jitter=0.2)
    for lw in w["layers"]:                      # (large enough for the attention's output to show in the logits)
        lw["wo"] = synth.f32_to_bf16(10 * synth.bf16_to_f32(lw["wo"]))
    om = OracleModel(cfg, w)
    parts = 256 // dh
    edges = [128 * parts * n for n in (1, 4, 8, 16, 32)]
    cap = edges[-1] + 256
    ctx = llma.Context(cfg, w, max_seq=cap, max_batch=1, max_k=32)
    ctx.enable_logits_dump(33)
    toks = synth.uniform_tokens(4, 1, 40, cfg.vocab)
    kk, vv = synth.make_kv_fill(cfg, 9, 1, cap, 0)
    kk[0][:, 5::37] = synth.f32_to_bf16(6 * synth.bf16_to_f32(kk[0][:, 5::37]))        # (rows with a few dominant keys: chunk maxima far apart)
    for edge in edges:
        for past in (edge - 33, edge - 16, edge - 1, edge, edge + 1):
            ctx.reset()
            ctx.kv_import(0, 0, torch.from_numpy(np.ascontiguousarray(kk[0][:, :past])).cuda(), torch.from_numpy(np.ascontiguousarray(vv[0][:, :past])).cuda(), past)
            cache = om.new_cache(past + 40)
            cache.k[0][:, :past] = synth.bf16_to_f32(kk[0][:, :past])
            cache.v[0][:, :past] = synth.bf16_to_f32(vv[0][:, :past])
            want = om.forward(toks[:33], cache, past)
            single = []
            for j in range(33):
                ctx.set_pending(int(toks[j]))
                ctx.verify_step([])
                single.append(ctx.logits(1)[0].copy())
            single = np.stack(single)
            err = float(np.abs(single - want).max() / np.abs(want).max())
            assert err <= RTOL, past
            for k in (8, 16, 32):
                ctx.truncate(past)
                ctx.set_pending(int(toks[0]))
                ctx.verify_step(toks[1:1 + k])
                assert np.array_equal(ctx.logits(k + 1), single[:k + 1]), (past, k)
    ctx.close()


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("rising", [True, False])
def test_prompt_over_scores_that_rise_or_fall(dh, rising):
    """a prompt pass on top of an imported cache whose scores grow (or shrink) by far more than 2^8 from chunk to chunk: the running reference
    of a row moves at every chunk, or only at the first; rows that see all of a group of 32 positions and rows whose end lies inside"""
    import paper_2304_04487_amd as llma
    cfg = synth.ModelCfg("rising", 2, 2 * dh, 2, dh, 64, 128, "bf16")
    w = synth.make_weights(cfg, 6, gain_jitter=0.2)
    for lw in w["layers"]:
        lw["wo"] = synth.f32_to_bf16(10 * synth.bf16_to_f32(lw["wo"]))
        lw["wqkv"] = synth.f32_to_bf16(6 * synth.bf16_to_f32(lw["wqkv"]))
    om = OracleModel(cfg, w)
    ctx = llma.Context(cfg, w, max_seq=1024, max_batch=1, max_k=8)
    ctx.enable_logits_dump(9)
    toks = synth.uniform_tokens(4, 2, 200, cfg.vocab)
    for past, rows in ((700, 60), (673, 97)):
        ctx.reset()
        cache = om.new_cache(past + 120)
        ramp = 1 + np.arange(past) / 16.0
        for l in range(cfg.n_layers):
            kk, vv = synth.make_kv_fill(cfg, 19, 1, past, l)
            k = synth.f32_to_bf16(synth.bf16_to_f32(kk[0]) * (ramp if rising else ramp[::-1])[None, :, None].astype(np.float32))
            cache.k[l][:, :past] = synth.bf16_to_f32(k)
            cache.v[l][:, :past] = synth.bf16_to_f32(vv[0])
            ctx.kv_import(0, l, torch.from_numpy(k).cuda(), torch.from_numpy(vv[0]).cuda(), past)
        ctx.prefill(toks[:rows + 1])
        ctx.verify_step(toks[rows + 1:rows + 9])
        want = om.forward(toks[:rows + 9], cache, past)[rows:]
        err = float(np.abs(ctx.logits(9) - want).max() / np.abs(want).max())
        assert err <= RISING_RTOL, past
    ctx.close()

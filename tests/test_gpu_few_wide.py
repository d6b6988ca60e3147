"""Decode passes of 5 to 32 streams, whose GEMMs take several feature blocks to a workgroup: block counts that
leave the last workgroup half empty, K with whole and partial batches and with K split over workgroups, all
operand types; against the oracle stream by stream."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
L, NEW = 12, 2


# (heads, head dim, d_model, d_ffn, vocab): gate/up of 2 x d_ffn / 32 blocks (three to a workgroup from 257 on, also
# with one or two in the last), QKV of 264 blocks (two), FFN down and O with K in several parts, a head of 257 .. 1000
@pytest.mark.parametrize("hq,hkv,hd,d,F,vocab,operand", [
    (4, 1, 64, 128, 8240, 16416, "f16"), (128, 2, 64, 96, 4144, 8224, "bf16"), (12, 2, 128, 1536, 8960, 32000, "f16"),
    (4, 2, 64, 160, 8192, 8256, "f16w8")])
@pytest.mark.parametrize("B", [5, 32])
def test_decode_of_several_streams(hq, hkv, hd, d, F, vocab, operand, B):
    cfg = synth.ModelCfg(1, d, hq, hkv, hd, F, vocab)
    std = 1.0 / np.sqrt(d)
    rng = np.random.default_rng(B * d)
    emb = synth.round_bf16(rng.standard_normal((B, L, d))).astype(np.float32)
    first = rng.integers(0, vocab, B).tolist()
    gm = GpuModel(cfg, seed=3, max_batch=B, max_seq=32, std=std, operand=operand)
    try:
        gm.prefill(emb, 4)
        tokens, logits = gm.decode(B, L, NEW, first)
    finally:
        gm.close()
    om = oracle_model(cfg, seed=3, std=std, w8=operand == "f16w8")
    tol = 8e-2 if operand == "bf16" else 2e-2
    for b in sorted({0, 1, B // 2, B - 1}):
        cache = O.new_cache(cfg, 32)
        O.dense_forward(om, emb[b], 4, cache)
        toks, want = O.decode(om, cache, L, first[b], NEW, return_logits=True)
        assert np.abs(logits[b, 0] - want[0]).max() <= tol
        if int(tokens[b, 0]) == toks[0]:
            assert np.abs(logits[b, 1] - want[1]).max() <= tol

"""Decode passes of 5 to 32 streams, whose GEMMs take several feature blocks to a workgroup: block counts that
leave the last workgroup half empty, K with whole and partial batches and with K split over workgroups, all
operand types; against the oracle stream by stream, and bit for bit against libvlac_safe.so, which takes one
feature block to a workgroup."""
import os

import numpy as np
import pytest

import paper_2502_02175_amd as V
import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
L, NEW = 12, 2
SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")


# (heads, head dim, d_model, d_ffn, vocab): gate/up of 2 x d_ffn / 32 blocks (three to a workgroup from 257 on, also
# with one or two in the last), FFN down and O with K in several parts, a head of 257 .. 1001; QKV of 264 blocks (two at a
# d_model of 1056, where FFN down and O are 33 blocks in 8 parts, the head 1001 blocks, four to a workgroup)
SHAPES = [
    (4, 1, 64, 128, 8240, 16416, "f16"), (128, 2, 64, 96, 4144, 8224, "bf16"), (12, 2, 128, 1536, 8960, 32000, "f16"),
    (4, 2, 64, 160, 8192, 8256, "f16w8")]
WIDE = [(128, 2, 64, 1056, 8240, 32032, o) for o in ("f16", "bf16", "f16w8")]


@pytest.mark.parametrize("hq,hkv,hd,d,F,vocab,operand", SHAPES + WIDE[:1])
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
        second, first_choice = np.sort(want[0])[-2:]
        if first_choice - second > 2 * tol:
            assert int(tokens[b, 0]) == toks[0]
        if int(tokens[b, 0]) == toks[0]:
            assert np.abs(logits[b, 1] - want[1]).max() <= tol


def run(cfg, B, operand):
    rng = np.random.default_rng(B)
    emb = synth.round_bf16(rng.standard_normal((B, L, cfg.d_model))).astype(np.float32)
    gm = GpuModel(cfg, seed=3, max_batch=B, max_seq=32, std=1.0 / np.sqrt(cfg.d_model), gen_device="cuda:0", operand=operand)
    try:
        gm.prefill(emb, 4)
        return (*gm.decode(B, L, NEW, rng.integers(0, cfg.vocab, B).tolist()), gm.kv.cpu().numpy().copy())
    finally:
        gm.close()


@pytest.mark.parametrize("hq,hkv,hd,d,F,vocab,operand", SHAPES + WIDE)
@pytest.mark.parametrize("B", [1, 4, 5, 17, 32])
def test_several_feature_blocks_change_no_bit(hq, hkv, hd, d, F, vocab, operand, B):
    """Up to 4 streams only the projections with a residual have a choice (the others make their norm themselves)."""
    assert os.path.exists(SAFE), "libvlac_safe.so is not built (python -m paper_2502_02175_amd.build)"
    cfg = synth.ModelCfg(1, d, hq, hkv, hd, F, vocab)
    try:
        V.use_library(None)
        want = run(cfg, B, operand)
        V.use_library(SAFE)
        got = run(cfg, B, operand)
    finally:
        V.use_library(None)
    assert np.isfinite(want[1]).all()
    for name, w, g in zip(("tokens", "logits", "cache"), want, got):
        np.testing.assert_array_equal(w, g, err_msg=name)

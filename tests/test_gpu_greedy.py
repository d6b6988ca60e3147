"""The greedy token is not taken from the logits themselves but from (greatest logit, its token) pairs that the
head's epilogue leaves per block of 32 features (combined over the two lane halves of a block, and then
over the blocks): it must be the first of the greatest of the returned logits all the same, in every kernel that
runs the head.  Here ties are the rule: head rows are copies of each other within a lane half (tokens that
differ in the bits 0, 1, 3 and 4), across the halves (bit 2) and across blocks; and no NaN wins."""
import numpy as np
import pytest

import synth
from helpers import GpuModel

pytestmark = pytest.mark.gpu
VOCAB = 96 + 32 * 40


def tied_head(cfg, seed, nan):
    import torch
    head = synth.make_head(cfg, seed, std=0.2)
    w = head["w_head"].clone()
    rng = np.random.default_rng(seed)
    loud = rng.permutation(np.arange(64, VOCAB - 64))[:24].tolist()
    copies = {}
    for i, t in enumerate(loud):
        row = (w[t].float() * 4).bfloat16()
        base = t & ~31
        other = {0: t ^ 1, 1: t ^ 8, 2: t ^ 16, 3: t ^ 4, 4: t ^ 20, 5: (base + 32 + (t & 31) ^ 5) % VOCAB}[i % 6]
        w[t] = w[other] = row
        copies[i % 6] = copies.get(i % 6, []) + [(min(t, other), max(t, other))]
    if nan:
        w[3] = w[VOCAB - 1] = float("nan")
        w[loud[0]] = float("nan")
    head["w_head"] = w
    return {k: v.to("cuda:0") for k, v in head.items()}, copies, torch


def first_greatest(x):
    return np.where(np.isnan(x), -np.inf, x).argmax(-1)  # (numpy: the first of equals)


# 1 and 4 streams: the norm fused into the head; 8: rows of an operand; 33 and 300: the one-stream kernel;
# 512: the many-rows kernel (16-bit weights), the one-stream kernel (8-bit weights)
@pytest.mark.parametrize("B", [1, 4, 8, 33, 300, 512])
@pytest.mark.parametrize("operand,nan", [("f16", False), ("bf16", True), ("f16w8", False)])
def test_token_is_the_first_of_the_greatest_logits(B, operand, nan):
    cfg = synth.ModelCfg(1, 64, 4, 4, 64, 96, VOCAB)
    n_vis, n_txt, n_new = 4, 4, 6
    gm = GpuModel(cfg, seed=2, max_batch=B, max_seq=32, std=0.1, operand=operand)
    try:
        head, copies, torch = tied_head(cfg, 5, nan)
        gm.V.vlac_set_head_weights(gm.ctx, head["g_final"], head["w_head"], head["embed"])
        rng = np.random.default_rng(B)
        ties = 0
        for _ in range(max(1, 24 // B)):
            emb = synth.round_bf16(rng.standard_normal((B, n_vis + n_txt, cfg.d_model)))
            got = gm.prefill(emb, n_vis)
            want = first_greatest(got["logits"])
            assert np.array_equal(got["token"], want)
            tok, logits = gm.decode(B, n_vis + n_txt, n_new, got["token"])
            assert np.array_equal(tok, first_greatest(logits))
            # the token that was looked up for the next pass is the one that was returned
            again, l2 = gm.decode(B, n_vis + n_txt, n_new, got["token"])
            assert np.array_equal(tok, again) and np.array_equal(logits, l2, equal_nan=True)
            top = np.nanmax(logits, -1, keepdims=True)
            ties += int(((logits == top).sum(-1) > 1).sum()) + int((got["logits"] == np.nanmax(got["logits"], -1, keepdims=True)).sum(-1).max() > 1)
        assert ties >= 4  # (about half of the tied rows are the greatest for some stream)
        if nan:
            assert np.isnan(got["logits"]).any()
    finally:
        gm.close()


def test_every_kind_of_tie_is_met():
    """Over many streams each way of being tied (within a lane half, across the halves, across blocks)
    decides tokens, and always for the lower one."""
    cfg = synth.ModelCfg(1, 64, 4, 4, 64, 96, VOCAB)
    B = 300
    gm = GpuModel(cfg, seed=2, max_batch=B, max_seq=32, std=0.1)
    try:
        head, copies, torch = tied_head(cfg, 5, False)
        gm.V.vlac_set_head_weights(gm.ctx, head["g_final"], head["w_head"], head["embed"])
        emb = synth.round_bf16(np.random.default_rng(1).standard_normal((B, 8, cfg.d_model)))
        got = gm.prefill(emb, 4)
        won = set(got["token"].tolist())
        for kind, pairs in copies.items():
            assert any(lo in won for lo, hi in pairs), kind
            assert all(np.array_equal(got["logits"][:, lo], got["logits"][:, hi]) for lo, hi in pairs), kind
            assert not any(hi in won for lo, hi in pairs), kind
    finally:
        gm.close()

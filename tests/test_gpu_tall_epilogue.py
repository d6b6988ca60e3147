"""What the many-rows GEMM does with its sums: query, key and value blocks of weight-tile counts that its
order of tiles treats differently (1 to 11 tiles, whole and half-filled last ones), residual rows and
partial rows turned round in LDS, with row counts that leave ragged row tiles, counted by the host and by
the device; against the oracle, and bit for bit against the build with full waits."""
import os

import numpy as np
import pytest

import synth
import paper_2502_02175_amd as V
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")
B, L, N_TXT = 2, 400, 8
LEFT = (515, 321, 97, 33)   # rows that the reuse lists of both streams leave


def passes(cfg, operand, emb, keeps):
    gm = GpuModel(cfg, seed=9, max_batch=B, max_seq=416, std=1.0 / np.sqrt(cfg.d_model), operand=operand)
    try:
        out = [gm.prefill(emb, L - N_TXT)]
        for i, k in enumerate(keeps):
            out.append(gm.prefill(emb + np.float32(0.125) * (i + 1), L - N_TXT, k))
        return out
    finally:
        gm.close()


# heads -> feature blocks of QKV: 12 (2 tiles), 8 (1), 40 (5), 88 (11), 64 (8)
@pytest.mark.parametrize("hq,hkv,hd,d,F,operand", [(4, 1, 64, 96, 208, "f16"), (4, 2, 64, 256, 688, "bf16"),
                                                   (12, 4, 64, 320, 528, "f16"), (36, 4, 64, 288, 1200, "f16"),
                                                   (12, 2, 128, 1536, 640, "f16")])
def test_many_rows_epilogues(hq, hkv, hd, d, F, operand):
    cfg = synth.ModelCfg(2, d, hq, hkv, hd, F, 96)
    rng = np.random.default_rng(d)
    emb = synth.round_bf16(rng.standard_normal((B, L, d))).astype(np.float32)
    keeps = []
    for left in LEFT:
        first = min(L - N_TXT, (2 * L - left) // 2 + 5)
        keeps.append([rng.permutation(L - N_TXT)[:n].tolist() for n in (first, min(L - N_TXT, 2 * L - left - first))])
    got = passes(cfg, operand, emb, keeps)
    try:
        V.use_library(SAFE)
        safe = passes(cfg, operand, emb, keeps)
    finally:
        V.use_library(None)
    for a, b in zip(got, safe):
        for k in ("hidden", "logits", "attn_mean"):
            assert np.array_equal(a[k], b[k], equal_nan=True)
    tol = 2e-2 if operand == "f16" else 8e-2
    om = oracle_model(cfg, seed=9, std=1.0 / np.sqrt(d))
    for b in range(B):
        cache = O.new_cache(cfg, 416)
        want = O.dense_forward(om, emb[b], L - N_TXT, cache)
        assert np.abs(got[0]["hidden"][b] - want["hidden"]).max() <= tol
        for i, k in enumerate(keeps):
            want = O.sparse_forward(om, emb[b] + np.float32(0.125) * (i + 1), L - N_TXT, cache, [k[b]] * 2)
            alive = ~np.isnan(want["hidden"][:, 0])
            assert np.abs(got[i + 1]["hidden"][b][alive] - want["hidden"][alive]).max() <= tol, (b, LEFT[i])

"""The one-stream GEMM kernel at the edges of its tiles: row counts around multiples of 32 and of
its blocks of 6 or 8 row tiles, 2 to 6 feature blocks per workgroup with a ragged last one, K in two parts or whole, K ranges
shorter and longer than what a wave has in flight and of unequal parts, 16-bit and 8-bit weights.
Against the oracle; the tolerance is that of the operand roundings."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
TOL = {"f16": 2e-2, "f16w8": 2e-2, "bf16": 8e-2}


@pytest.mark.parametrize("d,F,hq,operand", [
    (64, 272, 4, "f16"),       # one step of K: the second part has none
    (64, 272, 4, "f16w8"),
    (128, 272, 4, "f16"),      # 2 blocks per workgroup everywhere, K of 2 to 5 steps
    (320, 8240, 4, "f16"),     # gate/up: 515 blocks, 3 per workgroup (172), 5 with two row blocks; FFN down: 129 steps
    (576, 12320, 4, "f16"),    # gate/up: 770 blocks, 4 per workgroup (193); 36 k-tiles
    (576, 8240, 4, "bf16"),
    (1344, 1008, 4, "f16"),    # K of 21 steps in two parts of 11 and 10
    (320, 8240, 4, "f16w8"),
    (1344, 1008, 4, "f16w8"),
    (320, 272, 128, "f16"),    # QKV: 264 blocks, K in two parts, 2 per workgroup (132), 3 from 7 row tiles on (88, two row blocks)
    (320, 272, 128, "f16w8"),
    (128, 272, 256, "f16"),    # QKV: 520 blocks, K whole, 3 to 6 per workgroup
    (1536, 2048, 4, "bf16"),   # FFN down: 24 x 5 workgroups, 13 to 16 row tiles in two blocks
])
def test_rows_gemm_at_the_edges(d, F, hq, operand):
    cfg = synth.ModelCfg(2, d, hq, 2, 64, F, 96)
    std = 1.0 / np.sqrt(d)
    om = oracle_model(cfg, seed=2, std=std, w8=operand == "f16w8")
    gm = GpuModel(cfg, seed=2, max_batch=1, max_seq=512, std=std, operand=operand)
    try:
        n_vis = 496
        rng = np.random.default_rng(d + F)
        emb = synth.round_bf16(rng.standard_normal((n_vis + 8, d)))
        for L in (33, 64, 161, 193, 225, 256):            # row counts that the host knows
            cache = O.new_cache(cfg, 512)
            want = O.dense_forward(om, emb[-L:], L - 8, cache)
            got = gm.prefill(emb[None, -L:], L - 8)
            assert np.abs(got["hidden"][0] - want["hidden"]).max() <= TOL[operand], L
            assert np.abs(got["logits"][0] - want["logits"]).max() <= TOL[operand], L
        cache = O.new_cache(cfg, 512)
        O.dense_forward(om, emb, n_vis, cache)
        gm.prefill(emb[None], n_vis)
        for rows in (31, 97, 130, 211, 250, 385, 409, 490):         # ... and those that it does not
            keep = rng.permutation(n_vis)[:n_vis + 8 - rows].tolist()
            emb2 = synth.round_bf16(emb + 0.1 * rng.standard_normal(emb.shape))
            want = O.sparse_forward(om, emb2, n_vis, cache, [keep] * 2)
            got = gm.prefill(emb2[None], n_vis, [keep])
            alive = ~np.isnan(want["hidden"][:, 0])
            assert alive.sum() == rows
            assert np.abs(got["hidden"][0][alive] - want["hidden"][alive]).max() <= TOL[operand], rows
            assert np.abs(got["attn_mean"][:, 0] - want["attn_mean"]).max() <= TOL[operand], rows
    finally:
        gm.close()

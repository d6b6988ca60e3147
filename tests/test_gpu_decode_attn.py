"""Attention of the decode passes at the edges of its launch shapes: the positions where a wave
per key tile turns into waves that walk several, query heads that fill a part of a tile, a whole
one or more than one, and the LDS that the waves' parts take.  Logits against the oracle; the
tolerance is the operand rounding's, as everywhere."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("hq,hkv,hd,L", [
    (4, 4, 64, 30),      # one tile, then two
    (4, 4, 64, 510),     # sixteen tiles (one per wave), then seventeen (8 waves)
    (4, 2, 128, 511),
    (12, 2, 128, 1055),  # 6 columns; 33 tiles over 8 waves, then 34
    (32, 1, 64, 255),    # a whole tile of query heads
    (32, 1, 128, 255),   # ... whose parts fit LDS for 8 waves only: 8 tiles, then 9
    (40, 1, 64, 100),    # more query heads than a tile has columns
])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_decode_attention_at_the_edges(hq, hkv, hd, L, operand):
    cfg = synth.ModelCfg(2, 128, hq, hkv, hd, 160, 128)
    B, n_new, tol = 2, 3, TOL if operand == "f16" else 8e-2
    om = oracle_model(cfg, seed=5, std=0.05)
    gm = GpuModel(cfg, seed=5, max_batch=B, max_seq=(L + n_new + 31) // 32 * 32, std=0.05, operand=operand)
    try:
        emb = synth.round_bf16(np.random.default_rng(L + hq).standard_normal((B, L, cfg.d_model)))
        gm.prefill(emb, 0, want_stats=False, want_hidden=False)
        caches, first = [], []
        for b in range(B):
            caches.append(O.new_cache(cfg, gm.max_seq))
            first.append(O.dense_forward(om, emb[b], 0, caches[b])["token"])
        gt, gl = gm.decode(B, L, n_new, first)
        for b in range(B):
            tok = first[b]
            for t in range(n_new):  # the oracle follows the GPU's tokens, so every pass is compared
                want_tok, logits = O.decode(om, caches[b], L + t, tok, 1, return_logits=True)
                assert np.abs(gl[b, t] - logits[0]).max() <= tol, (b, t)
                top = np.sort(logits[0])
                if top[-1] - top[-2] > 2 * tol:
                    assert int(gt[b, t]) == want_tok[0]
                tok = int(gt[b, t])
    finally:
        gm.close()

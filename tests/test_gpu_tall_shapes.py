"""The many-rows GEMM's work items of 192 features (192 and 320 rows tall) beside those of 256: row
counts known to the host and not, ragged last blocks and last feature tiles, both operand types, and
bit for bit against the build whose hand-placed waits are full ones."""
import os

import numpy as np
import pytest

import synth
import paper_2502_02175_amd as V
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
KNOWN = (288, 320, 353, 404, 519, 640, 704)   # row counts of full prefills (of one stream's 736: below 512 rows the one-stream kernel, same oracle)
SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")


def passes(cfg, operand, emb, n_vis, keeps, std):
    gm = GpuModel(cfg, seed=4, max_batch=1, max_seq=736, std=std, operand=operand)
    try:
        out = []
        for L in KNOWN:
            out.append(gm.prefill(emb[None, -L:], L - 8))
        gm.prefill(emb[None], n_vis)
        for i, k in enumerate(keeps):
            out.append(gm.prefill(emb[None] + np.float32(0.125) * (i + 1), n_vis, [k]))
        return out
    finally:
        gm.close()


# (11008: gate/up of 688 feature blocks, 115 tiles of 192 features, the last of 4 blocks; 284 to 644 rows are
# what the reuse lists below leave of 704)
ITEMS = {284: (192, 192), 320: (192, 192), 353: (192, 192), 404: (256, 256), 519: (192, 320), 640: (192, 320), 644: (192, 192),
         704: (192, 192)}


@pytest.mark.parametrize("d,F,operand", [(320, 11008, "f16"), (256, 11008, "bf16")])
def test_items_of_192_features(d, F, operand):
    cfg = synth.ModelCfg(2, d, 4, 4, 64, F, 96)
    std, tol = 1.0 / np.sqrt(d), 2e-2 if operand == "f16" else 8e-2
    n_vis = 696
    rng = np.random.default_rng(d)
    emb = synth.round_bf16(rng.standard_normal((n_vis + 8, d))).astype(np.float32)
    for rows, items in ITEMS.items():  # which items the gate/up projection of each count runs
        assert V.vlac_plan_unsplit_gemm(2 * F, rows, 704)[:2] == items, rows
    keeps = [rng.permutation(n_vis)[:n].tolist() for n in (60, 185, 300, 351, 384, 420)]
    got = passes(cfg, operand, emb, n_vis, keeps, std)
    try:
        V.use_library(SAFE)
        safe = passes(cfg, operand, emb, n_vis, keeps, std)
    finally:
        V.use_library(None)
    for a, b in zip(got, safe):
        for k in ("hidden", "logits", "attn_mean"):
            assert np.array_equal(a[k], b[k], equal_nan=True)
    om = oracle_model(cfg, seed=4, std=std)
    for i, L in enumerate(KNOWN):
        want = O.dense_forward(om, emb[-L:], L - 8, O.new_cache(cfg, 736))
        assert np.abs(got[i]["hidden"][0] - want["hidden"]).max() <= tol, L
    cache = O.new_cache(cfg, 736)
    O.dense_forward(om, emb, n_vis, cache)
    for i, k in enumerate(keeps):
        want = O.sparse_forward(om, emb + np.float32(0.125) * (i + 1), n_vis, cache, [k] * 2)
        alive = ~np.isnan(want["hidden"][:, 0])
        assert np.abs(got[len(KNOWN) + i]["hidden"][0][alive] - want["hidden"][alive]).max() <= tol, len(k)

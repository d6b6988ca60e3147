"""Rows of more than 4096 values, whose row kernels keep 8 x 4 values per thread, ask for partial rows in two batches from
five parts on and make the final norm on the way, and whose plain norm reads the row twice: full and sparse prefills in
which the projections with a residual split K in 7, 6 and 4 parts (one-stream kernel, up to 511 rows) and as the many-rows
kernel does (600 rows, counted by the host and by the device), and a decode of five streams; against the oracle."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
N_TXT = 10


@pytest.mark.parametrize("d,F,operand", [(4128, 8192, "f16"), (5120, 8192, "bf16"), (8192, 8192, "f16")])
def test_rows_of_more_than_4096_values(d, F, operand):
    cfg = synth.ModelCfg(1, d, 4, 2, 64, F, 96)
    std = 1.0 / np.sqrt(d)
    om = oracle_model(cfg, seed=4, std=std)
    tol = 2e-2 if operand == "f16" else 8e-2
    rng = np.random.default_rng(d)
    gm = GpuModel(cfg, seed=4, max_batch=5, max_seq=320, std=std, operand=operand)
    try:
        for B, L, left in ((1, 190, (35, 150)), (2, 300, (90, 470))):
            emb = synth.round_bf16(rng.standard_normal((B, L, d))).astype(np.float32)
            caches = [O.new_cache(cfg, 320) for _ in range(B)]
            got = gm.prefill(emb, L - N_TXT)
            for b in range(B):
                want = O.dense_forward(om, emb[b], L - N_TXT, caches[b])
                assert np.abs(got["hidden"][b] - want["hidden"]).max() <= tol
                assert np.abs(got["logits"][b] - want["logits"]).max() <= tol
            for i, n in enumerate(left):
                e = emb + np.float32(0.125 * (i + 1))
                reuse = [rng.permutation(L - N_TXT)[:L - n // B].tolist() for _ in range(B)]
                got = gm.prefill(e, L - N_TXT, reuse)
                for b in range(B):
                    want = O.sparse_forward(om, e[b], L - N_TXT, caches[b], [reuse[b]])
                    alive = ~np.isnan(want["hidden"][:, 0])
                    assert np.array_equal(alive, ~np.isnan(got["hidden"][b][:, 0]))
                    assert np.abs(got["hidden"][b][alive] - want["hidden"][alive]).max() <= tol
                    assert np.abs(got["logits"][b] - want["logits"]).max() <= tol
        B, L = 5, 12
        emb = synth.round_bf16(rng.standard_normal((B, L, d))).astype(np.float32)
        got = gm.prefill(emb, L - N_TXT)
        first = rng.integers(0, cfg.vocab, B).tolist()
        _, logits = gm.decode(B, L, 1, first)
        for b in range(B):
            cache = O.new_cache(cfg, 320)
            want = O.dense_forward(om, emb[b], L - N_TXT, cache)
            assert np.abs(got["hidden"][b] - want["hidden"]).max() <= tol
            _, want = O.decode(om, cache, L, first[b], 1, return_logits=True)
            assert np.abs(logits[b, 0] - want[0]).max() <= tol
    finally:
        gm.close()

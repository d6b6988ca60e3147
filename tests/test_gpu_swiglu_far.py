"""SwiGLU where many gates lie beyond +-87, so that the quick quotient does not serve and the stores are made again, and
others are small or zero: every kernel with that epilogue (up to 32 rows with one and with several
feature blocks, one-stream, many-rows), against the oracle and bit for bit against the build with full waits."""
import os

import numpy as np
import pytest

import paper_2502_02175_amd as V
import synth
from oracle import vlac_oracle as O
from helpers import GpuModel

pytestmark = pytest.mark.gpu
SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")
D, SEED, N_TXT = 128, 6, 8


def model(F):
    cfg = synth.ModelCfg(1, D, 4, 2, 64, F, 96)
    w = dict(synth.make_layer(cfg, SEED, 0, std=1.0 / np.sqrt(D), gain_jitter=0.1))
    gu = w["w_gate_up"].clone()
    gu[:F] *= 64.0          # gates of some -250 .. 250; a block of them is zero
    gu[16:32] = 0.0
    w["w_gate_up"] = gu
    w["w_down"] = w["w_down"] / 32.0
    head = {k: v.float().numpy() for k, v in synth.make_head(cfg, SEED, gain_jitter=0.1, std=1.0 / np.sqrt(D)).items()}
    f64 = {k: v.float().numpy() for k, v in w.items()}
    return cfg, w, O.Model(cfg, lambda l: f64, head)


def run(cfg, w, emb, operand, decode):
    B, L, _ = emb.shape
    gm = GpuModel(cfg, SEED, max_batch=B, max_seq=(L + 33) // 32 * 32, std=1.0 / np.sqrt(D), operand=operand,
                  layer_source=lambda l: w)
    try:
        out = gm.prefill(emb, L - N_TXT)
        return out["hidden"], (gm.decode(B, L, 1, [5] * B)[1][:, 0] if decode else out["logits"])
    finally:
        gm.close()


# streams, tokens, FFN width (4224: gate/up of 264 blocks, two to a workgroup)
@pytest.mark.parametrize("B,L,F,decode", [(1, 10, 272, True), (5, 10, 4224, True), (1, 150, 272, False), (2, 300, 1040, False)])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_gates_beyond_87(B, L, F, decode, operand):
    cfg, w, om = model(F)
    emb = synth.round_bf16(np.random.default_rng(L).standard_normal((B, L, D))).astype(np.float32)
    hidden, logits = run(cfg, w, emb, operand, decode)
    try:
        V.use_library(SAFE)
        safe = run(cfg, w, emb, operand, decode)
    finally:
        V.use_library(None)
    assert np.array_equal(hidden, safe[0]) and np.array_equal(logits, safe[1])
    tol = 2e-2 if operand == "f16" else 8e-2
    for b in range(B):
        cache = O.new_cache(cfg, L + 8)
        want = O.dense_forward(om, emb[b], L - N_TXT, cache)
        assert np.abs(hidden[b] - want["hidden"]).max() <= tol
        ref = O.decode(om, cache, L, 5, 1, return_logits=True)[1][0] if decode else want["logits"]
        assert np.abs(logits[b] - ref).max() <= tol

"""The kernels that copy operand tiles global -> LDS with instructions the compiler does not
see (the one-stream and the many-rows GEMM of Alg. 2's recomputed rows, the attention kernel with
one query tile per wave) wait for those copies with hand-counted `s_waitcnt vmcnt(n)`.
libvlac_safe.so is the same library with every such wait replaced by a wait for everything; it
computes the same values in the same order.  Here both builds run the same prefills, over every
specialisation of those kernels (feature blocks per wave or workgroup, active row tiles, K steps
modulo the ring sizes, row-block sizes, both head dims, operand types), and every output and the
whole KV cache must agree BIT FOR BIT: an LDS read that overtakes its copy shows as a difference,
where a tolerance against the oracle could hide it."""
import os

import numpy as np
import pytest

import synth
import paper_2502_02175_amd as V
from helpers import GpuModel

pytestmark = pytest.mark.gpu
SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")

CASES = [
    # name, cfg, streams, visual, text tokens, reused tokens per prefill (per stream: k + 3 (b % 3))
    ("K steps 4 / 11", synth.ModelCfg(2, 256, 4, 4, 64, 688, 256), 6, 120, 24, (0, 10, 37, 61, 88, 110)),
    ("K steps 5 / 4 / 6", synth.ModelCfg(2, 320, 4, 4, 64, 384, 256), 6, 120, 24, (0, 10, 37, 61, 88, 110)),
    ("K steps 6 / 8 / 7", synth.ModelCfg(2, 384, 4, 2, 128, 448, 256), 6, 120, 24, (0, 10, 37, 61, 88, 110)),
    # wide enough for row blocks of 256 and 192 rows, long and many enough for the attention
    # kernel with one query tile per wave (streams with 65 rows or more), head dim 64 and 128
    ("head dim 64, 12 streams x 352", synth.ModelCfg(2, 1024, 16, 4, 64, 2816, 256), 12, 320, 32, (0, 150, 270)),
    ("head dim 128, 22 streams x 352", synth.ModelCfg(2, 1024, 8, 8, 128, 2816, 256), 22, 320, 32, (0, 200, 290)),
]


def run_case(cfg, B, n_vis, n_txt, reuse_counts, seed):
    import torch
    L = n_vis + n_txt
    rng = np.random.default_rng(seed)
    emb = synth.round_bf16(rng.standard_normal((len(reuse_counts) + 1, B, L, cfg.d_model)))
    gm = GpuModel(cfg, seed, max_batch=B, max_seq=(L + 31) // 32 * 32, std=0.05, gen_device="cuda:0")
    outs = []
    try:
        outs.append(gm.prefill(emb[0], n_vis))
        for i, k in enumerate(reuse_counts):
            reuse = [sorted(rng.permutation(n_vis)[:min(n_vis, k + 3 * (b % 3))].tolist()) for b in range(B)]
            if i == len(reuse_counts) - 1:       # one stream with few rows, one with nothing reused
                reuse[0] = list(range(n_vis - 8))
                reuse[1] = []
            outs.append(gm.prefill(emb[i + 1], n_vis, reuse))
        kv = gm.kv.cpu().numpy().copy()
    finally:
        gm.close()
    return outs, kv


@pytest.mark.parametrize("name,cfg,B,n_vis,n_txt,reuse_counts", CASES, ids=[c[0] for c in CASES])
def test_full_waits_change_no_bit(name, cfg, B, n_vis, n_txt, reuse_counts):
    assert os.path.exists(SAFE), "libvlac_safe.so is not built (python -m paper_2502_02175_amd.build)"
    try:
        V.use_library(None)
        ref, kv_ref = run_case(cfg, B, n_vis, n_txt, reuse_counts, seed=17)
        V.use_library(SAFE)
        got, kv_got = run_case(cfg, B, n_vis, n_txt, reuse_counts, seed=17)
    finally:
        V.use_library(None)
    assert np.isfinite(ref[0]["logits"]).all()
    for r, g in zip(ref, got):
        for key in ("logits", "token", "attn_mean", "hidden"):
            np.testing.assert_array_equal(r[key], g[key], err_msg=key)
    np.testing.assert_array_equal(kv_ref, kv_got)


# The one-stream GEMM (up to a capacity of 511 rows; 8-bit weights: up to 1023).  Its ring holds 5 chunks of
# 8 k-tiles (4 with more than 4 row tiles; half of that per part where two sets of waves share K).
ONE_STREAM = [
    # d, F, query heads, head dim, layers, operand: feature blocks per workgroup (QKV, gate/up, residual) and k-tiles of K
    (64, 272, 4, 64, 2, "f16"),       # 2, 2, 2; 4 k-tiles: one chunk, and a part of K that has none
    (128, 272, 4, 64, 2, "f16w8"),    # 2, 2, 2; 8 and 20 k-tiles: fewer chunks than the ring holds
    (320, 8240, 4, 64, 2, "f16"),     # 2, 3, 2; 20 and 516 k-tiles: as many chunks as the ring, and far more
    (320, 8240, 4, 64, 2, "f16w8"),
    (576, 12320, 4, 64, 2, "bf16"),   # 2, 4, 2; 36 k-tiles
    (1344, 1008, 4, 64, 2, "f16"),    # 2, 2, 2; 84 k-tiles in parts of 44 and 40
    (320, 272, 128, 64, 2, "bf16"),   # 2 or 3 by the row count, 2, 2; 20 k-tiles in parts of 12 and 8
    (320, 272, 128, 64, 2, "f16w8"),
    (128, 272, 256, 64, 1, "f16"),    # 3 to 6 by the row count, 2, 2; 8 and 1024 k-tiles
    (4096, 8256, 64, 128, 1, "f16"),   # 2 or 3, 4, 4: the residual projections over 4 feature blocks; enough workgroups
                                       # everywhere for 7 and 8 row tiles in one block
    (4096, 8256, 64, 128, 1, "f16w8"),
]


def run_one_stream(d, F, hq, hd, layers, operand, known, unknown):
    """Full prefills of `known` rows (a count the host has), sparse ones that leave `unknown` rows."""
    cfg = synth.ModelCfg(layers, d, hq, 2, hd, F, 96)
    top = max(known + unknown)
    L = max(unknown) + 40
    rng = np.random.default_rng(d + F)
    emb = synth.round_bf16(rng.standard_normal((max(top, L), d)))
    gm = GpuModel(cfg, 3, max_batch=1, max_seq=(max(top, L) + 31) // 32 * 32, std=1.0 / np.sqrt(d), gen_device="cuda:0",
                  operand=operand)
    try:
        outs = [gm.prefill(emb[None, :n], n - 8) for n in known]
        outs.append(gm.prefill(emb[None, :L], L - 8))
        for n in unknown:
            outs.append(gm.prefill(emb[None, :L] + np.float32(n / 1024.0), L - 8, [rng.permutation(L - 8)[:L - n].tolist()]))
        return outs, gm.kv.cpu().numpy().copy()
    finally:
        gm.close()


@pytest.mark.parametrize("d,F,hq,hd,layers,operand", ONE_STREAM)
def test_full_waits_change_no_bit_of_the_one_stream_gemm(d, F, hq, hd, layers, operand):
    """1 to 8 row tiles in one block where the launch allows, 2 blocks and more of equal and unequal
    size, full and ragged last tiles."""
    known = [33, 64, 95, 129, 161, 193, 225, 256]
    unknown = [34, 70, 127, 150, 190, 211, 256, 290, 409, 470]
    if operand == "f16w8":
        known += [288, 500, 993]
        unknown += [600]
    try:
        V.use_library(None)
        ref, kv_ref = run_one_stream(d, F, hq, hd, layers, operand, known, unknown)
        V.use_library(SAFE)
        got, kv_got = run_one_stream(d, F, hq, hd, layers, operand, known, unknown)
    finally:
        V.use_library(None)
    assert np.isfinite(ref[0]["logits"]).all()
    for i, (r, g) in enumerate(zip(ref, got)):
        for key in ("logits", "token", "attn_mean", "hidden"):
            np.testing.assert_array_equal(r[key], g[key], err_msg="%s of pass %d" % (key, i))
    np.testing.assert_array_equal(kv_ref, kv_got)

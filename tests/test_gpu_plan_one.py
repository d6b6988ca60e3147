"""The plan of a single stream (one launch) against the plan of several (two launches): which rows every layer
recomputes, for lists and per-layer counts that have to be clamped, sequence lengths around the 256 positions
that a workgroup takes at a time, and lists with entries that must be reported."""
import numpy as np
import pytest

import synth
import paper_2502_02175_amd as V
from helpers import GpuModel

pytestmark = pytest.mark.gpu
LAYERS = 5


def alive(emb, n_vis, order, counts, B):
    gm = GpuModel(synth.ModelCfg(LAYERS, 64, 4, 2, 64, 96, 64), seed=2, max_batch=B, max_seq=544, std=0.05)
    try:
        e = np.repeat(emb[None], B, 0)
        gm.prefill(e, n_vis)
        got = gm.prefill(e + np.float32(0.25), n_vis, [order] * B, None if counts is None else [counts] * B)
        return got["hidden"], got["attn_mean"]
    finally:
        gm.close()


@pytest.mark.parametrize("n_vis,n_txt,n_list", [(1, 1, 1), (200, 9, 0), (250, 6, 250), (250, 7, 120), (511, 20, 300)])
@pytest.mark.parametrize("counts", [None, [0, 10**6, 3, 50, -4], [-1, 7, 20, 20, 400], [9, 8, 7, 6, 5]])
def test_one_stream_plans_as_several(n_vis, n_txt, n_list, counts):
    rng = np.random.default_rng(n_vis + n_list)
    emb = synth.round_bf16(rng.standard_normal((n_vis + n_txt, 64))).astype(np.float32)
    order = rng.permutation(n_vis)[:n_list].tolist()
    one, s1 = alive(emb, n_vis, order, counts, 1)
    two, s2 = alive(emb, n_vis, order, counts, 2)
    cnt = len(order)
    m = max([0] + [min(max(c, 0), cnt) for c in (counts if counts is not None else [cnt])])
    want = np.ones(n_vis + n_txt, dtype=bool)
    want[order[:m]] = False
    for h in (one[0], two[0], two[1]):
        assert np.array_equal(~np.isnan(h[:, 0]), want)
    # (the K splits follow the capacity of the call: fp16 roundings apart)
    assert np.abs(one[0][want] - two[1][want]).max() <= 2e-2 and np.abs(s1[:, 0] - s2[:, 1]).max() <= 2e-2


@pytest.mark.parametrize("order", [[3, 3, 5], [1, 99], [-1, 2]])
def test_bad_entries_are_reported(order):
    gm = GpuModel(synth.ModelCfg(1, 64, 4, 2, 64, 96, 64), seed=2, max_batch=1, max_seq=32, std=0.05)
    try:
        emb = np.zeros((1, 20, 64), np.float32)
        gm.prefill(emb, 16)
        with pytest.raises(V.VlacError):
            gm.prefill(emb, 16, [order])
    finally:
        gm.close()

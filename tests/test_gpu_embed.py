"""GPU parity of vlac_embed_patches (the patch -> embedding projection for the recomputed
patches only) against the oracle, alone and feeding the sparse prefill."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu


def run_embed(gm, frames, patch, w_proj, reuse=None, layer_count=None, L=None, fill=-123.0):
    import torch
    V, dev = gm.V, gm.device
    B, H, W, _ = frames.shape
    L_v = (H // patch) * (W // patch)
    L = L or L_v
    out = torch.full((B, L, gm.cfg.d_model), fill, device=dev)
    ro = rc = lc = None
    stride = 1
    if reuse is not None:
        stride = max(1, max(len(r) for r in reuse))
        a = np.zeros((B, stride), dtype=np.int32)
        for b, r in enumerate(reuse):
            a[b, :len(r)] = r
        ro = torch.tensor(a, device=dev)
        rc = torch.tensor([len(r) for r in reuse], dtype=torch.int32, device=dev)
        if layer_count is not None:
            lc = torch.tensor(np.asarray(layer_count, dtype=np.int32), device=dev)
    V.vlac_embed_patches(gm.ctx, torch.tensor(frames, device=dev), B, H, W, patch,
                         torch.tensor(w_proj, device=dev).to(torch.bfloat16), ro, rc, stride, lc, out, L)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("H,W,patch", [(112, 112, 14), (224, 224, 14), (448, 224, 14), (60, 90, 6)])
def test_embed_matches_oracle(H, W, patch):
    cfg = synth.CONFIGS["tiny"]
    gm = GpuModel(cfg, seed=0, max_batch=3, max_seq=640)
    try:
        rng = np.random.default_rng(H + W)
        B, L_v = 3, (H // patch) * (W // patch)
        frames = rng.integers(0, 256, size=(B, H, W, 3), dtype=np.uint8)
        w = synth.round_bf16(synth.projection_matrix(cfg.d_model, patch, 9))
        reuse = [sorted(rng.choice(L_v, size=n, replace=False).tolist()) for n in (0, L_v // 3, L_v)]
        rng.shuffle(reuse[1])
        got = run_embed(gm, frames, patch, w, reuse, L=L_v + 5)
        for b in range(B):
            want = O.embed_patches(frames[b], patch, w, reuse[b])
            keep = ~np.isnan(want[:, 0])
            assert keep.sum() == L_v - len(reuse[b])
            assert not keep.any() or np.abs(got[b, :L_v][keep] - want[keep]).max() <= 1e-5
            assert np.all(got[b, :L_v][~keep] == -123.0)       # skipped rows are not written
            assert np.all(got[b, L_v:] == -123.0)
        # layer counts: only the first layer_count[b][0] entries of the list are skipped
        lc = [[0] * cfg.n_layers, [5] * cfg.n_layers, [L_v] * cfg.n_layers]
        got = run_embed(gm, frames, patch, w, reuse, lc)
        for b in range(B):
            want = O.embed_patches(frames[b], patch, w, reuse[b][:lc[b][0]])
            keep = ~np.isnan(want[:, 0])
            assert not keep.any() or np.abs(got[b][keep] - want[keep]).max() <= 1e-5
            assert np.all(got[b][~keep] == -123.0)
        # no lists: every patch
        got = run_embed(gm, frames, patch, w)
        for b in range(B):
            assert np.abs(got[b] - O.embed_patches(frames[b], patch, w)).max() <= 1e-5
    finally:
        gm.close()


@pytest.mark.parametrize("B,H,W,patch,skew", [
    (1, 13 * 5, 13 * 7, 13, 0),     # odd rows of pixels, 35 patches: one past a row tile
    (2, 26 * 2, 26 * 16, 26, 0),    # the largest patch: 127 k-tiles, exactly one row tile
    (1, 14, 14 * 33, 14, 1),        # buffers that allow no wide loads and stores
    (4, 256, 256, 4, 0),            # 256 groups of 64 patches: the wide form
    (4, 256, 256, 4, 1),
    (8, 3 * 40, 3 * 50, 3, 0),      # odd patches, the wide form with a ragged last group, 2 k-tiles
    (18, 14 * 30, 14 * 31, 14, 0),  # the wide form at its largest patch: 37 k-tiles, the last one padded,
    (18, 14 * 30, 14 * 31, 14, 1),  # 15 groups per stream, the last of 34 patches or less
    (7, 15 * 30, 15 * 40, 15, 0),   # larger patches: never the wide form
])
def test_embed_at_the_edges_of_its_tiles(B, H, W, patch, skew):
    """Every product is exact, so what is left is the rounding of an fp32 sum of 3 patch^2 terms
    of magnitude |w| <= 5 std: n 2^-24 sqrt(n) std-sized terms stay below 1e-5 here."""
    import torch
    cfg = synth.CONFIGS["tiny"]
    gm = GpuModel(cfg, seed=0, max_batch=B, max_seq=32)
    try:
        V, dev = gm.V, gm.device
        rng = np.random.default_rng(B + H + W + patch)
        L_v, dp, d = (H // patch) * (W // patch), 3 * patch * patch, cfg.d_model
        frames = rng.integers(0, 256, size=(B, H, W, 3), dtype=np.uint8)
        w = synth.round_bf16(synth.projection_matrix(d, patch, 9))
        reuse = [rng.choice(L_v, size=min(b, L_v), replace=False).tolist() for b in range(B)]
        order = torch.zeros((B, max(1, B)), dtype=torch.int32, device=dev)
        for b, r in enumerate(reuse):
            order[b, :len(r)] = torch.tensor(r, dtype=torch.int32)
        count = torch.tensor([len(r) for r in reuse], dtype=torch.int32, device=dev)
        wbuf = torch.zeros(dp * d + 8, dtype=torch.bfloat16, device=dev)[skew:skew + dp * d].view(dp, d)
        wbuf.copy_(torch.tensor(w))
        fbuf = torch.zeros(frames.size + 8, dtype=torch.uint8, device=dev)[skew:skew + frames.size].view(frames.shape)
        fbuf.copy_(torch.tensor(frames))
        out = torch.full((B * L_v * d + 8,), -7.0, device=dev)[skew:skew + B * L_v * d].view(B, L_v, d)
        V.vlac_embed_patches(gm.ctx, fbuf, B, H, W, patch, wbuf, order, count, order.shape[1], None, out, L_v)
        got = out.cpu().numpy()
        for b in range(B):
            want = O.embed_patches(frames[b], patch, w, reuse[b])
            keep = ~np.isnan(want[:, 0])
            assert np.abs(got[b][keep] - want[keep]).max() <= 1e-5
            assert np.all(got[b][~keep] == -7.0)
    finally:
        gm.close()


@pytest.mark.parametrize("B,H,W,patch", [
    (1, 14 * 3, 14 * 4, 14),       # 588 values: the last tile of 16 is padded
    (18, 14 * 30, 14 * 31, 14),    # the wide form
    (1, 13 * 3, 13 * 4, 13),
])
def test_large_and_infinite_weights(B, H, W, patch):
    """What is finite stays finite (weights near the top of the type, whose sums are not), and an
    infinite weight in the last row of w_proj gives infinities of the pixel's sign, not NaN."""
    cfg = synth.CONFIGS["tiny"]
    gm = GpuModel(cfg, seed=0, max_batch=B, max_seq=32)
    try:
        rng = np.random.default_rng(patch)
        frames = rng.integers(0, 256, size=(B, H, W, 3), dtype=np.uint8)
        w = synth.round_bf16(synth.projection_matrix(cfg.d_model, patch, 9))
        w[:, 1] = np.ldexp(w[:, 1], 125)                       # embeddings of up to about 1e38
        w[-1, 2] = np.inf
        w[0, 3] = -np.inf
        got = run_embed(gm, frames, patch, w)
        for b in (0, B - 1):
            want = O.embed_patches(frames[b], patch, w)
            big = 2.0 ** 125
            assert np.abs(want[:, 1]).max() < 3e38 and np.abs(got[b][:, 1] / big - want[:, 1] / big).max() <= 1e-5
            np.testing.assert_array_equal(got[b][:, 2:4], want[:, 2:4])
            rest = [0] + list(range(4, cfg.d_model))
            assert np.abs(got[b][:, rest] - want[:, rest]).max() <= 1e-5
    finally:
        gm.close()


def test_embed_feeds_the_sparse_prefill():
    """Two steps at the tiny configuration: frame -> Alg. 1 -> embeddings of the recomputed
    patches only -> sparse prefill, all on the GPU, against the oracle's chain."""
    import torch
    cfg = synth.CONFIGS["tiny"]
    H, p, n_txt, k = 112, 14, 16, 32
    L_v = (H // p) ** 2
    prev, cur, _ = synth.frame_pair(H, H, p, 16, seed=2)
    w = synth.round_bf16(synth.projection_matrix(cfg.d_model, p, 3))
    txt = synth.round_bf16(synth.text_embeddings(n_txt, cfg.d_model, 4))
    om = oracle_model(cfg, seed=1)
    gm = GpuModel(cfg, seed=1, max_batch=1, max_seq=128)
    try:
        cache = O.new_cache(cfg, 128)
        e0 = np.concatenate([O.embed_patches(prev, p, w), txt])
        want0 = O.dense_forward(om, e0, L_v, cache)
        g0 = np.concatenate([run_embed(gm, prev[None], p, w)[0], txt])
        got0 = gm.prefill(g0[None], L_v)
        assert np.abs(got0["logits"][0] - want0["logits"]).max() <= 2e-2
        reuse = O.select_static(prev, cur, p, 249, 250, k)
        sel = gm.select(prev[None], cur[None], p, 249, 250, k)
        assert sel["idx"][0] == reuse
        e1 = O.embed_patches(cur, p, w, reuse)
        g1 = run_embed(gm, cur[None], p, w, [sel["order"][0]], fill=float("nan"))[0]
        assert np.array_equal(np.isnan(g1[:, 0]), np.isnan(e1[:, 0]))
        want1 = O.sparse_forward(om, np.concatenate([np.nan_to_num(e1), txt]), L_v, cache, [reuse] * cfg.n_layers)
        got1 = gm.prefill(np.concatenate([g1, txt])[None], L_v, [sel["order"][0]])   # NaN rows are never read
        alive = ~np.isnan(want1["hidden"][:, 0])
        assert np.abs(got1["hidden"][0][alive] - want1["hidden"][alive]).max() <= 2e-2
        assert np.abs(got1["logits"][0] - want1["logits"]).max() <= 2e-2
        assert np.isfinite(got1["logits"]).all()
    finally:
        gm.close()


@pytest.mark.parametrize("B,H,W,patch,skew", [
    (12, 16 * 32, 16 * 32, 16, 0),  # 768 workgroups of 128 features and 32 patches: the last that list for themselves
    (13, 16 * 32, 16 * 32, 16, 0),  # one stream more: the list of the launch before
    (13, 16 * 32, 16 * 32, 16, 1),
    (97, 13 * 11, 13 * 11, 13, 0),  # the same with odd patches, a last group of 25 and less
    (8, 26 * 32, 26 * 32, 26, 0),   # one workgroup per CU: 512 of them
    (9, 26 * 32, 26 * 32, 26, 0),
])
def test_who_lists_the_live_patches(B, H, W, patch, skew):
    """Reuse lists of every length, shuffled and clamped by the layer count, on both sides of the limit; the sums are exact
    but for the fp32 rounding of 3 patch^2 terms (as above)."""
    import torch
    cfg = synth.CONFIGS["tiny"]
    gm = GpuModel(cfg, seed=0, max_batch=B, max_seq=32)
    try:
        V, dev = gm.V, gm.device
        rng = np.random.default_rng(B)
        L_v, d = (H // patch) * (W // patch), cfg.d_model
        frames = rng.integers(0, 256, size=(B, H, W, 3), dtype=np.uint8)
        w = synth.round_bf16(synth.projection_matrix(d, patch, 9))
        n = [L_v * b // (B - 1) for b in range(B)]
        order = np.stack([rng.permutation(L_v) for _ in range(B)]).astype(np.int32)
        lc = np.full((B, cfg.n_layers), L_v, np.int32)
        lc[1::3, 0] = 7
        fbuf = torch.zeros(frames.size + 8, dtype=torch.uint8, device=dev)[skew:skew + frames.size].view(frames.shape)
        fbuf.copy_(torch.tensor(frames))
        out = torch.full((B, L_v, d), -7.0, device=dev)
        V.vlac_embed_patches(gm.ctx, fbuf, B, H, W, patch, torch.tensor(w, device=dev).to(torch.bfloat16),
                             torch.tensor(order, device=dev), torch.tensor(n, dtype=torch.int32, device=dev), L_v,
                             torch.tensor(lc, device=dev), out, L_v)
        got = out.cpu().numpy()
        for b in range(B):
            m = min(n[b], lc[b, 0])
            keep = np.ones(L_v, bool)
            keep[order[b, :m]] = False
            assert np.array_equal(got[b, :, 0] != -7.0, keep), b
            if b % 4 == 0 or b == B - 1:
                want = O.embed_patches(frames[b], patch, w, order[b, :m].tolist())
                assert not keep.any() or np.abs(got[b][keep] - want[keep]).max() <= 1e-5
    finally:
        gm.close()

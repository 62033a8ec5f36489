"""One block at the edges of its kernels' tiles, splits and softmax range,
through the block call, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from _cases import download_slot, gemm_plan, relerr, upload_slot

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2608_29809_amd.runtime import ActiveSet, RegionCacheModel


def _block(gh, gw, counts, seed, edit=None, chains=None):
    """A bf16 reuse block of len(counts) chains over gh x gw tokens, `chains`
    of them (all by default) compared with the oracle: H of the active rows,
    K and V of the slot."""
    s = synth.ModelShape(layers=1, text_dim=1152, grid_h=gh, grid_w=gw, dtype="bf16", token_mode=True)
    W = synth.make_weights(s, seed=seed, stress=True)
    if edit:
        edit(W["layers"][0])
    B, N, C = len(counts), s.tokens, s.hidden
    rng = np.random.default_rng(seed)
    idx = [np.sort(rng.choice(N, size=n, replace=False)).astype(np.int32) for n in counts]
    slot = synth.make_cache_slot(s, B, seed)
    if edit:  # cached keys like the block's own
        slot["K"] = synth.bf16_round(slot["K"] * 0.1 + W["layers"][0]["qkv_b"][C:2 * C].reshape(1, 1, 16, 1, 72))
    x = synth.bf16_round(rng.standard_normal((B, N, C)).astype(np.float32))
    t_vec = rng.standard_normal(C).astype(np.float32)
    text = synth.make_text(s, B, seed)
    model = RegionCacheModel(s, W)
    cache = model.alloc_cache(B, 1)
    upload_slot(model, cache, 0, slot)
    tkv = model.prepare_text(model.to_storage(text))
    model.reuse_step(cache, 0, ActiveSet.from_lists(idx), model.to_storage(x), 0, -1, tkv,
                     t_vec=torch.from_numpy(t_vec).cuda())
    torch.cuda.synchronize()
    got = download_slot(cache, 0, 1, B)
    for b in range(B) if chains is None else chains:
        if not counts[b]:
            continue
        X, K, V, H, _ = O.reuse_block_tokens(s, W, x[b], idx[b], t_vec, text[b], slot["K"][0, b], slot["V"][0, b],
                                             slot["H"][0, b])
        # bf16 operands and storage (the tolerance of the block tests)
        assert relerr(got["H"][0, b][idx[b]], np.asarray(H)[idx[b]]) < 2e-2, (b, counts[b])
        assert relerr(got["K"][0, b], K) < 2e-2 and relerr(got["V"][0, b], V) < 2e-2, (b, counts[b])


@pytest.mark.parametrize("gh,gw,counts", [(8, 8, [1]), (8, 8, [64]), (8, 16, [33, 0, 128]), (8, 24, [32, 31, 65]),
                                          (16, 20, [129, 127]), (32, 32, [257, 255, 256])])
def test_edges(gh, gw, counts):
    """One to sixteen key tiles, query counts around the 32-query halves and
    the 128-query tiles, an empty chain."""
    print("self-attention", gh, gw, counts, flush=True)
    _block(gh, gw, counts, seed=gh + gw)


@pytest.mark.parametrize("counts", [[0, 0, 5], [7, 0, 0], [0] * 9 + [1, 0, 64, 0, 2] + [0] * 7, [1] * 16 + [3],
                                    [(5 * b) % 9 for b in range(70)]])
def test_many_chains(counts):
    """Rows found in their chains: empty chains first, last and in between,
    more chains than the kernel arguments hold offsets of (16)."""
    print("chains", counts, flush=True)
    _block(8, 8, counts, seed=len(counts))


@pytest.mark.parametrize("rows", [1009, 2449, 3969])
def test_large_gemm_tiles(rows):
    """Row counts that take large GEMM tiles, each with a last row tile that is
    not full: the MLP at 1009 rows (128x144 tiles, its MLP-down split in four),
    QKV in 256x144 and MLP-down in 128x144 tiles at 2449, every GEMM at 3969
    (QKV and MLP-up in 256x288 tiles, the last with 129 rows, the others in
    128x144, the last with one)."""
    print("large tiles", rows, flush=True)
    _block(64, 64, [rows], seed=rows)


# large tile (rows, columns) of QKV, both out-projections, the cross query,
# MLP-up and MLP-down, None for the small ones
@pytest.mark.parametrize("rows,tiles", [
    (2045, (None, None, None, (256, 144), (128, 144))), (6001, (None, (256, 144), (256, 144), (256, 144), (256, 144))),
    (11003, (None, (128, 144), (256, 288), (128, 288), (128, 144))),
    (16381, ((256, 288), (256, 288), (256, 288), (128, 288), (256, 288)))])
def test_large_gemm_tiles_of_many_rows(rows, tiles):
    """The other large tiles, each with a last row tile that is not full: many
    chains of 64 tokens (the GEMMs see rows only), of which those at the tile
    borders, the first and the last are compared."""
    shapes = ((3456, 1152, "qkv"), (1152, 1152, "resid"), (1152, 1152, "store"), (4608, 1152, "gelu"), (1152, 4608, "resid"))
    for (N, K, epi), tile in zip(shapes, tiles):
        p = gemm_plan(rows, N, K, epi)
        assert (p[1:3] if p[0] else None) == tile, (N, K, epi, p)
    print("large tiles of many rows", rows, flush=True)
    counts = [64] * (rows // 64) + [rows % 64]
    n = len(counts)
    _block(8, 8, counts, seed=rows, chains=sorted({0, 1, 2, 3, 4, n // 2, n - 5, n - 3, n - 2, n - 1}))


def test_vectors_aligned_to_4_bytes():
    """Biases and modulation tables that begin 4 bytes past a 16-byte boundary
    (views into a packed buffer, which rc_create takes), at a row count whose
    GEMMs take large tiles with aligned ones: the result is the oracle's."""
    import ctypes

    from paper_2608_29809_amd import abi
    print("vectors aligned to 4 bytes", flush=True)
    s = synth.ModelShape(layers=1, text_dim=1152, grid_h=64, grid_w=64, dtype="bf16", token_mode=True)
    W = synth.make_weights(s, seed=6, stress=True)
    rng = np.random.default_rng(6)
    idx = np.sort(rng.choice(s.tokens, 1009, replace=False)).astype(np.int32)
    assert gemm_plan(1009, 4608, 1152, "gelu")[0]
    slot = synth.make_cache_slot(s, 1, 6)
    x = synth.bf16_round(rng.standard_normal((1, s.tokens, s.hidden)).astype(np.float32))
    t_vec = rng.standard_normal(s.hidden).astype(np.float32)
    text = synth.make_text(s, 1, 6)
    model = RegionCacheModel(s, W)
    keep = []
    for f in abi.LAYER_FIELDS:
        if not f.endswith("_w"):
            v = torch.from_numpy(np.ascontiguousarray(W["layers"][0][f]).reshape(-1))
            keep.append(torch.zeros(v.numel() + 1, device="cuda"))
            keep[-1][1:] = v
            setattr(model._layers[0], f, keep[-1].data_ptr() + 4)
    abi.rc_destroy(model.ctx)
    ctx = ctypes.c_void_p()
    abi.rc_create(ctypes.byref(model._cfg), ctypes.byref(model._w), ctypes.byref(ctx))
    model.ctx = ctx
    cache = model.alloc_cache(1, 1)
    upload_slot(model, cache, 0, slot)
    model.reuse_step(cache, 0, ActiveSet.from_lists([idx]), model.to_storage(x), 0, -1,
                     model.prepare_text(model.to_storage(text)), t_vec=torch.from_numpy(t_vec).cuda())
    torch.cuda.synchronize()
    got = download_slot(cache, 0, 1, 1)
    X, K, V, H, _ = O.reuse_block_tokens(s, W, x[0], idx, t_vec, text[0], slot["K"][0, 0], slot["V"][0, 0], slot["H"][0, 0])
    assert relerr(got["H"][0, 0][idx], np.asarray(H)[idx]) < 2e-2
    assert relerr(got["K"][0, 0], K) < 2e-2 and relerr(got["V"][0, 0], V) < 2e-2


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_softmax_range(sign):
    """All logits of every query near +-136 (+-196 in base 2), outside the range
    of the fixed reference: the workgroups start again relative to their
    maxima.  Queries and keys are 4 and +-4 plus a tenth of their usual
    variation; rounding them to bf16 (half a unit of 2^-6) moves a logit by
    about 4 * 0.0045 * sqrt(2 * 72) / sqrt(72) = 0.025, and the attention by a
    few per cent of a mean of hundreds of values, well under 2e-2 of H."""

    def edit(lw):
        C = 1152
        lw["qkv_w"][:2 * C] *= 0.1
        lw["qkv_w"][:] = synth.bf16_round(lw["qkv_w"])
        lw["qkv_b"][:C] = 4.0
        lw["qkv_b"][C:2 * C] = 4.0 * sign

    print("softmax range", sign, flush=True)
    _block(16, 16, [200, 3], seed=5, edit=edit)


@pytest.mark.parametrize("text_len,valid", [(120, [120, 1, 57]), (64, [64, 33, 5]), (40, None)])
def test_cross_attention_of_many_rows(text_len, valid):
    """The cross-attention that takes projected queries (more than 256 tiles
    of 64 rows and a head): chains of different length with padded prompts,
    one or two text tiles, the maps of the first, last and padded columns."""
    print("cross-attention", text_len, valid, flush=True)
    s = synth.ModelShape(layers=1, text_dim=1152, text_len=text_len, grid_h=64, grid_w=32, dtype="bf16", token_mode=True)
    W = synth.make_weights(s, seed=7, stress=True)
    rng = np.random.default_rng(7)
    counts = [1281, 1, 999]
    idx = [np.sort(rng.choice(s.tokens, size=n, replace=False)).astype(np.int32) for n in counts]
    slot = synth.make_cache_slot(s, 3, 7)
    x = synth.bf16_round(rng.standard_normal((3, s.tokens, s.hidden)).astype(np.float32))
    t_vec = rng.standard_normal(s.hidden).astype(np.float32)
    text = synth.make_text(s, 3, 7)
    delta = [0, 3, 4, 17, 31, 38, text_len - 1]
    model = RegionCacheModel(s, W)
    cache = model.alloc_cache(3, 1)
    upload_slot(model, cache, 0, slot)
    maps = torch.zeros((3, s.tokens, len(delta)), device="cuda")
    model.reuse_step(cache, 0, ActiveSet.from_lists(idx), model.to_storage(x), 0, -1,
                     model.prepare_text(model.to_storage(text)), delta, maps, t_vec=torch.from_numpy(t_vec).cuda(),
                     text_valid=None if valid is None else torch.tensor(valid, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    got = download_slot(cache, 0, 1, 3)
    for b, n in enumerate(counts):
        nv = text_len if valid is None else valid[b]
        cols = [j for j in delta if j < nv]
        X, K, V, H, m = O.reuse_block_tokens(s, W, x[b], idx[b], t_vec, text[b, :nv], slot["K"][0, b], slot["V"][0, b],
                                             slot["H"][0, b], cols)
        assert relerr(got["H"][0, b][idx[b]], np.asarray(H)[idx[b]]) < 2e-2, b
        g = maps[b].cpu().numpy()[idx[b]]
        m = np.asarray(m)
        m = m[idx[b]] if m.shape[0] == s.tokens else m
        assert relerr(g[:, [delta.index(j) for j in cols]], m) < 2e-2, b
        assert not g[:, [i for i, j in enumerate(delta) if j >= nv]].any()  # padded tokens have probability 0


@pytest.mark.parametrize("layers,batch", [(33, 1), (2, 3)])
def test_text_of_all_blocks(layers, batch):
    """The text keys and values that one launch writes for up to 32 blocks:
    every block's own weights at its own place, a second launch past 32, rows
    past a tile, zero padding."""
    print("text", layers, batch, flush=True)
    s = synth.ModelShape(layers=1, mlp=128, text_dim=1152, grid_h=8, grid_w=8, dtype="bf16", token_mode=True)
    W = synth.make_weights(s, seed=3)
    lw = W["layers"][0]
    W["layers"] = [dict(lw, xkv_w=synth.bf16_round(lw["xkv_w"] * (1 + l / 64)), xkv_b=lw["xkv_b"] + l) for l in range(layers)]
    s = synth.ModelShape(layers=layers, mlp=128, text_dim=1152, grid_h=8, grid_w=8, dtype="bf16", token_mode=True)
    text = synth.make_text(s, batch, 4)
    model = RegionCacheModel(s, W)
    kv = model.prepare_text(model.to_storage(text)).view(torch.bfloat16).float().cpu().numpy()
    kv = kv.reshape(layers, batch, 2, 16, 128 * 72)
    for l in range(layers):
        for b in range(batch):
            k, v = (a.transpose(1, 0, 2) for a in O.text_kv(W["layers"][l], text[b], 16))  # [heads, tokens, 72]
            gk, gv = kv[l, b, 0].reshape(16, 128, 72), kv[l, b, 1].reshape(16, 72, 128).transpose(0, 2, 1)
            # one bf16 rounding of an fp32 sum of bf16 products
            assert relerr(gk[:, :120], k) < 2.0 ** -8 and relerr(gv[:, :120], v) < 2.0 ** -8, (l, b)
            assert not gk[:, 120:].any() and not gv[:, 120:].any()

"""Localisation and compaction at the edges of their kernels, against the
oracle: grids that are not multiples of a workgroup or of a word, one to eight
columns, radii, several chains, constant maps and infinities."""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2608_29809_amd.runtime import RegionCacheModel, compact_mask

_MODELS = {}


def _model(gh, gw):
    if (gh, gw) not in _MODELS:
        s = synth.ModelShape(layers=1, mlp=128, text_dim=1152, grid_h=gh, grid_w=gw, dtype="bf16", token_mode=True)
        _MODELS[gh, gw] = RegionCacheModel(s, synth.make_weights(s, seed=0))
    return _MODELS[gh, gw]


@pytest.mark.parametrize("gh,gw,batch,nd,radius", [(8, 8, 1, 1, 1), (8, 24, 1, 8, 2), (64, 33, 1, 3, 4), (33, 64, 3, 5, 0),
                                                   (64, 64, 1, 6, 1), (65, 64, 1, 6, 1), (128, 128, 2, 7, 3),
                                                   (8, 8, 300, 2, 1), (16, 12, 90, 4, 1), (64, 48, 7, 1, 2), (32, 32, 17, 8, 1)])
def test_localize_edges(gh, gw, batch, nd, radius):
    print("localize", gh, gw, batch, nd, radius, flush=True)
    rng = np.random.default_rng(gh * gw + nd)
    N = gh * gw
    maps = rng.uniform(0.0, 1.0, (batch, N, nd)).astype(np.float32) ** 4
    maps[:, :, 0] = 0.25  # constant: selects nothing
    if nd > 2:
        maps[0, 5, 1] = np.inf  # the range is infinite: every score is 0 or not a number
    act_thr = 0.9
    mask, act = _model(gh, gw).localize(torch.from_numpy(maps).cuda(), nd, act_thr, radius)
    mask = mask.cpu().numpy()
    base = 0
    for b in range(batch):
        sel = np.zeros(N, bool)
        for j in range(nd):  # the rule in the library's float32 arithmetic
            lo, hi = maps[b, :, j].min(), maps[b, :, j].max()
            if hi > lo:
                with np.errstate(invalid="ignore", over="ignore"):
                    sel |= (maps[b, :, j] - lo) * (np.float32(1.0) / (hi - lo)) >= np.float32(act_thr)
        ref = O.dilate(sel.reshape(gh, gw), radius).reshape(-1).astype(np.uint8)
        assert np.array_equal(mask[b], ref), b
        n = int(ref.sum())
        assert act.host[b + 1] - act.host[b] == n
        assert np.array_equal(act.idx[base:base + n].cpu().numpy(), np.flatnonzero(ref)), b
        base += n
    assert act.offsets.cpu().tolist() == list(act.host)


@pytest.mark.parametrize("batch,tokens", [(1, 1), (2, 63), (3, 1025), (1, 16384), (2, 16385), (1, 65535),
                                          (40, 1), (700, 3), (300, 64), (20, 1000), (257, 64), (64, 1024), (5, 16384),
                                          (3, 65535)])
def test_compact_edges(batch, tokens):
    print("compact", batch, tokens, flush=True)
    masks = (np.random.default_rng(tokens).random((batch, tokens)) < 0.4).astype(np.uint8) * 3
    masks[-1, -1] = 1
    act = compact_mask(torch.from_numpy(masks).cuda())
    idx, off = O.compact((masks != 0).astype(np.uint8))
    assert list(act.host) == off.tolist()
    assert np.array_equal(act.idx[:off[-1]].cpu().numpy(), idx)

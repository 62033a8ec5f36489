"""Infinities that an operand of a step holds reach only the results that
depend on them."""
import numpy as np
import pytest
import torch

import synth
from _cases import run_block

pytestmark = pytest.mark.gpu

C = 1152


def _block(dtype, gh, gw, idx, edit=None, text_kv=None):
    s = synth.ModelShape(layers=1, text_dim=C, grid_h=gh, grid_w=gw, dtype=dtype, token_mode=True)
    W = synth.make_weights(s, seed=8, stress=True)
    if edit:
        edit(W["layers"][0])
    rng = np.random.default_rng(8)
    x = synth.bf16_round(rng.standard_normal((len(idx), s.tokens, C)).astype(np.float32))
    return run_block(s, W, idx, synth.make_cache_slot(s, len(idx), 8), x, rng.standard_normal(C).astype(np.float32),
                     synth.make_text(s, len(idx), 8), text_kv)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinite_bias(dtype):
    """A column of the MLP-down whose bias is infinite is infinite (its gate is
    near 1), and the others are what they are without it."""
    print("infinite bias", dtype, flush=True)
    idx = [np.arange(0, 64, 3, dtype=np.int32)]
    ref = _block(dtype, 8, 8, idx)["H"][0, 0][idx[0]]

    def edit(lw):
        lw["fc2_b"][7], lw["fc2_b"][640] = np.inf, -np.inf

    got = _block(dtype, 8, 8, idx, edit)["H"][0, 0][idx[0]]
    assert (got[:, 7] == np.inf).all() and (got[:, 640] == -np.inf).all()
    rest = np.setdiff1d(np.arange(C), [7, 640])
    assert np.array_equal(got[:, rest], ref[:, rest])


@pytest.mark.parametrize("rows", [100, 2000])
@pytest.mark.parametrize("dim", [3, 70])
def test_infinite_text_key(rows, dim):
    """A text key of minus infinity in one dimension, where every query is
    positive, has probability 0: the same result as with a key of -1e30.
    Both forms of the cross-attention, a dimension of its first and of its
    last operand."""
    print("infinite text key", rows, dim, flush=True)
    idx = [np.sort(np.random.default_rng(1).choice(2048, rows, replace=False)).astype(np.int32)]

    def edit(lw):  # queries of 50 plus their usual few units in that dimension of every head
        lw["xq_b"][dim::72] = 50.0

    out = []
    for value in (-1e30, -float("inf")):
        def text_kv(kv):  # keys [layer, chain][head][128][72], then the values
            kv.view(2, 16, 128, 72)[0, :, 5, dim] = value
        out.append(_block("bf16", 32, 64, idx, edit, text_kv)["H"][0, 0][idx[0]])
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1])

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

"""The bf16 self-attention outside the range of its fixed softmax reference:
restarts relative to the queries' maxima, in every form of the kernel and
mixed over the key splits, and values far from 1."""
import numpy as np
import pytest

import oracle as O
import synth
from _cases import attention_plan, relerr, run_block

pytestmark = pytest.mark.gpu

C = 1152


def _case(gh, gw, idx, first, logits, value=1.0, tiny=False):
    """One block whose cached tokens have logits near logits[0] (tokens below
    `first`) and logits[1] (the others and the active ones) in base 2, and
    values of +-2 `value` in opposite signs for the two.  Queries and the
    active tokens' keys are 4 and k plus a tenth of their usual variation; a
    logit is 72 * 4 k / sqrt(72), 48.97 k in base 2, plus or minus about 1."""
    s = synth.ModelShape(layers=1, text_dim=C, grid_h=gh, grid_w=gw, dtype="bf16", token_mode=True)
    N, B = s.tokens, len(idx)
    rng = np.random.default_rng(N + B)
    W = synth.make_weights(s, seed=N, stress=True)
    lw = W["layers"][0]
    lw["qkv_w"][:2 * C] = synth.bf16_round(lw["qkv_w"][:2 * C] * np.float32(0.1))
    lw["qkv_b"][:C] = 4.0
    lw["qkv_b"][C:2 * C] = logits[1] / 48.97
    early = (np.arange(N) < first)[:, None]
    slot = synth.make_cache_slot(s, B, N)
    slot["K"] = synth.bf16_round(slot["K"] * np.float32(0.02) + np.where(early, *logits).astype(np.float32) / np.float32(48.97))
    sign = rng.choice([-2.0, 2.0], (16, 1, 72))
    slot["V"] = synth.bf16_round(((slot["V"] * 0.3 + np.where(early, sign, -sign)) * value).astype(np.float32))
    x = synth.bf16_round(rng.standard_normal((B, N, C)).astype(np.float32))
    if value > 1:  # (cross-attention scores of such rows would leave fp32's precision)
        lw["xq_w"][:] = 0.0
    if tiny:  # the attention of the cached values is all that reaches the output
        x[:] = 0.0
        for k in ("xproj_w", "xproj_b", "fc2_w", "fc2_b", "proj_b"):
            lw[k][:] = 0.0
        lw["qkv_w"][2 * C:] = 0.0
        lw["qkv_b"][2 * C:] = 0.0
    t_vec = rng.standard_normal(C).astype(np.float32)
    text = synth.make_text(s, B, N)
    got = run_block(s, W, idx, slot, x, t_vec, text)
    for b in range(B):
        _, K, V, H, _ = O.reuse_block_tokens(s, W, x[b], idx[b], t_vec, text[b], slot["K"][0, b], slot["V"][0, b],
                                             slot["H"][0, b])
        # bf16 operands and storage; rounding queries and keys to bf16 moves a logit by about 0.025
        assert relerr(got["K"][0, b], K) < 2e-2 and relerr(got["V"][0, b], V) < 2e-2, b
        g = got["H"][0, b][idx[b]]
        assert np.isfinite(g).all(), b
        assert relerr(g, np.asarray(H)[idx[b]]) < 2e-2, b


@pytest.mark.parametrize("gh,gw,counts,plan,first", [(64, 64, [723], (1, 5), 768), (32, 64, [1088] * 2, (2, 3), 640),
                                                     (32, 32, [704] * 6, (2, 1), 320)])
@pytest.mark.parametrize("logits", [(196.0, 196.0), (-196.0, -196.0), (196.0, 0.0), (-196.0, 0.0), (72.0, 67.5), (-60.0, -36.0)])
def test_restart(gh, gw, counts, plan, first, logits):
    """Logits outside the range of the fixed reference for all tokens, for the
    first key split only (the whole of it, so that it restarts and the others
    don't), and on the two sides of the range with like weights, one or two
    32-query halves per wave."""
    assert attention_plan(counts, gh * gw) == plan
    print("restart", counts, plan, logits, flush=True)
    rng = np.random.default_rng(counts[0])
    idx = [np.sort(first + rng.choice(gh * gw - first, size=n, replace=False)).astype(np.int32) for n in counts]
    _case(gh, gw, idx, first, logits)


@pytest.mark.parametrize("logit,value", [(67.5, 2.0 ** 52), (67.5, 2.0 ** 58), (-82.0, 2.0 ** -72)])
def test_values_far_from_one(logit, value):
    """Denominators near both ends of the range with values whose products
    leave that of fp32: 128 keys per split at 2^67.5 give 2^74.5 times the
    values, at 2^-82 2^-75."""
    assert attention_plan([40], 1024) == (1, 8)
    print("values", logit, value, flush=True)
    _case(32, 32, [np.arange(40, dtype=np.int32) * 7], 0, (logit, logit), value, tiny=value < 1)

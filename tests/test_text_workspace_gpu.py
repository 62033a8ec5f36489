"""rc_prepare_text with the workspace its stages hold at least."""
import ctypes as C

import pytest
import torch

import synth
from _cases import relerr, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 5])
def test_text_preparation_in_little_workspace(batch):
    """Room for the two hidden-wide activations only (a workspace sized for
    another call may have no more): the first product is then not split over
    K.  Nothing is written past the workspace, and the result is that of a
    split one but for the order of its sums."""
    from paper_2608_29809_amd import abi
    from paper_2608_29809_amd.runtime import RegionCacheModel
    print("text workspace", batch, flush=True)
    s = synth.ModelShape(layers=2, mlp=128, grid_h=8, grid_w=8, dtype="bf16")
    model = RegionCacheModel(s, synth.make_weights(s, seed=3))
    txt = model.to_storage(synth.make_text(s, batch, 3))
    ref = model.prepare_text(txt)
    need = 2 * ((batch * s.text_len * s.hidden * 2 + 255) // 256 * 256)
    assert need < abi.rc_workspace_bytes(model.ctx, 1, batch)
    ws = torch.full((need + 4096,), 77, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(ref)
    p = lambda t: C.c_void_p(t.data_ptr())
    abi.rc_prepare_text(model.ctx, p(txt), batch, p(out), p(ws), need, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert bool((ws[need:] == 77).all())
    # three products with bf16 results: a changed fp32 sum may round an activation the other way (2^-8)
    assert relerr(to_np(out.view(torch.bfloat16)), to_np(ref.view(torch.bfloat16))) < 2.0 ** -7
    with pytest.raises(abi.RcError, match="RC_ERR_CAPACITY"):
        abi.rc_prepare_text(model.ctx, p(txt), batch, p(out), p(ws), need - 1, None)

"""The surrogate's first two layers, computed in one pass down 64-pixel
columns, at the edges of its patches and runs: fields of fewer rows than a
patch or fewer columns than a tile, ragged last patches, the halo columns that
wrap, and more patches than work-groups, so that a run of patches goes on,
ends with a field and begins again in the next."""
import numpy as np
import pytest

from oracle import srg_oracle as S
from tests.gpu_util import rel_l2
from tests.test_gpu_surrogate import S_IN, S_OUT, TOL_G, TOL_Y, _rand_params, _rounded, _srg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W", [(1, 3, 3), (1, 4, 64), (2, 5, 65), (3, 7, 127), (1, 9, 128),
                                   (20, 165, 66)])
def test_first_two_layers_at_patch_edges(B, H, W):
    """Output (through both layers) and the weight gradients of layers 0 and 1
    (the second reads the stored activations of the first), within the bounds
    of the same quantities at other sizes."""
    import torch
    from paper_1908_03876_amd import abi
    print(f"{B}x{H}x{W}", flush=True)
    rng = np.random.default_rng(B * 1000 + H * 10 + W)
    params = _rand_params(rng)
    s = _srg(params, B, H, W)
    x, dy = rng.normal(0, 3.0, (B, H, W)), rng.standard_normal((B, H, W))
    xt, dyt = (torch.tensor(a, dtype=torch.float32, device="cuda") for a in (x, dy))
    y = torch.empty_like(xt)
    abi.mrt_srg_forward(s.handle, xt, y, B, H, W)
    abi.mrt_srg_backward(s.handle, xt, dyt, None, True, B, H, W)
    torch.cuda.synchronize()
    ref_p = _rounded(params)
    y_ref, acts = S.forward(ref_p, x, S_IN, S_OUT, bf16=True)
    _, grads = S.backward(ref_p, acts, dy, S_IN, S_OUT, bf16=True)
    assert rel_l2(y.double().cpu().numpy(), y_ref) <= TOL_Y
    for layer in (0, 1):
        gw = s.get_param(layer, 2).reshape(grads[layer][0].shape)
        assert rel_l2(gw, grads[layer][0]) <= TOL_G, layer
        assert rel_l2(s.get_param(layer, 3), grads[layer][1]) <= TOL_G, layer


@pytest.mark.parametrize("B,H,W", [(800, 3, 5), (257, 12, 63), (52, 62, 19), (1, 4, 49200),
                                   (60, 61, 20), (100, 11, 130)])
def test_first_two_layers_on_many_patches(B, H, W):
    """Both sides of the line between one pass and a pass per layer, where a
    work-group has more than a patch."""
    test_first_two_layers_at_patch_edges(B, H, W)

"""The three expert weight gradients in one launch: both tile sizes, remainders of both, empty experts, accumulation."""
import pytest
import torch

from spes_workloads import custom_config, layer_inputs

from test_gpu_layer import _full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(T=300, d=136, M=8, f=264, k=2, n_trainable=8),                              # 128 x 128 tiles, 8 columns / rows over
    dict(T=300, d=776, M=16, f=520, k=2, n_trainable=16),                            # 576 tiles of 256 x 256
    dict(T=600, d=776, M=4, f=1000, k=4, n_trainable=4),                             # 192 tiles of 256 x 256, 600 rows a head
    dict(T=600, d=776, M=4, f=520, k=4, n_trainable=4),                              # 420 of 128 x 128 (144 full ones)
    dict(T=200, d=128, M=8, f=384, k=1, n_trainable=8, bias="normal", bias_scale=8.0),   # experts without a row
    dict(T=300, d=136, M=8, f=264, k=2, n_trainable=3, dtype="f32"),
    # fp32 results far from square; the transposed sets have fewer tiles and leave the last blocks of the grid idle
    dict(T=70, d=72, M=4, f=24, k=2, n_trainable=3, dtype="f32"),
    dict(T=64, d=1032, M=4, f=8, k=1, n_trainable=4, dtype="f32"),
    dict(T=200, d=8, M=4, f=1504, k=2, n_trainable=4, dtype="f32"),                  # 32-row tiles
    dict(T=130, d=128, M=16, f=3080, k=2, n_trainable=16, dtype="f32"),              # 64-row tiles
])
def test_wgrad_sets(kw, device):
    kw = {"dtype": "bf16", "router_sigma": 0.3, "trainable": "random", **kw}
    L, _, _ = _full_parity(layer_inputs(custom_config(**kw)), device, "wgrad sets")
    once = [t.clone() for t in (L.d_w_gate, L.d_w_up, L.d_w_down)]
    L.fwd(); L.bwd(1); torch.cuda.synchronize()
    for a, b in zip(once, (L.d_w_gate, L.d_w_up, L.d_w_down)):
        assert torch.equal(2 * a, b)                        # x + x is exact

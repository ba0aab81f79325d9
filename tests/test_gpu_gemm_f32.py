"""fp32 expert GEMMs on the matrix cores: both row tiles, remainders of rows, columns and k, experts without a row, any number of experts."""
import pytest
import torch

from spes_workloads import custom_config, layer_inputs

from harness import DeviceLayer
from test_gpu_layer import _full_parity

pytestmark = pytest.mark.gpu

# case, rows per tile (test_plan.py checks it)
CASES = [
    (dict(T=1, d=8, M=3, f=8, k=1, n_trainable=1), 32),                                              # one row, a quarter of a K-tile
    (dict(T=33, d=32, M=1, f=128, k=1, n_trainable=1), 32),                                          # one row beyond a tile, whole K-tiles
    (dict(T=67, d=136, M=7, f=40, k=3, n_trainable=5), 32),                                          # odd number of experts
    (dict(T=130, d=520, M=10, f=264, k=2, n_trainable=10, bias="normal", bias_scale=8.0), 32),       # experts without a row
    (dict(T=300, d=200, M=33, f=328, k=4, n_trainable=9, renorm=1), 32),
    (dict(T=1000, d=1032, M=12, f=1032, k=2, n_trainable=3), 64),                                    # remainders of eight columns
    (dict(T=2048, d=136, M=12, f=72, k=8, n_trainable=5, bias="normal", bias_scale=2.0), 64),        # short contractions, many rows
    (dict(T=600, d=264, M=8, f=1000, k=4, n_trainable=2), 32),                                       # shares of k in two, and in four
]


@pytest.mark.parametrize("kw,rows", CASES)
def test_f32_layer(kw, rows, device):
    kw = {"router_sigma": 0.3, "trainable": "random", **kw}
    _full_parity(layer_inputs(custom_config(**kw)), device, f"fp32, {rows}-row tiles")


@pytest.mark.parametrize("T,d,f", [(60, 136, 200), (700, 40, 328)])
def test_f32_values_stay_with_their_expert(T, d, f, device):
    """NaN weights of one expert: every result of tokens and experts that have nothing to do with it stays bit for bit."""
    L = DeviceLayer(layer_inputs(custom_config(T=T, d=d, M=5, f=f, k=2, n_trainable=5, router_sigma=0.3)), device)
    outs = []
    for poisoned in (False, True):
        if poisoned:
            for w in (L.w_gate, L.w_up, L.w_down):
                w[2] = float("nan")
        L.fwd(); L.bwd(); torch.cuda.synchronize()
        outs.append([t.detach().clone() for t in (L.y, L.dx, L.d_w_gate, L.d_w_up, L.d_w_down)])
    clean = ~(L.idx == 2).any(dim=1).to(outs[0][0].device)
    others = torch.tensor([0, 1, 3, 4], device=device)
    assert clean.any() and not clean.all()
    for i, (a, b) in enumerate(zip(*outs)):
        pick = clean if i < 2 else others
        assert torch.equal(a[pick], b[pick]) and torch.isfinite(b[pick]).all(), i

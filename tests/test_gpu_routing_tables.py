"""Routing tables against the oracle, bit for bit, around the sizes where a block, a vector of pairs or the one launch ends."""
import pytest
import torch

from oracle import spes_oracle as O
from spes_workloads import custom_config, layer_inputs

from harness import DeviceLayer, check_routing, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,M,k,scale", [
    (1, 4, 1, 0.5), (1023, 5, 1, 0.5), (1024, 64, 1, 0.5), (1025, 8, 1, 8.0), (683, 16, 3, 0.5), (2051, 64, 2, 2.0),
    (4096, 16, 8, 0.5), (4096, 9, 8, 30.0), (4097, 16, 8, 0.5),          # 32768 pairs: the last of the one launch; then three
])
def test_tables(T, M, k, scale, device):
    inp = layer_inputs(custom_config(T=T, d=8, M=M, f=8, k=k, n_trainable=1, bias="normal", bias_scale=scale, router_sigma=0.3))
    L = DeviceLayer(inp, device)
    L.fwd(); torch.cuda.synchronize()
    fwd = O.moe_forward(inp["x"], inp["w_router"], inp["router_bias"], inp["w_gate"], inp["w_up"], inp["w_down"], k, 0)
    check_routing(L, fwd)
    assert rel_err(L.host(L.y), fwd["y"]) <= 1e-5

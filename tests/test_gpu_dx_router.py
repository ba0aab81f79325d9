"""The router's part of dx and its weight gradient on the matrix cores, alone: with experts of zero weights nothing else is left of dx."""
import pytest
import torch

from spes_workloads import custom_config, layer_inputs

from harness import DeviceLayer

pytestmark = pytest.mark.gpu

# one token, remainders of 16 tokens and of 64 columns, whole and partial sets of 64 experts, 16 and 64 tokens a wavefront, each number
# of rows per token that has a kernel of its own and one that has none
CASES = [dict(T=1, d=72, M=8, k=1), dict(T=17, d=264, M=24, k=3), dict(T=65, d=520, M=64, k=8), dict(T=250, d=64, M=16, k=2),
         dict(T=1030, d=776, M=40, k=4), dict(T=8200, d=2056, M=32, k=1)]


@pytest.mark.parametrize("kw", CASES)
@pytest.mark.parametrize("accumulate", [0, 1])
def test_router_part_alone(kw, accumulate, device):
    L = DeviceLayer(layer_inputs(custom_config(f=64, n_trainable=1, dtype="bf16", router_sigma=0.3, **kw)), device)
    print(f"[case] {kw}", flush=True)
    L.w_gate.zero_(); L.w_up.zero_()
    L.d_w_router.fill_(0.5)
    L.fwd()
    L.aux(0.5, 2.0 * kw["T"])                     # gradients of the order of 1
    L.bwd(accumulate); torch.cuda.synchronize()
    # the products' operands are bf16(dlogits), x and W_r; sums of n terms in fp32 are off by at most n 2^-24 of the sum of magnitudes, and
    # dx is rounded to bf16 once
    dl, w, x = L.view("dlogits").bfloat16().double(), L.w_router.double(), L.x.double()
    assert dl.abs().max() > 1e-3
    want, mag = dl @ w, dl.abs() @ w.abs()
    assert ((L.dx.double() - want).abs() <= 2.0 ** -8 * want.abs() + kw["M"] * 2.0 ** -24 * mag).all()
    want, mag = dl.t() @ x + 0.5 * accumulate, dl.abs().t() @ x.abs() + 0.5
    assert ((L.d_w_router.double() - want).abs() <= (kw["T"] + 64) * 2.0 ** -24 * mag).all()

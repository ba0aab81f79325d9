"""The router's part of dx and its weight gradient on the matrix cores: alone (with experts of zero weights nothing else is left of dx), and
beside the sum of the experts' rows."""
import pytest
import torch

import paper_2602_11543_amd as S
from spes_workloads import custom_config, layer_inputs

from harness import DeviceLayer

pytestmark = pytest.mark.gpu

# one token, remainders of 16 tokens and of 64 columns, whole and partial sets of 64 experts, 16 and 64 tokens a block
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


def _expert_rows(L):
    """The experts' parts of the input gradient in expert-contiguous order: the region behind dgate, its partials, da, db and gate * h."""
    T, d, f, k = L.cfg.T, L.cfg.d, L.cfg.f, L.cfg.k
    at = S.spes_moe_ctx_describe(L.shape)["dgate"]
    for size in (T * k * 4, (-(-f // 64) + 1) * T * k * 4, *[T * k * f * 2] * 3):
        at += -(-size // 256) * 256
    return L.ctx[at:][:T * k * d * 2].view(torch.bfloat16).view(T * k, d)


# 16, 32 and 64 tokens a block, each with a last group that is not whole; last columns of 8, 128 and 200, rows of whole lines and others; up to
# eight rows a token, and one, five and eight more
@pytest.mark.parametrize("T,d,M", [(250, 520, 16), (300, 384, 16), (1030, 456, 40), (4100, 2056, 24), (8203, 2056, 16)])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 16])
def test_expert_rows_and_router_part(T, d, M, k, device):
    """dx is the fp32 sum of a token's rows, slot by slot, plus the bf16 router part, rounded to bf16, bit for bit: with two powers of two in
    every column of W_r the router part before its rounding is exact in any order."""
    L = DeviceLayer(layer_inputs(custom_config(T=T, d=d, M=M, f=64, k=k, n_trainable=1, dtype="bf16", router_sigma=0.3)), device)
    print(f"[case] {T} {d} {M} {k}", flush=True)
    c = torch.arange(d, device=device)
    L.w_router.zero_()
    pair = torch.stack([c % M, (c + 1 + c // M % (M - 1)) % M])
    L.w_router[pair[0], c] = 0.125
    L.w_router[pair[1], c] = -0.25
    L.fwd()
    L.aux(0.5, 2.0 * T)                           # gradients of the order of 1
    L.bwd(); torch.cuda.synchronize()
    dl = L.view("dlogits").bfloat16().float()
    first, second = dl[:, pair[0]] * 0.125, dl[:, pair[1]] * -0.25
    rows, at = _expert_rows(L), L.view("inv").long().view(T, k)
    want = torch.zeros(T, d, device=device)
    for j in range(k):
        want += rows[at[:, j]].float()
    assert want.abs().max() > 1e-2 and first.abs().max() > 1e-2
    want = (want + (first + second).bfloat16().float()).bfloat16()
    # eight bits each, so the sum fits 24 where the exponents lie no more than 14 apart
    lo, hi = torch.minimum(first.abs(), second.abs()), torch.maximum(first.abs(), second.abs())
    exact = (lo * 2.0 ** 14 >= hi)
    assert exact.float().mean() > 0.9
    assert torch.equal(L.dx[exact], want[exact])

"""A result's bits follow from its operands: not from the tile, the XCD or the batch that a token falls into."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2602_11543_amd as S
from spes_workloads import bf16_round, custom_config, layer_inputs

from harness import DeviceLayer

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16 if t.element_size() == 2 else torch.int32)


def _correction(L):
    """What bf16 a and b miss of h: the region ahead of h."""
    at, h = S.spes_moe_ctx_describe(L.shape)["h"], L.view("h")
    size = -(-h.numel() * 2 // 256) * 256
    return L.ctx[at - size:][:h.numel() * 2].view(torch.bfloat16).view(h.shape)


def _equal_tokens(kw, n_base, device):
    """A layer whose T tokens are copies of n_base ones, in turn; each copy's number; what forward and backward say per token."""
    kw = {"router_sigma": 0.3, "n_trainable": 1, **kw}
    inp = layer_inputs(custom_config(**kw))
    copy_of = torch.arange(kw["T"]) % n_base
    inp["x"], inp["dy"] = inp["x"][copy_of.numpy()], inp["dy"][copy_of.numpy()]
    L = DeviceLayer(inp, device)
    print(f"[case] {kw} {n_base}", flush=True)
    L.fwd(); L.bwd(); torch.cuda.synchronize()
    row = L.view("inv").long().view(L.cfg.T, L.cfg.k)
    out = dict(y=L.y, dx=L.dx, **{n: L.view(n) for n in ("dgate", "dlogits")}, **{n: L.view(n)[row] for n in ("a", "b", "h")})
    if L.cfg.dtype == "bf16":
        out["correction"] = _correction(L)[row]
    return L, copy_of.to(device), out


# Long contractions and experts with several row tiles: 64-, 128- and 256-row ones (those with a half-height last tile, with a column
# tail and on half-width tiles as well: launches of few tiles, which run at half the height), launches with both whole tiles and such that are
# cut in two, and both tiles of fp32 layers.
SKEWED = dict(bias="normal", bias_scale=2.0)
POSITIONS = [
    (dict(T=384, d=1032, M=8, f=776, k=1, dtype="bf16", **SKEWED), 96, 64), (dict(T=192, d=2048, M=8, f=1024, k=2, dtype="bf16", **SKEWED), 64, 64),
    (dict(T=760, d=1032, M=8, f=392, k=1, dtype="bf16", **SKEWED), 190, 128),
    (dict(T=1800, d=1024, M=8, f=968, k=2, dtype="bf16"), 450, 256), (dict(T=1803, d=1032, M=8, f=1024, k=1, dtype="bf16", **SKEWED), 401, 256),
    (dict(T=4452, d=184, M=1, f=4040, k=1, dtype="bf16"), 100, 256),
    (dict(T=290, d=520, M=8, f=264, k=2), 70, 32), (dict(T=4100, d=264, M=8, f=520, k=4), 1000, 64),
]


@pytest.mark.parametrize("kw,n_base,rows", POSITIONS)
def test_equal_tokens_have_equal_results(kw, n_base, rows, device):
    L, copy_of, out = _equal_tokens(kw, n_base, device)
    assert int(L.count.max()) > rows, "more than one row tile"
    if rows == 256:
        assert any(n > 256 and 0 < n % 256 <= 128 for n in L.count.tolist()), "a half-height last tile"
    for name, t in out.items():
        assert torch.equal(_bits(t), _bits(t[:n_base])[copy_of]), name


def test_a_token_has_the_same_output_in_any_batch(device):
    """One set of weights, batches that run on 64-, 128- and 256-row tiles, the last one with the router on its tall tiles."""
    inp = layer_inputs(custom_config(T=9000, d=1032, M=8, f=776, k=2, dtype="bf16", n_trainable=0, router_sigma=0.3))
    first = None
    for T in (190, 380, 2000, 9000):
        L = DeviceLayer({**inp, "cfg": dataclasses.replace(inp["cfg"], T=T), "x": inp["x"][:T], "dy": inp["dy"][:T]}, device)
        L.fwd(); torch.cuda.synchronize()
        first = L.y if first is None else first
        assert torch.equal(_bits(L.y[:190]), _bits(first)), T


# 64-, 128- and 256-row tiles and fp32, several K-tiles with a remainder in both contractions
@pytest.mark.parametrize("T,dtype", [(90, "bf16"), (180, "bf16"), (700, "bf16"), (180, "f32")])
def test_equal_experts_have_equal_results(T, dtype, device):
    """Experts that are copies of one another (an upcycled layer's first step) give a token's rows equal bits, so that its gate gradients are
    equal, and with renormalised gates nothing but rounding is left of the score gradients."""
    L = DeviceLayer(layer_inputs(custom_config(T=T, d=1032, M=8, f=776, k=4, renorm=1, n_trainable=2, dtype=dtype, router_sigma=0.3)), device)
    print(f"[case] {T} {dtype}", flush=True)
    for w in (L.w_gate, L.w_up, L.w_down):
        w[1:] = w[:1].clone()
    L.fwd(); L.bwd(); torch.cuda.synchronize()
    row = L.view("inv").long().view(T, L.cfg.k)
    out = {n: L.view(n)[row] for n in ("a", "b", "h", "yp")}
    if dtype == "bf16":
        out["correction"] = _correction(L)[row]
    out["dgate"] = L.view("dgate")
    for name, t in out.items():
        assert torch.equal(_bits(t), _bits(t[:, :1]).expand(_bits(t).shape)), name
    # g_i (D sum_{j != i} g_j - sum_{j != i} D g_j) and g_i (D - D sum_j g_j): products, sums of at most 64 terms by halves, and gates that
    # add up to 1 but for their own rounding, each at most 2^-24 of D: fewer than 32 of them
    assert (L.view("dlogits").abs().amax(1) <= 32 * 2.0 ** -24 * L.view("dgate").abs().amax(1)).all()


def _pairs_whose_correction_shows_the_rounding(n):
    """a in [20, 32) and b in [16, 32), 24 bits each as three times eight, whose (a - bf16 a) bf16 b + a (b - bf16 b) is another bf16 value
    when the first product is rounded than when the second one is: the first is exact, the second has up to 40 bits."""
    rng = np.random.default_rng(1)
    low = 160, 128
    digits = [np.stack([rng.integers(lo, 256, 1 << 21), rng.integers(0, 256, 1 << 21), rng.integers(0, 256, 1 << 21)]) for lo in low]
    a, b = (np.ldexp((d[0] * 65536 + d[1] * 256 + d[2]).astype(np.float64), -19) for d in digits)
    ar, br = bf16_round(a.astype(np.float32)).astype(np.float64), bf16_round(b.astype(np.float32)).astype(np.float64)
    to_bf16 = lambda v: bf16_round(v.astype(np.float32))
    second, first = to_bf16((a - ar) * br + (a * (b - br)).astype(np.float32).astype(np.float64)), to_bf16((a - ar) * br + a * (b - br))
    pick = np.nonzero(first != second)[0][:n]
    assert len(pick) == n
    return [d[:, pick] for d in digits], second[pick]


@pytest.mark.parametrize("T", [40, 90, 300])        # 64-row, 128-row and 256-row tiles, the last with a half-height one
def test_the_correction_of_h_rounds_the_second_product(T, device):
    """Where the gate is saturated (sigmoid and its derivative 1 and 0) one rounding is left, and it is the same on every tile."""
    f = 64
    (ga, gb), want = _pairs_whose_correction_shows_the_rounding(f)
    L = DeviceLayer(layer_inputs(custom_config(T=T, d=904, M=1, f=f, k=1, n_trainable=0, dtype="bf16")), device)
    L.x.zero_(); L.w_gate.zero_(); L.w_up.zero_()
    for i in range(3):
        L.x[:, i] = 2.0 ** (-8 * i)
        L.w_gate[0, :, i], L.w_up[0, :, i] = (torch.from_numpy(g[i] / 8.0).to(device, torch.bfloat16) for g in (ga, gb))
    L.fwd(); torch.cuda.synchronize()
    assert torch.equal(_correction(L).float(), torch.from_numpy(want).to(device).expand(T, f))


# trainable experts on either side of the line between two tiles of the weight gradients
MASKS = [(dict(T=1032, d=512, M=16, f=512, k=8, dtype="bf16"), (10, 11)),
         (dict(T=3001, d=136, M=32, f=120, k=8), (14, 15)), (dict(T=150, d=128, M=32, f=128, k=4), (21, 22))]


@pytest.mark.parametrize("kw,numbers", MASKS)
def test_weight_gradients_under_any_mask(kw, numbers, device):
    """Expert e's gradients have the same bits whichever others are trainable."""
    few, more = numbers
    L = DeviceLayer(layer_inputs(custom_config(router_sigma=0.3, n_trainable=few, **kw)), device)
    print(f"[case] {kw} {numbers}", flush=True)
    L.fwd()
    got = []
    for n in (few, more, 1):
        L.set_mask([int(e < n) for e in range(kw["M"])])
        L.bwd(); torch.cuda.synchronize()
        got.append([t[:n] for t in (L.d_w_gate, L.d_w_up, L.d_w_down)] + [L.dx.clone(), L.d_w_router.clone()])
    for other in got[1:]:
        for i, (a, b) in enumerate(zip(got[0], other)):
            n = min(len(a), len(b))
            assert torch.equal(_bits(a[:n]), _bits(b[:n])), i

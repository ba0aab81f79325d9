"""The main loop of the expert GEMMs: contractions of one to a few K-tiles with and without a remainder on each row tile, and
nothing from beyond a contraction range, a tile or an expert in any result."""
import numpy as np
import pytest
import torch

from spes_workloads import custom_config, layer_inputs

from harness import DeviceLayer
from test_gpu_layer import _full_parity

pytestmark = pytest.mark.gpu

# tokens, d_model, experts, d_ff, top-k: both widths are contraction lengths (forward and backward), 64 to a K-tile
CASES = [
    # 64-row tiles: 1, 2, 3, 5, 8, 9 and 13 K-tiles
    (40, 64, 4, 128, 2), (40, 72, 4, 184, 2), (60, 320, 8, 512, 2), (60, 520, 8, 576, 2), (60, 776, 8, 832, 2),
    # 128-row tiles
    (96, 64, 2, 128, 2), (150, 328, 4, 136, 2), (150, 1000, 4, 200, 2),
    # 256-row tiles, full and half-width columns; launches of this size cut them in two (FULL_HEIGHT has those that do not)
    (300, 960, 2, 64, 2), (300, 968, 2, 136, 2), (300, 1024, 2, 320, 2), (700, 1096, 3, 72, 2),
]


@pytest.mark.parametrize("T,d,M,f,k", CASES)
def test_contraction_lengths(T, d, M, f, k, device):
    kw = dict(T=T, d=d, M=M, f=f, k=k, n_trainable=min(3, M), trainable="random", dtype="bf16", router_sigma=0.3)
    _full_parity(layer_inputs(custom_config(**kw)), device, "contraction lengths")


# contractions of 17 and 18 K-tiles, the last one short, for up to 64 experts on 64-row and on 256-row tiles
@pytest.mark.parametrize("T,d,M,f,k", [(300, 1096, 64, 1128, 4), (3300, 1096, 33, 136, 8)])
def test_first_k_tiles_of_many_experts(T, d, M, f, k, device):
    kw = dict(T=T, d=d, M=M, f=f, k=k, n_trainable=2, trainable="random", dtype="bf16", router_sigma=0.02, bias="normal")
    _full_parity(layer_inputs(custom_config(**kw)), device, "many experts")


# One expert and more than 128 tiles of 256 rows in a launch, so that whole ones are left: T, d_model, d_ff, and how many in the GEMMs
# gate + up, SwiGLU backward, down projection and input gradient, the column tail of the latter two on its own (test_plan.py counts them).
# One, two and three K-tiles with and without a remainder on the tile of each.
FULL_HEIGHT = [
    *[(4452, d, 4040, (512, 256, 0), (0, 0)) for d in (56, 64, 72, 128, 184)],          # SwiGLU backward of 256 whole tiles and 16 that are cut
    *[(5120, d, 1024, (160, 160, 0), (0, 0)) for d in (72, 184)],                      # on half-width tiles
    *[(5120, 1024, f, (0, 0, 160), (0, 0)) for f in (56, 64, 72, 136)],                # input gradient and down projection, half-width
    *[(10240, 1000, f, (0, 0, 160), (0, 0)) for f in (56, 72, 136)],                   # full-width
    (33600, 72, 296, (393, 131, 131), (131, 0)), (33600, 264, 72, (131, 131, 131), (0, 131)),     # column tails
]


@pytest.mark.parametrize("T,d,f", [case[:3] for case in FULL_HEIGHT])
def test_contraction_lengths_at_full_height(T, d, f, device):
    kw = dict(T=T, d=d, M=1, f=f, k=1, n_trainable=1, dtype="bf16")
    _full_parity(layer_inputs(custom_config(**kw)), device, "full height")


# one expert's rows around the heights of full and half tiles; with whole columns, a column tail, and on half-width tiles: launches of a few
# tiles, all of them half-height
@pytest.mark.parametrize("T", [128, 129, 256, 257, 384, 385, 641])
@pytest.mark.parametrize("d,f", [(904, 136), (1032, 328), (1024, 256)])
def test_last_rows(T, d, f, device):
    kw = dict(T=T, d=d, M=1, f=f, k=1, n_trainable=1, dtype="bf16", router_sigma=0.3)
    _full_parity(layer_inputs(custom_config(**kw)), device, "last rows")


# full tiles of the forward launch beyond a whole round of 256, by one expert's rows times the columns: 32 that are cut in two, alone and
# beside half-height tiles, 167 that are not; the backward has launches of 9, 16 and 18, which are cut, and of 144 and 207, which are not
@pytest.mark.parametrize("T,d,f", [(2248, 256, 4096), (2148, 256, 4608), (2200, 128, 6016)])
def test_last_round_of_full_tiles(T, d, f, device):
    kw = dict(T=T, d=d, M=1, f=f, k=1, n_trainable=1, dtype="bf16", router_sigma=0.3)
    _full_parity(layer_inputs(custom_config(**kw)), device, "last round")


# 64-, 128- and 256-row tiles, the last in launches of few, and of more than 128 in gate + up and the SwiGLU backward or in the other two
@pytest.mark.parametrize("T,d,f", [(60, 136, 200), (200, 1000, 136), (700, 960, 328), (700, 520, 520), (4400, 136, 2000), (6000, 1000, 136)])
def test_values_stay_with_their_expert(T, d, f, device):
    """NaN weights of one expert: every result of tokens and experts that have nothing to do with it stays bit for bit."""
    cfg = custom_config(T=T, d=d, M=5, f=f, k=2, n_trainable=5, dtype="bf16", router_sigma=0.3)
    L = DeviceLayer(layer_inputs(cfg), device)
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
        assert torch.equal(a[pick].view(torch.uint8), b[pick].view(torch.uint8)), i
        assert torch.isfinite(b[pick].float()).all(), i

"""Expert GEMMs on 64-, 128- and 256-row tiles: both sides of each line of the rule, remainders of rows and columns, empty experts."""
import pytest

from spes_workloads import custom_config, layer_inputs

from test_gpu_layer import _full_parity

pytestmark = pytest.mark.gpu

# (256-row tiles in launches of up to 128 of them run as pairs of half-height ones; test_gpu_gemm_loop.py has larger ones)
# case, rows per tile, and how full tiles cut the columns of the down projection: a tail of that many columns on half-width
# tiles, half-width tiles throughout, or full ones (test_plan.py checks both)
CASES = [
    (dict(T=1, d=904, M=4, f=8, k=1, n_trainable=2), 64, "short"),                                   # one row in the launch
    (dict(T=96, d=904, M=8, f=136, k=4, n_trainable=3), 64, "short"),                                # 48 a head: the last 64-row case
    (dict(T=97, d=904, M=8, f=264, k=4, n_trainable=3, bias="normal", bias_scale=2.0), 128, "short"),    # full and ragged tiles
    (dict(T=192, d=1032, M=8, f=72, k=4, n_trainable=3, bias="normal", bias_scale=8.0), 128, "short"),   # 96 a head, experts without a row
    (dict(T=193, d=904, M=8, f=136, k=4, n_trainable=3), 256, "full"),
    (dict(T=260, d=1032, M=8, f=328, k=4, n_trainable=3), 256, 8),                                   # column tails of 8 and 72
    (dict(T=300, d=1024, M=8, f=512, k=4, n_trainable=3), 256, "half"),                              # half-width launches
    (dict(T=300, d=1152, M=6, f=640, k=2, n_trainable=2), 256, 128),                                 # tails exactly half a tile wide
    (dict(T=300, d=1088, M=6, f=576, k=2, renorm=1, n_trainable=3), 256, 64),                        # a quarter
    (dict(T=512, d=896, M=4, f=200, k=2, n_trainable=2), 64, "short"),                               # short contraction, 256 a head
    (dict(T=1100, d=264, M=16, f=1048, k=8, n_trainable=2), 128, "short"),                           # 378 full tiles, 1.48 rounds
    (dict(T=1040, d=256, M=8, f=1024, k=4, n_trainable=2), 256, "half"),                             # 160 full tiles
    (dict(T=1023, d=640, M=4, f=136, k=2, n_trainable=2), 64, "short"),                              # shorter one, 511.5 a head
    (dict(T=64, d=136, M=8, f=552, k=2, n_trainable=8, bias="normal", bias_scale=8.0), 64, "short"),     # d_ff > 4 d_model
    (dict(T=400, d=136, M=8, f=544, k=2, n_trainable=2), 64, "short"),                               # 100 a head, d_ff = 4 d_model ...
    (dict(T=400, d=136, M=8, f=552, k=2, n_trainable=2), 256, "full"),                               # ... and beyond
    (dict(T=1536, d=768, M=8, f=1024, k=2, n_trainable=2), 256, "half"),                             # 128 full tiles
    (dict(T=1040, d=768, M=64, f=1664, k=4, n_trainable=2), 128, "short"),                           # 624 full tiles, 65 a head
    (dict(T=3072, d=520, M=64, f=2080, k=4, n_trainable=2), 128, "short"),                           # 1360, d_model with a column tail
    (dict(T=1600, d=768, M=64, f=2304, k=4, n_trainable=2), 256, "full"),                            # 1026, none
]


@pytest.mark.parametrize("kw,rows,down", CASES)
def test_row_tiles(kw, rows, down, device):
    kw = {"dtype": "bf16", "router_sigma": 0.3, "trainable": "random", **kw}
    _full_parity(layer_inputs(custom_config(**kw)), device, f"{rows}-row tiles")

"""Expert GEMMs on 64-, 128- and 256-row tiles: both sides of each line of the rule, remainders of rows and columns, empty experts."""
import pytest

from spes_workloads import custom_config, layer_inputs

from test_gpu_layer import _full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(T=1, d=904, M=4, f=8, k=1, n_trainable=2),                                   # one row in the launch
    dict(T=96, d=904, M=8, f=136, k=4, n_trainable=3),                                # 48 a head: the last 64-row case
    dict(T=97, d=904, M=8, f=264, k=4, n_trainable=3, bias="normal", bias_scale=2.0),    # 128 rows, full and ragged tiles
    dict(T=192, d=1032, M=8, f=72, k=4, n_trainable=3, bias="normal", bias_scale=8.0),   # 96 a head, experts without a row
    dict(T=193, d=904, M=8, f=136, k=4, n_trainable=3),                               # 256 rows
    dict(T=260, d=1032, M=8, f=328, k=4, n_trainable=3),                              # 256 rows, column tails of 8 and 72
    dict(T=300, d=1024, M=8, f=512, k=4, n_trainable=3),                              # 256 rows, half-width launches
    dict(T=512, d=896, M=4, f=200, k=2, n_trainable=2),                               # short contraction, 256 a head
    dict(T=1100, d=264, M=16, f=1048, k=8, n_trainable=2),                            # 128 rows: 378 full tiles, 1.48 rounds
    dict(T=1040, d=256, M=8, f=1024, k=4, n_trainable=2),                             # 256 rows: 160 full tiles
    dict(T=1023, d=640, M=4, f=136, k=2, n_trainable=2),                              # shorter one, 511.5 a head
    dict(T=64, d=136, M=8, f=552, k=2, n_trainable=8, bias="normal", bias_scale=8.0),    # d_ff > 4 d_model
])
def test_row_tiles(kw, device):
    kw = {"dtype": "bf16", "router_sigma": 0.3, "trainable": "random", **kw}
    _full_parity(layer_inputs(custom_config(**kw)), device, "row tiles")

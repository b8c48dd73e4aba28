"""The fp32 path's activations in the epilogues of its products: each tile size, features that fill a tile and that do not."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# (hidden, ffn, tokens): 16-, 32- and 64-wide tiles of the up projection and of the gradient behind the down projection; ffn of less than half a tile,
# not a multiple of one, and one short vector past it; a hidden width no 16-byte load takes (the stand-alone kernels)
@pytest.mark.parametrize("hidden,ffn,tokens", [(64, 4, 5), (64, 36, 33), (96, 260, 131), (64, 1028, 300), (128, 1540, 700), (30, 44, 17), (64, 2052, 520)])
@pytest.mark.parametrize("mlp,bias", [("swiglu", True), ("gelu", False)])
def test_f32_fused_activations(hidden, ffn, tokens, mlp, bias):
    shape = SI.StageShape(f"f32act{hidden}.{ffn}", 1, hidden, 2, 1, 16, ffn, 2, dtype="fp32", x_std=1.0, dy_std=1.0, w_std=0.1, mlp_kind=mlp, bias=bias)
    w = Hp.Workload(shape, [[0, (tokens + 1) // 2, tokens], [0, 3]])
    print(f"[f32 activation] {hidden} {ffn} {tokens} {mlp} bias{bias}", flush=True)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL["fp32"], shape.name)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, order=SI.ready_order(w.M, 3), n_streams=2, keep_raw=True))
    print(f"[f32 activation] {hidden} {ffn} {mlp}: worst {worst:.2e}", flush=True)

"""The weight gradients of all layers of a task in one launch: each way the list can be cut, against the oracle."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# (layers, hidden, q heads, kv heads, head_dim, ffn, dtype, tokens)
CASES = [
    (9, 64, 1, 1, 64, 64, "bf16", 33),        # two lists; 64 x 64 tiles; K one past a step
    (2, 320, 5, 1, 64, 448, "bf16", 1500),    # 256-row tiles, ragged at both edges, every one cut along K
    (2, 1024, 8, 8, 128, 2816, "bf16", 520),  # one whole round of tiles and a cut rest
    (9, 32, 2, 1, 16, 48, "fp32", 65),        # two lists of 32 x 32 tiles
    (2, 30, 1, 1, 16, 44, "fp32", 17),        # rows that are not whole float4s
    (1, 516, 4, 2, 128, 900, "fp32", 100),    # 64 x 64 tiles, ragged
]


@pytest.mark.parametrize("layers,hidden,nq,nkv,d,ffn,dtype,tokens", CASES)
def test_grouped_weight_gradients(layers, hidden, nq, nkv, d, ffn, dtype, tokens):
    """Rounding of the storage types as in the other parity tests; a tile, range or product in the wrong place is an error of order one."""
    shape = SI.StageShape(f"wgroup{layers}.{hidden}.{ffn}", layers, hidden, nq, nkv, d, ffn, 2, dtype=dtype, x_std=1.0, dy_std=1.0,
                          w_std=0.5 / np.sqrt(hidden))
    w = Hp.Workload(shape, [[0, tokens // 3, tokens]])
    print(f"[wgrad group] {shape.name} {dtype} {tokens} tokens", flush=True)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, keep_raw=True))
    print(f"[wgrad group] {shape.name}: worst {worst:.2e}", flush=True)

"""Rotary embedding and head norm at every head dimension: vectors per head that are and are not a power of two, rows and heads past what a
workgroup or a thread takes at once."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype", [(16, "fp32"), (32, "fp32"), (48, "fp32"), (64, "fp32"), (80, "fp32"), (96, "fp32"), (112, "fp32"), (128, "fp32"),
                                     (64, "bf16"), (80, "bf16"), (128, "bf16")])
@pytest.mark.parametrize("rope,qk_norm", [(True, False), (False, True), (True, True)])
def test_rope_and_head_norm(d, dtype, rope, qk_norm):
    """12 query and 4 key heads (eight turns of two heads a thread); segments past a query tile of 256 rows and of one row."""
    shape = SI.StageShape(f"heads{d}", 1, 64, 12, 4, d, 64, 2, dtype=dtype, x_std=1.0, dy_std=1.0, w_std=0.06, rope=rope, rope_base=700.0, qk_norm=qk_norm)
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum([1, 259, 37])], [0, 17]])
    print(f"[head variants] d{d} {dtype} rope{rope} qk_norm{qk_norm}", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    print(f"[head variants] d{d} {dtype}: worst {worst:.2e}", flush=True)


@pytest.mark.parametrize("d,dtype,nq,lengths", [
    (64, "bf16", 1, [[32] * 3 + [31, 1], [1] * 40]), (80, "bf16", 4, [[51, 52, 1], [1, 257]]), (128, "bf16", 1, [[16, 15], [255, 17]]),
    (16, "fp32", 1, [[1] * 5, [128, 129, 3]]), (48, "fp32", 3, [[42, 41], [43, 1, 256]]), (128, "fp32", 2, [[16, 17, 1], [8] * 9])])
def test_rope_blocks_of_a_tile(d, dtype, nq, lengths):
    """As many blocks of rows are launched for a tile as the longest segment has: segments of one block, one row more and one less, and
    of a tile; head counts that a thread's heads do and do not divide."""
    shape = SI.StageShape(f"ropeblocks{d}", 1, 64, nq, nq, d, 64, 2, dtype=dtype, x_std=1.0, dy_std=1.0, w_std=0.06, rope=True, rope_base=700.0)
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(n)] for n in lengths])
    print(f"[rope blocks] d{d} {dtype} {nq} heads", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    print(f"[rope blocks] d{d} {dtype}: worst {worst:.2e}", flush=True)

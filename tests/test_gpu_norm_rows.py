"""RMSNorm backward with 2, 4 and 8 rows per workgroup (by the number of rows), through a stage of hidden 1024."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# one row; one past a workgroup of two; the last counts of 2 and of 4 rows per workgroup on 256 CUs and the next ones
@pytest.mark.parametrize("tokens,dtype,rows", [(1, "bf16", 2), (3, "fp32", 2), (1020, "bf16", 2), (1020, "fp32", 2), (1021, "bf16", 4),
                                               (1021, "fp32", 4), (2040, "bf16", 4), (2040, "fp32", 4), (2041, "bf16", 8), (2041, "fp32", 8)])
def test_norm_backward_rows(tokens, dtype, rows):
    """The storage type's tolerance: a row left out of or counted twice in a gain gradient moves it by about 1 / sqrt(tokens)
    of itself or more, 2.2e-2 at the largest size, and a dx row missed is an error of order one."""
    import torch
    import paper_2605_18750_amd as R
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    assert R.rrfp_rmsnorm_bwd_rows(tokens, 1024, R.STAGE_DTYPE_FP32 if dtype == "fp32" else R.STAGE_DTYPE_BF16) == rows
    shape = SI.StageShape(f"normrows{tokens}", 1, 1024, 1, 1, 64, 64, 2, dtype=dtype, x_std=1.0, dy_std=1.0, w_std=0.02)
    cu = [0] + [c for c in range(200, tokens, 200)] + [tokens]
    w = Hp.Workload(shape, [cu])
    print(f"[norm rows] {tokens} {dtype}", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL[dtype], f"{tokens}")
    print(f"[norm rows] {tokens} {dtype}: worst {worst:.2e}", flush=True)

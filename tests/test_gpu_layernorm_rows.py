"""LayerNorm backward and bias column sums, vector and scalar kernels, at the edges of their rows, chunks and column blocks."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# (hidden, ffn, dtype, tokens): odd hidden (scalar); one vector; three; the last that stay in registers; rows around 8 and 64
@pytest.mark.parametrize("hidden,ffn,dtype,tokens", [(30, 44, "fp32", 65), (36, 44, "fp32", 7), (64, 64, "bf16", 1), (320, 192, "bf16", 129),
                                                     (1280, 320, "bf16", 72), (2048, 64, "fp32", 9), (4096, 64, "bf16", 63), (4160, 64, "bf16", 10)])
def test_layernorm_and_bias_gradients(hidden, ffn, dtype, tokens):
    """The storage type's tolerance; a row, chunk or column block missed moves a gradient by 1 / sqrt(129) of itself or more."""
    shape = SI.StageShape(f"lnrows{hidden}", 1, hidden, 1, 1, 64, ffn, 2, dtype=dtype, mlp_kind="gelu", causal=False, x_std=1.0, dy_std=1.0,
                          w_std=0.02, norm_kind="layer", bias=True)
    w = Hp.Workload(shape, [[0, (tokens + 1) // 2, tokens]] if tokens > 1 else [[0, 1]])
    print(f"[layernorm rows] {hidden} {ffn} {dtype} {tokens}", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    print(f"[layernorm rows] {hidden} {dtype} {tokens}: worst {worst:.2e}", flush=True)

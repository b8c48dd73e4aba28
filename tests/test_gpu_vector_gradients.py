"""The vector gradients of a B task, listed and summed together at its end: more sums than one launch takes, odd widths, the split bias
behind a head norm."""
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# (layers, hidden, ffn, dtype, norm_kind, bias, qk_norm, tokens): 66 sums (two launches, none of them of a bias); 17 layers = 136 sums and 68
# tensors with biases, the lists' limit met inside both; widths that take the kernel of single columns; key block apart, 70 sums
@pytest.mark.parametrize("layers,hidden,ffn,dtype,norm_kind,bias,qk_norm,tokens", [
    (33, 32, 32, "fp32", "rms", False, False, 40), (17, 32, 32, "fp32", "layer", True, False, 65), (2, 30, 44, "fp32", "rms", True, False, 66),
    (2, 64, 64, "bf16", "layer", True, True, 130), (7, 64, 64, "bf16", "rms", True, True, 33)])
def test_vector_gradients_of_a_task(layers, hidden, ffn, dtype, norm_kind, bias, qk_norm, tokens):
    """The storage type's tolerance; a sum missed or taken before its rows leaves NaN or another layer's values in the slot."""
    shape = SI.StageShape(f"vector{layers}.{hidden}", layers, hidden, 2, 1, 64 if dtype == "bf16" else 16, ffn, 2, dtype=dtype, x_std=1.0, dy_std=1.0,
                          w_std=0.02, norm_kind=norm_kind, bias=bias, qk_norm=qk_norm)
    w = Hp.Workload(shape, [[0, 7, tokens], [0, 1]])
    print(f"[vector gradients] {shape.name} {dtype} {norm_kind} bias{bias} qk{qk_norm} {tokens}", flush=True)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, order=SI.ready_order(w.M, 5), n_streams=2, keep_raw=True))
    print(f"[vector gradients] {shape.name}: worst {worst:.2e}", flush=True)

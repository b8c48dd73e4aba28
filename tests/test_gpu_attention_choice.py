"""The bf16 path's attention on both sides of the rules that choose its kernels, with ragged segments."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


def _plans(shape, w):
    import paper_2605_18750_amd as R
    dtype = R.STAGE_DTYPE_FP32 if shape.dtype == "fp32" else R.STAGE_DTYPE_BF16
    return ["".join("xd"[v] for v in R.rrfp_attn_plan(cu, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, int(shape.causal), dtype).values()) for cu in w.cus]


def _check(shape, lengths, plans=None):
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(n)] for n in lengths])
    print(f"[attention choice] {shape.name} causal{shape.causal} {shape.dtype} {_plans(shape, w)}", flush=True)
    if plans is not None:
        assert _plans(shape, w) == plans
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL[shape.dtype], shape.name)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, order=SI.ready_order(w.M, 3), n_streams=2, keep_raw=True))
    print(f"[attention choice] {shape.name}: worst {worst:.2e}", flush=True)


@pytest.mark.parametrize("d,causal,nkv", [(64, True, 64), (64, False, 16), (64, True, 4), (80, True, 16), (80, False, 64), (128, True, 8), (128, False, 64)])
def test_attention_choice_of_kernels(d, causal, nkv):
    """64 query heads: 256 tokens (64 rows a CU on 256 CUs) may take the kernels that deal the other side to the wavefronts, and dQ does, 257 not.
    Segments of one row, around a block of 32 and a tile of 128, and past what eight wavefronts take in one turn with 600 tokens of 4 heads."""
    for nq, kv, lengths in ((64, nkv, [[1, 31, 33, 127, 64], [32, 96, 129]]), (4, 4 if d == 80 or nkv == 64 else 2, [[1, 2, 255, 342], [289]])):
        _check(SI.StageShape(f"choice{d}.{nq}.{kv}", 1, 64, nq, kv, d, 64, 2, x_std=1.0, dy_std=1.0, w_std=0.06, causal=causal), lengths)


# (dtype, d, causal, q heads, kv heads, segments of the microbatches, their forward, dK/dV and dQ kernels: d dealt, x tiled).  Tiles of which one, two
# and all sub-tiles are launched, the last one of a longest segment one row long; every kernel of one choice beside the others of the other;
# one head, whose sub-tiles alone spread over the chip; as many query heads of a KV head as there are subsets, and more; 600 tokens of heads that fill it
CASES = [
    ("bf16", 64, True, 1, 1, [[32] * 9 + [1, 31], [33, 32, 1], [257, 256, 64]], ["ddd", "ddd", "ddd"]),
    ("bf16", 64, False, 16, 1, [[1, 31, 33, 127, 64], [129, 128]], ["ddd", "ddd"]),
    ("bf16", 64, True, 8, 2, [[32, 31] * 16 + [32] * 30, [160] * 10, [257, 160] * 4], ["dxd", "xxd", "xxd"]),
    ("bf16", 80, True, 4, 4, [[32, 1, 17], [33, 255, 2], [257, 31]], ["dxd", "dxd", "dxd"]),
    ("bf16", 80, False, 16, 4, [[97] * 8, [200, 1, 64]], ["xxx", "dxd"]),
    ("bf16", 128, True, 32, 4, [[16, 9, 32, 1] * 6, [256, 129, 97], [70] * 7], ["dxd", "xxd", "xxd"]),
    ("fp32", 64, True, 1, 1, [[16] * 9 + [1, 15], [17, 16, 1], [257, 256, 64]], ["ddd", "ddd", "ddd"]),
    ("fp32", 48, False, 4, 2, [[64] * 20 + [33], [257, 160, 129] * 4], ["dxd", "dxx"]),
    ("fp32", 64, True, 16, 4, [[97] * 8, [130] * 10, [64] * 20], ["dxd", "xxx", "dxd"]),
    ("fp32", 128, True, 16, 16, [[130] * 5, [16, 1, 9] * 20, [300] * 3], ["xxd", "ddd", "xxd"]),
]


@pytest.mark.parametrize("dtype,d,causal,nq,nkv,lengths,plans", CASES)
def test_attention_kernels_and_sub_tiles(dtype, d, causal, nq, nkv, lengths, plans):
    """The storage type's tolerance; a sub-tile left out or done twice, or a block of dS that only the other kind writes, is an error of order one."""
    shape = SI.StageShape(f"subtiles{d}.{nq}.{nkv}", 1, 64, nq, nkv, d, 64, 2, dtype=dtype, x_std=1.0, dy_std=1.0, w_std=0.06, causal=causal)
    _check(shape, lengths, plans)

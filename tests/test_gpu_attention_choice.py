"""The bf16 path's attention on both sides of the rule that chooses its kernels, with ragged segments."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,causal,nkv", [(64, True, 64), (64, False, 16), (64, True, 4), (80, True, 16), (80, False, 64), (128, True, 8), (128, False, 64)])
def test_attention_choice_of_kernels(d, causal, nkv):
    """64 query heads: 256 tokens (64 rows a CU on 256 CUs) take the kernels that deal the other side to the wavefronts, 257 the tiled ones.
    Segments of one row, around a block of 32 and a tile of 128, and past what eight wavefronts take in one turn with 600 tokens of 4 heads."""
    for nq, kv, lengths in ((64, nkv, [[1, 31, 33, 127, 64], [32, 96, 129]]), (4, 4 if d == 80 or nkv == 64 else 2, [[1, 2, 255, 342], [289]])):
        shape = SI.StageShape(f"choice{d}.{nq}.{kv}", 1, 64, nq, kv, d, 64, 2, x_std=1.0, dy_std=1.0, w_std=0.06, causal=causal)
        w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(n)] for n in lengths])
        print(f"[attention choice] d{d} causal{causal} heads {nq}/{kv}", flush=True)
        got = Hp.run_gpu(w, keep_raw=True)
        worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL["bf16"], shape.name)
        Hp.assert_bit_identical(got, Hp.run_gpu(w, order=SI.ready_order(w.M, 3), n_streams=2, keep_raw=True))
        print(f"[attention choice] d{d} heads {nq}/{kv}: worst {worst:.2e}", flush=True)

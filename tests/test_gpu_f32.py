"""The fp32 matrix-instruction kernels at the edges of their tiles, against fp64 definitions."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu

# (M, N, K): one element; one short of, at and past a 32- and a 64-tile; K below, at and past a chunk of 8 and a step of
# 32; outputs of 127 and 128+ tiles of 64 x 64 (the last size of the small kernel, the first of the tile kernel)
GEMM_SHAPES = [(1, 1, 1), (31, 33, 7), (32, 64, 8), (63, 65, 33), (70, 45, 31), (8 * 64 + 1, 14 * 64, 40), (8 * 64, 15 * 64 + 63, 9),
               (8 * 64, 16 * 64, 32), (8 * 64 + 7, 16 * 64 + 3, 70), (1025, 516, 129)]
# one short of, at and past a 16-tile, a chunk of 16 k and the k range of a wavefront; 96 tiles of 32 x 32 (the last size of the 16-tile
# kernel) and 99, 97
TINY_SHAPES = [(15, 17, 15), (16, 16, 16), (17, 31, 129), (33, 47, 513), (8 * 32, 12 * 32, 130), (8 * 32 + 1, 11 * 32, 127), (1, 97 * 32, 20)]

# the tile kernel with 16-byte loads: ragged tiles, K of one to seven steps of 32 (its loop has six), whole and not
VEC_SHAPES = [(516, 1028, 4), (700, 900, 36), (520, 1044, 64), (512, 1024, 100), (580, 960, 160), (516, 1088, 188), (640, 900, 228)]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("pad", [0, 3])
def test_f32_gemm_tile_edges(ta, tb, pad):
    """pad = 3: leading dimensions and start addresses that no 16-byte load could take.  Bound per element: K products and
    K sums, each within 2^-24 of its exact value."""
    import torch
    import paper_2605_18750_amd as R
    from paper_2605_18750_amd import harness as Hn
    for M, N, K in GEMM_SHAPES + TINY_SHAPES + VEC_SHAPES:
        print(f"[f32 gemm] M{M} N{N} K{K} ta{ta} tb{tb} pad{pad}", flush=True)
        shp = [(K, M) if ta else (M, K), (N, K) if tb else (K, N), (M, N)]
        A, B, Rr = [SI.make_tensor(7, f"f32{M}.{N}.{K}{n}", s, 1.0, "fp32") for n, s in zip("ABR", shp)]
        ref = (A.f64.T if ta else A.f64) @ (B.f64.T if tb else B.f64) + Rr.f64
        mag = np.abs(A.f64.T if ta else A.f64) @ np.abs(B.f64.T if tb else B.f64) + np.abs(Rr.f64)
        dev = []
        for t, s in zip((A, B, Rr), shp):
            buf = torch.full((s[0] * (s[1] + pad) + pad,), float("nan"), dtype=torch.float32, device="cuda:0")
            v = buf[pad:].view(s[0], s[1] + pad)[:, :s[1]]
            v.copy_(Hn.to_device(t.storage, "fp32"))
            dev.append(v)
        C = torch.full((M, N + pad), float("nan"), dtype=torch.float32, device="cuda:0")
        R.rrfp_gemm(dev[0], dev[1], C, dev[2], M, N, K, shp[0][1] + pad, shp[1][1] + pad, N + pad, N + pad, ta, tb, 0, 0)
        torch.cuda.synchronize()
        got = C.cpu().to(torch.float64).numpy()
        assert np.isnan(got[:, N:]).all(), "columns past N written"
        assert (np.abs(got[:, :N] - ref) <= (2 * K + 2) * 2.0 ** -24 * mag).all(), (M, N, K)


@pytest.mark.parametrize("d,causal,nq,nkv", [(16, True, 4, 2), (32, False, 2, 2), (48, True, 3, 1), (64, True, 2, 2), (80, False, 4, 1),
                                             (96, True, 2, 1), (112, False, 2, 2), (128, True, 2, 1)])
def test_f32_attention_tile_edges(d, causal, nq, nkv):
    """Every head dimension, with and without grouped heads; segments around the 16 rows of a wavefront, the 32 of a step,
    the 64 of a workgroup and the 128 / 256 of the host's tiles."""
    shape = SI.StageShape(f"f32attn{d}", 1, 32, nq, nkv, d, 32, 2, dtype="fp32", x_std=1.0, dy_std=1.0, w_std=0.15, causal=causal)
    lengths = [[1, 15, 16, 17, 31, 32, 33, 63, 64, 65], [127, 129, 257]]
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(n)] for n in lengths])
    print(f"[f32 attention] d{d} causal{causal} heads {nq}/{nkv}", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL["fp32"], f"d{d}")
    print(f"[f32 attention] d{d}: worst {worst:.2e}", flush=True)


@pytest.mark.parametrize("d,causal,nkv", [(16, True, 64), (32, False, 8), (48, True, 16), (64, True, 4), (80, False, 16), (96, True, 32),
                                          (112, False, 16), (128, True, 4)])
def test_f32_attention_choice_of_kernels(d, causal, nkv):
    """64 query heads: from 512 tokens on (2 x 64 rows a CU on 256 CUs) the 64-row kernels run, at 87 the ones that deal the other side to the
    wavefronts, at 511 the one or the other.  Segments around 16 and 128 rows (one and all blocks of eight wavefronts)."""
    shape = SI.StageShape(f"f32choice{d}", 1, 32, 64, nkv, d, 32, 2, dtype="fp32", x_std=1.0, dy_std=1.0, w_std=0.15, causal=causal)
    lengths = [[1, 17, 127, 129, 15, 223], [16, 144, 128, 223], [17, 15, 55]]
    assert [sum(n) for n in lengths] == [512, 511, 87]
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(n)] for n in lengths])
    print(f"[f32 attention] d{d} causal{causal} heads 64/{nkv}", flush=True)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL["fp32"], f"d{d}")
    Hp.assert_bit_identical(got, Hp.run_gpu(w, keep_raw=True))
    print(f"[f32 attention] d{d}: worst {worst:.2e}", flush=True)


def test_f32_attention_many_segments():
    """33 000 segments of one or two tokens: 132 000 sub-tiles of queries and 66 000 of keys, more than the 65 535 workgroups a
    grid takes in y."""
    shape = SI.StageShape("f32manysegments", 1, 32, 2, 1, 16, 32, 1, dtype="fp32", x_std=1.0, dy_std=1.0, w_std=0.15)
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum(1 + np.arange(33000) % 2)]])
    print(f"[f32 attention] {len(w.cus[0]) - 1} segments, {w.cus[0][-1]} tokens", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL["fp32"], "many segments")
    print(f"[f32 attention] many segments: worst {worst:.2e}", flush=True)


def test_f32_attention_many_segments_of_one_head():
    """16 400 segments of a token and one of 64: the kernels that deal the other side to the wavefronts, four sub-tiles a segment, 65 604 of them
    in the forward and dQ kernels."""
    import paper_2605_18750_amd as R
    shape = SI.StageShape("f32manysegments1", 1, 32, 1, 1, 16, 32, 1, dtype="fp32", x_std=1.0, dy_std=1.0, w_std=0.15)
    w = Hp.Workload(shape, [[0] + [int(v) for v in np.cumsum([1] * 9000 + [64] + [1] * 7400)]])
    assert R.rrfp_attn_plan(w.cus[0], 1, 1, 16, 1, R.STAGE_DTYPE_FP32) == dict(forward=True, dkv=False, dq=True)
    print(f"[f32 attention] {len(w.cus[0]) - 1} segments of one head", flush=True)
    worst = Hp.compare(Hp.run_gpu(w), Hp.run_oracle(w), Hp.TOL["fp32"], "many segments, one head")
    print(f"[f32 attention] many segments of one head: worst {worst:.2e}", flush=True)

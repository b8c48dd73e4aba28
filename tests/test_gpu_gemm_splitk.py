"""The bf16 GEMM forms with A K-contiguous, contracted in ranges: partial planes in the workspace, finished by one kernel."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


# (M, N, K, trans_b): one row; a ragged last tile row and column; ranges of unequal depth; 128- and 256-row tiles; few and
# many ranges; one tile
@pytest.mark.parametrize("M,N,K,tb", [(1, 512, 4096, 0), (300, 2056, 4128, 0), (513, 4104, 12320, 1), (129, 264, 3072, 1), (2048, 4096, 11008, 0),
                                      (256, 8192, 4096, 1), (77, 72, 4096, 0)])
@pytest.mark.parametrize("out_fp32,with_r", [(1, 0), (1, 1), (0, 0)])
def test_split_contraction_matches_fp64(M, N, K, tb, out_fp32, with_r):
    """fp32 sums of exact products: error within sqrt(K) 2^-24 of the largest sum of magnitudes, bf16 output 2^-8 more."""
    import torch
    import paper_2605_18750_amd as R
    from paper_2605_18750_amd import harness as Hn
    plan = R.rrfp_gemm_plan(M, N, K, 0, tb, R.STAGE_DTYPE_FP32 if out_fp32 else R.STAGE_DTYPE_BF16, have_scratch=True)
    print(f"[splitk] M{M} N{N} K{K} tb{tb} f32{out_fp32} r{with_r}: {plan}", flush=True)
    assert plan["split_k"] > 1
    g = torch.Generator().manual_seed(M + N + K)
    A, B = torch.randn((M, K), generator=g).bfloat16().cuda(), torch.randn((N, K) if tb else (K, N), generator=g).bfloat16().cuda()
    Rr = torch.randn((M, N), generator=g).cuda() if with_r else None
    ref = A.double() @ (B.double().t().contiguous() if tb else B.double())
    if with_r:
        ref = ref + Rr.double()
    nbytes = plan["split_k"] * M * N * 4
    outs = []
    for size in (nbytes, nbytes, nbytes - 256):          # the same call twice; a workspace one range too small
        ws = torch.full((nbytes + 256,), 0xFF, dtype=torch.uint8, device="cuda:0")       # NaN planes, and a guard behind them
        C = torch.full((M + 1, N), float("nan"), dtype=torch.float32 if out_fp32 else torch.bfloat16, device="cuda:0")
        R.rrfp_gemm(A, B, C, Rr, M, N, K, K, B.shape[1], N, N, 0, tb, 1, 0 if out_fp32 else 1, R.RRFP_GEMM_MFMA, workspace=ws, workspace_bytes=size)
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xFF).all()), "written past the workspace"
        assert bool(torch.isnan(C[M:]).all()), "rows past M were written"
        err = float((C[:M].double() - ref).abs().max() / ref.abs().max())
        assert err <= (2e-5 if out_fp32 else 1e-2), (size, err)
        outs.append(C[:M].clone())
    assert torch.equal(outs[0], outs[1]), "two calls differ"


# one row or column block; K of one step, one more, fewer steps than wavefronts, a ragged last step; M and N around the tile
@pytest.mark.parametrize("M,N,K", [(8, 8, 1), (8, 64, 32), (64, 72, 33), (72, 56, 200), (136, 64, 256), (56, 136, 257), (1536, 512, 777)])
def test_small_weight_gradient_matches_fp64(M, N, K):
    _small(M, N, K, 1, 0, 1, 0)


@pytest.mark.parametrize("M,N,K,tb", [(1, 8, 32, 0), (63, 64, 64, 1), (65, 72, 288, 0), (129, 512, 512, 1), (777, 1024, 512, 0), (200, 56, 1056, 1)])
@pytest.mark.parametrize("out_fp32,with_r", [(1, 0), (1, 1), (0, 0)])
def test_small_outputs_match_fp64(M, N, K, tb, out_fp32, with_r):
    _small(M, N, K, 0, tb, out_fp32, with_r)


# The two tile edges on both sides of the rule (32 while there are at most 512 such tiles on 256 CUs), ragged in every direction, K of a
# whole number of steps and of 1, 31 and 33 more where the form takes them; steps that do not divide by the wavefronts or the steps ahead
@pytest.mark.parametrize("M,N,K,ta,tb,tiles", [(512, 1024, 512, 0, 1, 512), (513, 1000, 544, 0, 1, 144), (545, 968, 288, 0, 0, 144), (32, 40, 1312, 0, 0, 2),
                                               (33, 24, 96, 0, 1, 2), (520, 1032, 257, 1, 0, 153), (40, 16, 1025, 1, 0, 2), (24, 72, 63, 1, 0, 2)])
def test_small_tile_edges_match_fp64(M, N, K, ta, tb, tiles):
    import paper_2605_18750_amd as R
    assert R.rrfp_gemm_plan(M, N, K, ta, tb, R.STAGE_DTYPE_FP32, have_scratch=True)["main_workgroups"] == tiles
    _small(M, N, K, ta, tb, 1, 0)


def _small(M, N, K, ta, tb, out_fp32, with_r):
    """Operands end in NaN rows that must not be read into a result; error bounds as above."""
    import torch
    import paper_2605_18750_amd as R
    plan = R.rrfp_gemm_plan(M, N, K, ta, tb, R.STAGE_DTYPE_FP32 if out_fp32 else R.STAGE_DTYPE_BF16, have_scratch=True)
    print(f"[small gemm] M{M} N{N} K{K} ta{ta} tb{tb} f32{out_fp32} r{with_r}: {plan}", flush=True)
    assert plan["kernel"] == 3
    g = torch.Generator().manual_seed(M + N + K)
    full = [torch.randn((r + 64, c), generator=g).bfloat16().cuda() for r, c in ((K, M) if ta else (M, K), (N, K) if tb else (K, N))]
    for t in full:
        t[-64:] = float("nan")
    A, B = full[0][:-64], full[1][:-64]
    Rr = torch.randn((M, N), generator=g).cuda() if with_r else None
    ref = (A.double().t().contiguous() if ta else A.double()) @ (B.double().t().contiguous() if tb else B.double())
    if with_r:
        ref = ref + Rr.double()
    ws = torch.zeros(256, dtype=torch.uint8, device="cuda:0")
    C = torch.full((M + 1, N), float("nan"), dtype=torch.float32 if out_fp32 else torch.bfloat16, device="cuda:0")
    R.rrfp_gemm(A, B, C, Rr, M, N, K, A.shape[1], B.shape[1], N, N, ta, tb, 1, 0 if out_fp32 else 1, R.RRFP_GEMM_MFMA, workspace=ws, workspace_bytes=256)
    torch.cuda.synchronize()
    assert bool(torch.isnan(C[M:]).all()), "rows past M were written"
    err = float((C[:M].double() - ref).abs().max() / ref.abs().max())
    assert err <= (2e-5 if out_fp32 else 1e-2), err


@pytest.mark.parametrize("mlp,bias,norm", [("swiglu", False, "rms"), ("swiglu", True, "rms"), ("gelu", True, "layer"), ("gelu", False, "rms")])
def test_stage_with_split_contractions_matches_oracle(mlp, bias, norm):
    """Every fused epilogue behind the planes: activations forward and backward, biases, residuals, half outputs and the scale
    of dO.  Hidden 2048 at 150 tokens and at one: all the products of F and B are split (150: two tile rows, the second ragged)."""
    import paper_2605_18750_amd as R
    from paper_2605_18750_amd import harness as Hn
    shape = SI.StageShape(f"splitk_{mlp}{bias}{norm}", 1, 2048, 16, 8, 128, 2048, 2, w_std=0.02, mlp_kind=mlp, bias=bias, norm_kind=norm)
    w = Hp.Workload(shape, [[0, 60, 150], [0, 1]])
    scratch = R.stage_scratch_bytes(Hn.make_config(shape, 150, 2, n_microbatches=2))
    F32, BF, n_up = R.STAGE_DTYPE_FP32, R.STAGE_DTYPE_BF16, 4096 if mlp == "swiglu" else 2048
    for T in (150, 1):
        for N, K, tb, out in ((4096, 2048, 0, BF), (2048, 2048, 0, F32), (n_up, 2048, 0, BF), (2048, 2048, 1, BF), (2048, n_up, 1, F32), (2048, 4096, 1, F32)):
            assert R.rrfp_gemm_plan(T, N, K, 0, tb, out, workspace_bytes=scratch)["split_k"] > 1, (T, N, K)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL["bf16"], "splitk stage")
    print(f"[splitk] stage {mlp} bias{bias} {norm}: worst {worst:.2e}", flush=True)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, order=SI.ready_order(w.M, 5), n_streams=3, keep_raw=True))


def test_bits_do_not_hang_on_the_limits_of_the_stage():
    """The same microbatches through stages made for more tokens and more segments: the same bits, ranges and planes of the
    products and partial rows of the norm backward included."""
    shape = SI.StageShape("splitk_limits", 1, 2048, 16, 8, 128, 1024, 2, w_std=0.02)
    w = Hp.Workload(shape, [[0, 60, 150], [0, 1]])
    print("[splitk] limits of the stage", flush=True)
    first = Hp.run_gpu(w, keep_raw=True)
    for more in (dict(max_tokens=4096), dict(max_segments=40)):
        Hp.assert_bit_identical(first, Hp.run_gpu(w, keep_raw=True, **more))

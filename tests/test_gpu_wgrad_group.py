"""The weight gradients of all layers of a task in one launch: each way the list can be cut, against fp64 and the oracle."""
import numpy as np
import pytest

import stage_inputs as SI
from tests import helpers as Hp

pytestmark = pytest.mark.gpu


def _products(layers, hidden, nq, nkv, d, ffn):
    """(M, N) of the weight gradients in the order a SwiGLU stage lists them."""
    return [(hidden, (nq + 2 * nkv) * d), (nq * d, hidden), (hidden, 2 * ffn), (ffn, hidden)] * layers


# (layers, hidden, q heads, kv heads, head_dim, ffn, dtype, tokens, cut)
CASES = [
    (9, 64, 1, 1, 64, 64, "bf16", 33, dict(full=56, tail=0, ranges=0)),           # two lists; 64 x 64 tiles; K one past a step
    (2, 320, 5, 1, 64, 448, "bf16", 1500, dict(full=330, tail=0, ranges=0)),      # 64 x 64 tiles, two rounds, K of many steps
    (2, 1024, 8, 8, 128, 2816, "bf16", 520, dict(full=392, tail=0, ranges=1)),    # 256-row tiles, none cut
    (1, 832, 13, 1, 64, 1600, "bf16", 2100, dict(full=0, tail=112, ranges=2)),    # every tile cut, ragged edges, a short last range
    (2, 1088, 17, 17, 64, 2880, "bf16", 1100, dict(full=512, tail=18, ranges=4)), # whole rounds and a cut rest, ragged edges, a short last range
    (9, 32, 2, 1, 16, 48, "fp32", 65, None),        # two lists of 32 x 32 tiles
    (2, 30, 1, 1, 16, 44, "fp32", 17, None),        # rows that are not whole float4s
    (1, 516, 4, 2, 128, 900, "fp32", 100, None),    # 64 x 64 tiles, ragged
]


@pytest.mark.parametrize("layers,hidden,nq,nkv,d,ffn,dtype,tokens,cut", CASES)
def test_grouped_weight_gradients(layers, hidden, nq, nkv, d, ffn, dtype, tokens, cut):
    """Rounding of the storage types as in the other parity tests; a tile, range or product in the wrong place is an error of order one."""
    import paper_2605_18750_amd as R
    if cut:
        assert R.rrfp_wgrad_group_plan(_products(min(layers, 8), hidden, nq, nkv, d, ffn), tokens) == cut
    shape = SI.StageShape(f"wgroup{layers}.{hidden}.{ffn}", layers, hidden, nq, nkv, d, ffn, 2, dtype=dtype, x_std=1.0, dy_std=1.0,
                          w_std=0.5 / np.sqrt(hidden))
    w = Hp.Workload(shape, [[0, tokens // 3, tokens]])
    print(f"[wgrad group] {shape.name} {dtype} {tokens} tokens", flush=True)
    got = Hp.run_gpu(w, keep_raw=True)
    worst = Hp.compare(got, Hp.run_oracle(w), Hp.TOL[dtype], shape.name)
    Hp.assert_bit_identical(got, Hp.run_gpu(w, keep_raw=True))
    print(f"[wgrad group] {shape.name}: worst {worst:.2e}", flush=True)


# (products, K, workspace in planes of 256 KB, cut): every tile cut; a cut rest within one product and over three; less workspace
# than the cut asks for; 64 x 64 tiles; one product whose last step has one row of K
LISTS = [
    (_products(1, 832, 13, 1, 64, 1600), 2100, None, dict(full=0, tail=112, ranges=2)),
    (_products(2, 1088, 17, 17, 64, 2880), 1100, None, dict(full=512, tail=18, ranges=4)),
    ([(2376, 3176), (8, 16), (2384, 1368), (2080, 2656), (112, 888), (328, 3160)], 1473, None, dict(full=256, tail=64, ranges=3)),
    (_products(2, 1088, 17, 17, 64, 2880), 1100, 18 * 3, dict(full=512, tail=18, ranges=3)),
    (_products(1, 72, 1, 1, 64, 136), 65, None, dict(full=24, tail=0, ranges=0)),
    ([(1032, 2056)], 4129, None, dict(full=0, tail=45, ranges=5)),
    # 128 x 128 tiles, ragged: less than a step, one and a bit, five and a bit, the most of the rule for one round; two rounds
    (_products(2, 504, 8, 2, 64, 1400), 31, None, dict(full=344, tail=0, ranges=-1)),
    (_products(2, 504, 8, 2, 64, 1400), 33, None, dict(full=344, tail=0, ranges=-1)),
    (_products(2, 504, 8, 2, 64, 1400), 165, None, dict(full=344, tail=0, ranges=-1)),
    (_products(2, 504, 8, 2, 64, 1400), 320, None, dict(full=344, tail=0, ranges=-1)),
    (_products(2, 504, 8, 2, 64, 1400), 321, None, dict(full=88, tail=0, ranges=1)),
    (_products(2, 504, 8, 2, 64, 1400), 100, None, dict(full=344, tail=0, ranges=-1)),
    ([(2376, 3176), (3000, 2056), (1032, 6152)], 64, None, dict(full=1324, tail=0, ranges=-1)),
    ([(2376, 3176), (3000, 2056), (1032, 6152)], 65, None, dict(full=363, tail=0, ranges=1)),
    ([(2376, 3176), (3000, 2056), (1032, 6152)], 97, None, dict(full=363, tail=0, ranges=1)),
    # one 256-row tile per workgroup, K of one group of four steps
    (_products(4, 512, 8, 2, 64, 1536), 97, None, dict(full=184, tail=0, ranges=1)),
    # workgroups that walk two tiles, of 1, 5, 9 and 12 steps (a workgroup takes them in groups of four)
    ([(2376, 3176), (4096, 2056), (1032, 6152)], 31, None, dict(full=399, tail=0, ranges=1)),
    ([(2376, 3176), (4096, 2056), (1032, 6152)], 131, None, dict(full=399, tail=0, ranges=1)),
    ([(2376, 3176), (4096, 2056), (1032, 6152)], 257, None, dict(full=399, tail=0, ranges=1)),
    ([(2376, 3176), (4096, 2056), (1032, 6152)], 384, None, dict(full=399, tail=0, ranges=1)),
    # workgroups that walk two and three tiles of a single group: 1, 3 and 4 steps
    ([(2376, 3176), (4096, 2056), (1032, 6152), (2000, 3384), (3176, 2000)], 32, None, dict(full=615, tail=0, ranges=1)),
    ([(2376, 3176), (4096, 2056), (1032, 6152), (2000, 3384), (3176, 2000)], 65, None, dict(full=615, tail=0, ranges=1)),
    ([(2376, 3176), (4096, 2056), (1032, 6152), (2000, 3384), (3176, 2000)], 128, None, dict(full=615, tail=0, ranges=1)),
    # the most products a launch takes, of unequal tile counts, in each tile size
    ([(72, 136), (136, 72)] * 16, 97, None, dict(full=192, tail=0, ranges=0)),
    ([(136, 264), (264, 8)] * 16, 300, None, dict(full=144, tail=0, ranges=-1)),
    ([(520, 776), (8, 264)] * 16, 97, None, dict(full=224, tail=0, ranges=1)),
]


@pytest.mark.parametrize("products,K,planes,cut", LISTS)
def test_group_matches_fp64(products, K, planes, cut):
    """fp32 sums of exact products: error within sqrt(K) 2^-24 of the largest sum of magnitudes.  Operands end in NaN rows that must not
    be read into a result; nothing is written past an output or the workspace."""
    import torch
    import paper_2605_18750_amd as R
    nbytes = (16 * 256 if planes is None else planes) << 18
    print(f"[wgrad group] {len(products)} products K{K} workspace {nbytes >> 18} planes: {cut}", flush=True)
    assert R.rrfp_wgrad_group_plan(products, K, workspace_bytes=nbytes) == cut
    g = torch.Generator().manual_seed(K + len(products))

    def operand(width):
        t = torch.full((K + 64, width), float("nan"))
        t[:K] = torch.randn((K, width), generator=g)
        return t.bfloat16().cuda()

    A, B = [operand(m) for m, _ in products], [operand(n) for _, n in products]
    need = cut["ranges"] * cut["tail"] << 18 if cut["ranges"] > 1 else 256
    ws = torch.full((nbytes + 256,), 0xFF, dtype=torch.uint8, device="cuda:0")      # NaN planes
    outs = []
    for _ in range(2):
        C = [torch.full((m + 1, n), float("nan"), device="cuda:0") for m, n in products]
        R.rrfp_wgrad_group(A, B, C, products, K, R.STAGE_DTYPE_BF16, workspace=ws, workspace_bytes=nbytes)
        torch.cuda.synchronize()
        assert bool((ws[need:] == 0xFF).all()), "written past the planes"
        for (m, n), a, b, c in zip(products, A, B, C):
            assert bool(torch.isnan(c[m:]).all()), "rows past M were written"
            ref = a[:K].double().t().contiguous() @ b[:K].double()
            err = float((c[:m].double() - ref).abs().max() / ref.abs().max())
            assert err <= 2e-5, (m, n, err)
        outs.append([c[:m].clone() for (m, _), c in zip(products, C)])
    assert all(torch.equal(x, y) for x, y in zip(*outs)), "two calls differ"

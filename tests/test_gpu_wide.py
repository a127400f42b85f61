"""The wide contraction kernels (256x256 and 256x192 tiles of four waves, the
library's own choice for large outputs) and the grouped launch of the
backward's weight gradients, at the sizes where they can go wrong: one, two
and three k-steps (fewer than the five LDS slots hold), k-rows past the end
of an outer-contiguous pair, ragged last tiles, every operand layout; the
128x128 tile from the eight k-steps on at which it is chosen, with split
partials; and layers whose group is split, spread over several
rounds, or takes the input gradient in."""
import pytest
import torch

from paper_2007_00072_amd import lib
from paper_2007_00072_amd.inputs import make_tensor
from test_gpu_layer import check_encoder, run_encoder, small
from test_gpu_plan import _launches

pytestmark = pytest.mark.gpu
DT = {"f16": (lib.DM_F16, torch.float16, 2.0 ** -11), "bf16": (lib.DM_BF16, torch.bfloat16, 2.0 ** -8)}


def contraction(dtype, a_trans, b_trans, M, N, K, want, bias=False, out_f32=False, ws_parts=0):
    """The library's own choice for these sizes: kernel and split factor
    `want`, and the result.  ws_parts: scratch for that many partials."""
    code, td, _ = DT[dtype]
    A = make_tensor((K, M) if a_trans else (M, K), dtype, 3).cuda()
    B = make_tensor((N, K) if b_trans else (K, N), dtype, 4).cuda()
    bv = make_tensor((N,), dtype, 5).cuda() if bias else None
    # (a band of rows after the output that no store may reach)
    C = torch.full((M + 8, N), 7.0, dtype=torch.float32 if out_f32 else td, device="cuda")
    ws = torch.full((ws_parts * M * N + 8,), 7.0, dtype=torch.float32, device="cuda")
    lib.plan_log(True)
    lib.contract(code, 1, M, N, K, 1.0, A, int(a_trans), 0, B, int(b_trans), 0, bv, C, int(out_f32), 0, -1, 0,
                 ws if ws_parts else None, ws_parts * M * N * 4)
    torch.cuda.synchronize()
    ran = [(r.tile_cfg, r.splits) for r in lib.plan_log_read()]
    lib.plan_log(False)
    assert ran == [want], (ran, want)
    assert (C[M:] == 7.0).all() and (ws[ws_parts * M * N:] == 7.0).all()
    a = (A.t() if a_trans else A).float()
    b = (B.t() if b_trans else B).float()
    ref = a.double() @ b.double().contiguous()
    if bias:
        ref = ref + bv.double()
    # fp32 accumulation of K products of magnitude ~1, one rounding to the
    # output type: |err| <= u |ref| + K 2^-23 (rms of a product's sum sqrt K)
    u = 2.0 ** -23 if out_f32 else DT[dtype][2]
    bound = u * ref.abs() + (K ** 0.5) * 2.0 ** -20 + K * 2.0 ** -23
    worst = ((C[:M].double() - ref).abs() / bound).max().item()
    assert worst <= 1.0, worst


# 15 x 14 tiles of 256: 3/4 of the CUs have one
@pytest.mark.parametrize("a_trans,b_trans", [(False, True), (False, False), (True, True), (True, False)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [64, 128, 192, 320])
def test_wide_contract(dtype, a_trans, b_trans, K):
    contraction(dtype, a_trans, b_trans, 3720, 3464, K, (26, 1), bias=True)


@pytest.mark.parametrize("K", [8, 56, 72, 200, 328])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_wide_contract_ragged_k(dtype, K):
    # both operands outer-contiguous: the last step's missing k-rows are zeros
    contraction(dtype, True, False, 3720, 3464, K, (26, 1), out_f32=dtype == "f16")


@pytest.mark.parametrize("a_trans", [False, True])
def test_wide_contract_192(a_trans):
    # 16 x 15 tiles of 256 x 192 fit one round where 256 x 256 leaves CUs idle
    contraction("f16", a_trans, True, 4088, 2880, 256, (27, 1), bias=True)


# the 128x128 tile: 3 x 3 tiles with ragged last ones
@pytest.mark.parametrize("a_trans,b_trans", [(False, True), (False, False), (True, True), (True, False)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [512, 576, 640])
def test_mid_contract(dtype, a_trans, b_trans, K):
    contraction(dtype, a_trans, b_trans, 264, 328, K, (28, 1), bias=True)
    contraction(dtype, a_trans, b_trans, 8, 136, K, (28, 1), out_f32=True)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [520, 568, 584])
def test_mid_contract_ragged_k(dtype, K):
    contraction(dtype, True, False, 264, 328, K, (28, 1), out_f32=dtype == "f16")


# split sums: pieces of eight steps, of nine with a last one of six, and (both
# operands outer-contiguous) a last one that ends inside a step
@pytest.mark.parametrize("a_trans,b_trans,K", [(False, True, 2048), (False, False, 2112), (True, True, 2112),
                                               (True, False, 2048), (True, False, 2056)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_mid_contract_split(dtype, a_trans, b_trans, K):
    contraction(dtype, a_trans, b_trans, 264, 328, K, (28, 4), bias=True, ws_parts=4)
    contraction(dtype, a_trans, b_trans, 264, 328, K, (28, 3), out_f32=True, ws_parts=3)


def grads_label(labels):
    return [lab for lab in labels if lab.startswith("B4+7+12")]


@pytest.mark.parametrize("name,shape,want", [
    # 192 weight-gradient tiles, k of 512 tokens, input gradient on its own
    ("bert_large_f16", dict(B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=4096), "B4+7+12+19 weight_grads"),
    # ragged tokens: 1000 = 15 steps of 64 and 40
    ("bert_base_bf16", dict(B=5, J=200, K=200, H=16, P=64, W=64, I=1024, F=4096), None),
])
def test_layer_with_grouped_weight_gradients(name, shape, want):
    wl = small(name, **shape)
    _, labels = _launches(wl)
    assert grads_label(labels) and "B4 linear2_dw" not in labels and "B12+19 out_dw+qkv_dw" not in labels, labels
    if want:
        assert want in labels
    check_encoder(wl, layer=1)


@pytest.mark.parametrize("name,shape", [
    # 192 tiles, unsplit
    ("bert_large_f16", dict(B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=4096)),
    # BERT-base widths, 12288 tokens: 108 tiles, so the token sums are split
    # and the grid has more than one round
    ("bert_base_bf16", dict(B=96, J=128, K=128, H=12, P=64, W=64, I=768, F=3072)),
    # the same split over 5000 tokens, no multiple of 64
    ("bert_base_bf16", dict(B=25, J=200, K=200, H=12, P=64, W=64, I=768, F=3072)),
])
def test_group_and_separate_launches_agree(name, shape):
    # a plan entry that names one of the contractions separates the group
    wl = small(name, **shape)
    T, I, F = shape["B"] * shape["J"], shape["I"], shape["F"]
    L0, _, _, _, y0, dx0 = run_encoder(wl)
    g0 = {n: t.clone() for n, t in L0.grads.items()}
    recs, labels = _launches(wl)
    assert grads_label(labels), labels
    dw1 = next(r for r in recs if (r.M, r.N, r.K) == (F, I, T) and not r.a_kcontig)
    assert (dw1.splits > 1) == (T > 4096)
    plan = lib.Plan([lib.ContractChoice(*dw1.key(), 15, 1)], 0)
    _, labels = _launches(wl, plan)
    assert not grads_label(labels) and "B7 linear1_dw" in labels
    L1, _, _, _, y1, dx1 = run_encoder(wl, plan=plan)
    assert torch.equal(y0, y1)
    # (the input gradient's sums of 3 I products in another order, one rounding to the storage type)
    assert (dx0.float() - dx1.float()).norm() <= 2.0 ** -8 * dx1.float().norm()
    for n, t in L1.grads.items():
        # T products per sum, fp32 accumulation in another order
        assert (g0[n] - t).abs().max().item() <= T ** 0.5 * 2.0 ** -20 * max(t.abs().max().item(), 1e-3), n


@pytest.mark.parametrize("layout", ["ibj", "bji"])
def test_mha_on_wide_tiles(layout):
    # the paper's [i][b][j] order: outputs contiguous along the tokens run as
    # their transposes (bias along m, stacked weights as the outer-contiguous
    # first operand), the Q/K/V weight gradient with its row sums on 128x128
    # tiles; 520 tokens: ragged last tiles
    from paper_2007_00072_amd.inputs import WORKLOADS, Shape
    from test_gpu_layer import check_mha
    wl = WORKLOADS["mha_large_f16"].with_(shape=Shape(B=5, J=104, K=104, H=8, P=64, W=64, I=512), layout=layout, p_attn=0.1)
    check_mha(wl, self_attention=True)
    check_mha(wl, self_attention=2)


@pytest.mark.parametrize("shape,grouped", [
    # 15 wide heads, 512 tokens: no more than a tie is expected, separate launches
    (dict(B=4, J=128, K=128, H=15, P=64, W=64, I=960, F=3840), False),
    # the same width on 400 (ragged) and 2048 tokens: one grid
    (dict(B=2, J=200, K=200, H=15, P=64, W=64, I=960, F=3840), True),
    (dict(B=16, J=128, K=128, H=15, P=64, W=64, I=960, F=3840), True),
])
def test_group_only_where_it_pays(shape, grouped):
    _, labels = _launches(small("bert_base_bf16", **shape))
    assert bool(grads_label(labels)) == grouped, labels

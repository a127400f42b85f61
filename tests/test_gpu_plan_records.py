"""Launch records given back as a plan: the same kernels, split factors and
launch grouping run again, with the same results bit for bit."""
import pytest
import torch

from paper_2007_00072_amd import lib
from paper_2007_00072_amd.inputs import WORKLOADS, Shape, make_activation, make_params
from test_gpu_layer import check_encoder, run_encoder, small
from test_gpu_plan import _launches

pytestmark = pytest.mark.gpu


def choices(recs):
    return [(r.key(), r.label, r.tile_cfg, r.splits) for r in recs]


@pytest.mark.parametrize("name,shape", [
    # weight gradients in one grid (with the input gradient), split partials summed by the LayerNorm kernels
    ("bert_large_f16", dict(B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=4096)),
    # split weight gradients in one grid, the input gradient on its own or not
    ("bert_base_bf16", dict(B=32, J=128, K=128, H=12, P=64, W=64, I=768, F=3072)),
    # ragged tokens, separate launches
    ("bert_base_bf16", dict(B=5, J=200, K=200, H=12, P=64, W=64, I=768, F=3072)),
    # split pieces of two 64-wide steps
    ("bert_large_f16", dict(B=1, J=72, K=72, H=12, P=64, W=64, I=768, F=1024)),
    # the paired launch (widths that give every contraction a key of its own)
    ("bert_large_f16", dict(B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=1152)),
])
def test_encoder_records_as_a_plan(name, shape):
    wl = small(name, **shape)
    recs, labels = _launches(wl)
    L0, _, _, _, y0, dx0 = run_encoder(wl)
    plan = lib.Plan(recs, 0)
    recs2, labels2 = _launches(wl, plan)
    assert labels2 == labels and choices(recs2) == choices(recs)
    L1, _, _, _, y1, dx1 = run_encoder(wl, plan=plan)
    assert torch.equal(y0, y1) and torch.equal(dx0, dx1)
    for n, g in L0.grads.items():
        assert torch.equal(g, L1.grads[n]), n


@pytest.mark.parametrize("layout", ["ibj", "bji"])
def test_attention_records_as_a_plan(layout):
    # (the [i][b][j] order runs outputs contiguous along the tokens as their transposes)
    from paper_2007_00072_amd.runner import MultiHeadAttention, desc_for
    wl = WORKLOADS["mha_large_f16"].with_(shape=Shape(B=5, J=104, K=104, H=8, P=64, W=64, I=512), layout=layout)
    x, dy = make_activation(wl, 0).cuda(), make_activation(wl, 1).cuda()

    def run(plan):
        M = MultiHeadAttention(desc_for(wl, self_attention=True, plan=plan), make_params(wl), "cuda")
        lib.plan_log(True)
        y = M.forward(x)
        dx = M.backward(x, dy)[0]
        torch.cuda.synchronize()
        recs = lib.plan_log_read()
        lib.plan_log(False)
        return recs, y, dx, {n: g for n, g in M.grads.items() if g is not None}

    recs, y0, dx0, g0 = run(None)
    assert any(r.tile_cfg >= 26 for r in recs)
    recs2, y1, dx1, g1 = run(lib.Plan(recs, 0))
    assert choices(recs2) == choices(recs)
    assert torch.equal(y0, y1) and torch.equal(dx0, dx1)
    for n in g0:
        assert torch.equal(g0[n], g1[n]), n


def test_entry_for_the_input_gradient_keeps_the_weight_gradients_together():
    wl = small("bert_large_f16", B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=4096)
    s = wl.shape
    key = (s.B * s.J, s.I, 3 * s.I, 1, lib.DM_F16, 1, 0)
    _, labels = _launches(wl, lib.Plan([lib.ContractChoice(*key, 15, 1)], 0))
    assert "B18 qkv_dx" in labels and "B4+7+12+19 weight_grads" in labels, labels


@pytest.mark.parametrize("name", ["bert_large_f16", "bert_base_bf16"])
@pytest.mark.parametrize("cfg,splits", [(26, 1), (27, 1), (28, 1), (26, 2), (27, 3), (28, 3)])
def test_every_contraction_on_a_named_wide_kernel(name, cfg, splits):
    # k of 256 to 520 (four to nine 64-wide steps, the last of 8 k-rows),
    # ragged last tiles; what the kernel does not take (the input bias sums,
    # a ragged k next to an operand contiguous along it, a 192-wide operand
    # contiguous along its rows) falls back
    wl = small(name, B=5, J=104, K=104, H=4, P=64, W=64, I=256, F=512).with_(p_attn=0.1)
    recs, _ = _launches(wl)
    plan = lib.Plan([lib.ContractChoice(*k, cfg, splits) for k in {r.key() for r in recs}], 0, {"dO_transposed": 0})
    recs2, labels = _launches(wl, plan)
    ran = [r.tile_cfg for r in recs2]
    assert ran.count(cfg) >= (4 if cfg == 27 else 9), ran
    # (Linear 2's partials, summed by the LayerNorm kernel, go down to two k-steps a piece)
    assert splits == 1 or sum(r.splits == splits for r in recs2) >= 1, [(r.label, r.splits) for r in recs2]
    check_encoder(wl, layer=1, plan=plan)

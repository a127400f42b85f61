"""Attention at key lengths that are no multiple of the kernels' tiles: the
forward's padded score tile (32 keys), the key-block backward's last block
(128 or 256 keys), rows longer than 1024 keys, causal masks that leave out
whole key tiles and query steps, and one key tile in all."""
import pytest
import torch

from paper_2007_00072_amd import lib
from paper_2007_00072_amd.inputs import WORKLOADS, Shape
from test_gpu_layer import check_encoder, check_mha, run_encoder, small
from test_gpu_plan import _launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["bert_large_f16", "bert_base_bf16"])
@pytest.mark.parametrize("J,causal", [(8, False), (40, False), (136, False), (200, True), (264, False), (392, True)])
def test_encoder_key_lengths(name, J, causal):
    wl = small(name, B=2, J=J, K=J, H=4, P=64, W=64, I=256, F=512).with_(p_attn=0.1)
    _, labels = _launches(wl, None)
    assert "F2-4 qkt_softmax_gamma" in labels and "B13-17 score_bwd_keys" in labels, labels
    check_encoder(wl, layer=1, causal=causal)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("J,K", [(72, 24), (24, 136), (40, 776), (16, 1032), (32, 1096)])
def test_mha_key_lengths(dtype, J, K):
    # cross attention; 776 to 1096 keys: tiles above 64 KB of LDS, rows of
    # two and four 8-element vectors per lane
    wl = WORKLOADS["mha_large_f16"].with_(shape=Shape(B=2, J=J, K=K, H=2, P=64, W=64, I=128), dtype=dtype, layout="bji",
                                          p_attn=0.1)
    check_mha(wl, self_attention=False)


@pytest.mark.parametrize("B,H,J,causal", [
    (24, 8, 248, False),  # 192 blocks of 256 keys, one a head, padded
    (18, 8, 392, True),   # 288 blocks, two a head, the second padded, steps before it left out
    (17, 8, 392, True),   # the same on 128-key blocks
])
def test_key_padding_leaves_neighbours_alone(B, H, J, causal):
    # against the row form of the same backward
    wl = small("bert_large_f16", B=B, J=J, K=J, H=H, P=64, W=64, I=64 * H, F=512).with_(p_attn=0.1)
    L0, _, _, _, y0, dx0 = run_encoder(wl, causal=causal)
    L1, _, _, _, y1, dx1 = run_encoder(wl, causal=causal, plan=lib.Plan((), attn_path=1))
    assert lib.attn_backward_form(L0.desc) and not lib.attn_backward_form(L1.desc)
    # the two forms round d(alpha) and P's products at different places
    assert (dx0.float() - dx1.float()).norm() <= 3e-3 * dx1.float().norm()
    for n in ("wq", "wk", "wv"):
        assert (L0.grads[n] - L1.grads[n]).norm() <= 3e-3 * L1.grads[n].norm(), n


@pytest.mark.parametrize("name", ["bert_large_f16", "bert_base_bf16"])
@pytest.mark.parametrize("J", [72, 136])
def test_causal_on_separate_launches(name, J):
    # QK^T, the masked softmax and Gamma one by one (and their backward), which
    # a plan may ask for at any length and longer rows run by themselves
    wl = small(name, B=2, J=J, K=J, H=4, P=64, W=64, I=256, F=512).with_(p_attn=0.1)
    plan = lib.Plan((), attn_path=1)
    _, labels = _launches(wl, plan)
    assert {"F2 qkt", "F3 softmax", "F4 gamma", "B13 gamma_dx1", "B15 softmax_bwd"} <= set(labels), labels
    check_encoder(wl, layer=1, causal=True, plan=plan)


@pytest.mark.parametrize("name,causal", [("bert_large_f16", True), ("bert_base_bf16", True), ("bert_base_bf16", False)])
def test_rows_beyond_the_chip(name, causal):
    # 2056 keys: separate forward launches, the key-block backward on what
    # they wrote (under the mask it leaves out blocks where P has to be zero)
    wl = small(name, B=1, J=2056, K=2056, H=2, P=64, W=64, I=128, F=256).with_(p_attn=0.1)
    _, labels = _launches(wl, None)
    assert {"F2 qkt", "F3 softmax", "F4 gamma", "B13-17 score_bwd_keys"} <= set(labels), labels
    check_encoder(wl, layer=1, causal=causal)

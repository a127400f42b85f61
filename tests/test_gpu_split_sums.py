"""Split contractions whose partials the next LayerNorm kernel sums (output
projection, Linear 2, Linear 1 dX): every split count up to eight, row counts
below and off the kernels' tiles, widths of the column-split backward (320 to
1024 columns), of the row form (the partials are then summed by themselves)
and of several vectors per lane, against the oracle."""
import pytest

from test_gpu_layer import check_encoder, small
from test_gpu_plan import _launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["bert_large_f16", "bert_base_bf16"])
@pytest.mark.parametrize("shape,bwd", [
    (dict(B=1, J=8, H=5, I=320, F=512), True),     # five k-steps in two pieces
    (dict(B=1, J=72, H=12, I=768, F=1032), True),  # ragged k, up to eight pieces
    (dict(B=2, J=40, H=4, I=256, F=1024), False),  # row form of the LayerNorm backward
    (dict(B=3, J=200, H=16, I=1024, F=520), True),  # four pieces of 256; 520 in 320 + 200
    (dict(B=1, J=136, H=17, I=1088, F=512), False),  # rows of three vectors per lane
])
def test_encoder_split_sums(name, shape, bwd):
    wl = small(name, K=shape["J"], P=64, W=64, **shape).with_(p_attn=0.1, bias_std=0.05, random_ln=True)
    recs, _ = _launches(wl)
    ran = {r.label.decode(): r.splits for r in recs}
    for lab in ("F5 out", "F9 linear2") + (("B6 linear1_dx",) if bwd else ()):
        assert ran[lab] > 1, (lab, ran)
    check_encoder(wl, layer=2)

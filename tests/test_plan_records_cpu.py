"""plan_create takes every configuration that a launch record of a 16-bit
contraction can name, and refuses the others (host code, no GPU)."""
import pytest


@pytest.mark.parametrize("M,N,K,wide", [
    (4096, 3072, 1024, True),   # 256x256 and 256x192 tiles alone
    (64, 1024, 512, True),      # 128x128 tiles from k = 512 up
    (512, 512, 8, True),        # a weight gradient of the grouped launch, 8 tokens
    (64, 64, 1024, True),       # the same of a 64-wide layer, split along its tokens
    (64, 64, 64, False),        # no launch runs these on the wide kernels
    (128, 128, 504, False),
    (50176, 128, 128, True),    # 196 tiles of 256x256, half of each outside the output
])
@pytest.mark.parametrize("cfg", [-2, -1, 0, 25, 26, 27, 28, 29])
def test_plan_entry_range(M, N, K, wide, cfg):
    from paper_2007_00072_amd import lib
    entry = lib.ContractChoice(M, N, K, 1, lib.DM_F16, 1, 1, cfg, 1)
    assert lib.plan_cfg_ok(entry.key(), cfg) == (0 <= cfg <= (28 if wide else 25))
    if 0 <= cfg <= (28 if wide else 25):
        assert lib.Plan([entry], 0).handle
    else:
        with pytest.raises(lib.DmError):
            lib.Plan([entry], 0)

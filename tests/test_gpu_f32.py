"""The float32 contraction kernel at the edges of its 32x32 tiles and 64-wide
k-steps: sizes that are no multiple of 4 (pieces that are not 16-byte
aligned or end inside a row), one and several steps, batches."""
import pytest
import torch

from paper_2007_00072_amd import lib
from paper_2007_00072_amd.inputs import make_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("batch,M,N,K", [(1, 1, 1, 1), (2, 33, 31, 65), (1, 32, 64, 64), (3, 17, 70, 130), (1, 96, 40, 63)])
def test_f32_contract_edges(a_trans, b_trans, batch, M, N, K):
    A = make_tensor((batch, K, M) if a_trans else (batch, M, K), "f32", 21).cuda()
    B = make_tensor((batch, N, K) if b_trans else (batch, K, N), "f32", 22).cuda()
    bias = make_tensor((N,), "f32", 23).cuda()
    C = torch.full((batch * M * N + 8,), 7.0, dtype=torch.float32, device="cuda")
    lib.contract(lib.DM_F32, batch, M, N, K, 0.5, A, a_trans, M * K, B, b_trans, N * K, bias, C, 0, M * N)
    torch.cuda.synchronize()
    a = (A.transpose(1, 2) if a_trans else A).double().contiguous()
    b = (B.transpose(1, 2) if b_trans else B).double().contiguous()
    ref = 0.5 * torch.matmul(a, b) + bias.double()
    assert (C[batch * M * N:] == 7.0).all()
    # K fp32 products of magnitude ~1 added in fp32: error <= K u times the sum of magnitudes
    bound = 2.0 ** -23 * (K * 0.5 * torch.matmul(a.abs(), b.abs()) + ref.abs() + 1)
    assert ((C[:batch * M * N].view(batch, M, N).double() - ref).abs() <= bound).all()


def test_f32_contract_many_tiles():
    # 131070 x 129 tiles: 2^24 and more blocks of 256 threads, which one row of
    # a grid does not hold; sampled rows against float64
    M, N, K = 131070 * 32, 129 * 32, 4
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 70 GB")
    A, B = make_tensor((M, K), "f32", 21).cuda(), make_tensor((N, K), "f32", 22).cuda()
    C = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    lib.contract(lib.DM_F32, 1, M, N, K, 1.0, A, 0, 0, B, 1, 0, None, C, 1, 0)
    torch.cuda.synchronize()
    for r in (0, 31, 1 << 20, M - 100, M - 33, M - 1):
        ref = B.double() @ A[r].double()
        bound = 2.0 ** -22 * (B.double().abs() @ A[r].double().abs())
        assert ((C[r].double() - ref).abs() <= bound).all(), r

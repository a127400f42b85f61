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

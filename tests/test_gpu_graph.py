"""The encoder-layer step inside a HIP graph: the library issues no
allocation, copy, memset or synchronisation inside a step, so a captured
forward + backward replays the same kernels on the same buffers.  Every
replay, with eager steps and host synchronisations between replays, must
write exactly what an eager step writes (all kernels are deterministic)."""
import pytest
import torch

from paper_2007_00072_amd.inputs import make_activation, make_params
from paper_2007_00072_amd.runner import EncoderLayer, desc_for
from test_gpu_layer import DEV, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,shape", [
    ("bert_large_f16", dict(B=2, J=128, K=128, H=4, P=64, W=64, I=256, F=1024)),
    ("bert_base_bf16", dict(B=2, J=128, K=128, H=4, P=64, W=64, I=256, F=1024)),
    # score tiles above 64 KB of LDS (asked for at each launch), split sums
    ("bert_base_bf16", dict(B=1, J=1096, K=1096, H=4, P=64, W=64, I=256, F=1024)),
    # the grouped weight gradients
    ("bert_large_f16", dict(B=4, J=128, K=128, H=16, P=64, W=64, I=1024, F=4096)),
])
def test_encoder_step_graph_replays_match_eager(name, shape):
    wl = small(name, **shape)
    L = EncoderLayer(desc_for(wl, 1), make_params(wl, layer=1), DEV)
    x = make_activation(wl, 0).to(DEV)
    dy = make_activation(wl, 1).to(DEV)
    y = torch.empty_like(x)
    dx = torch.empty_like(x)

    def step():
        L.forward(x, y)
        L.backward(x, dy, dx)

    step()
    torch.cuda.synchronize()
    ref = (y.clone(), dx.clone(), {n: t.clone() for n, t in L.grads.items()})
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for rep in range(3):
        y.zero_()
        dx.zero_()
        for t in L.grads.values():
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref[0]), rep
        assert torch.equal(dx, ref[1]), rep
        for n, t in L.grads.items():
            assert torch.equal(t, ref[2][n]), (rep, n)
        step()   # eager work between replays
        torch.cuda.synchronize()

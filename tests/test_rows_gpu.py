"""The fp32-product kernels (channel layout) at the edges of their tiles: 16
tokens a wave and tile, four waves a unit, units of 64 to 512 tokens chosen by
the batch's size.  Forward (fp32) and backward (both dtypes) against the fp64
oracles, with the tolerances of test_parity_gpu.py and test_backward_gpu.py.
"""
import pytest
import torch

from paper_2606_07317_amd import inputs
from tests.test_backward_gpu import NAMES, TOL, close_scaled, run_backward
from tests.test_parity_gpu import close, say, small

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def G():
    from paper_2606_07317_amd import gbla
    gbla.load_library()
    return gbla


# lengths about the tile (16), the wave's quarter and the unit (64, 128, 256,
# 512), and what a conv window of three earlier tokens sees across each
EDGES = [2, 3, 4, 15, 16, 17, 63, 64, 65, 66, 67, 128, 131, 255, 257, 511, 512, 515]
DIMS = [(32, inputs.F32, 4), (32, inputs.BF16, 3), (64, inputs.F32, 2), (64, inputs.BF16, 4),
        (128, inputs.F32, 4), (128, inputs.BF16, 4)]


def _case(d, dtype, width, seed, **kw):
    return small("ragged64_d128", head_dim=d, dtype=dtype, conv_width=width, seed=seed, **kw)


# heads = 1: units of 64 tokens; heads = 24: units of 512 (fp32 forward: 128)
@pytest.mark.parametrize("heads", [1, 24])
@pytest.mark.parametrize("d,dtype,width", DIMS)
def test_backward_edges(G, dev, d, dtype, width, heads):
    from oracle import gbla_backward
    say("backward edges", d, dtype, width, heads)
    inp = inputs.make_inputs(_case(d, dtype, width, 51, heads=heads), lengths=EDGES)
    dy = inputs.make_cotangent(inp)
    got = run_backward(G, inp, dy, dev)
    ref = gbla_backward.backward_inputs(inp, dy)
    for n in NAMES:
        close_scaled(got[n], ref[n], TOL[dtype], n)


@pytest.mark.parametrize("heads", [1, 24])
@pytest.mark.parametrize("d,width", [(32, 4), (64, 3), (128, 4)])
def test_fp32_forward_edges(G, dev, orc, d, width, heads):
    say("fp32 forward edges", d, width, heads)
    inp = inputs.make_inputs(_case(d, inputs.F32, width, 52, heads=heads), lengths=EDGES)
    t = inputs.device_tensors(inp, dev)
    y = G.forward(t["q"], t["k"], t["v"], t["a"], t["r"], t["conv_w"], t["gamma"], eps=inp.eps,
                  cu_seqlens=t["cu_seqlens"], max_seqlen=t["max_seqlen"])
    torch.cuda.synchronize()
    close(y.cpu().numpy(), orc.forward_inputs(inp)["y"], 1e-5, "y")

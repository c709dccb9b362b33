"""The row products' tile shapes (two stages, three stages of B, quarters of a
short last round): which one runs depends on the rows per expert and on the
number of tiles only, and all add in the same order, so a token's results are
the same bits whichever batch it sits in."""
import pytest
import torch

from paper_2609_36070_amd.layer import DeviceLayer
from paper_2609_36070_amd.workloads import Workload, make_inputs
from tests.parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,fs", [(2560, 1280, 256), (1792, 2304, 0)])
def test_shapes_bitwise(d, f, fs):
    """2 experts: 2500 tokens run two stages (1250 rows per expert, 70 to 180
    tiles per launch), 1900 three stages (950 rows), 300 quarters (up to 40
    tiles).  K loops of 20 to 80 steps, whole and ragged turns of the six- and
    four-step loops."""
    sizes = (2500, 1900, 300)
    big = Workload("shapes", T=sizes[0], d=d, E=2, k=1, f=f, f_s=fs, backward=True)
    say(f"[gpu] shapes d={d} f={f} f_s={fs}")
    inp = make_inputs(big, 5)
    layers = [DeviceLayer(big.scaled(T=T), dict(inp, X=inp["X"][:T], dY=inp["dY"][:T])) for T in sizes]
    # the same routes: batches of different sizes may sum their logits in different orders
    for layer in layers:
        layer.route()
    torch.cuda.synchronize()
    for layer in layers[1:]:
        layer.topk_idx.copy_(layers[0].topk_idx[:layer.w.T])
        layer.topk_w.copy_(layers[0].topk_w[:layer.w.T])
    for layer in layers:
        layer.plan()
        layer.forward()
        layer.backward()
    torch.cuda.synchronize()
    for layer in layers[1:]:
        T = layer.w.T
        assert torch.equal(layers[0].Y[:T], layer.Y), T
        assert torch.equal(layers[0].dX[:T], layer.dX), T
        assert torch.equal(layers[0].dZ[:T], layer.dZ), T

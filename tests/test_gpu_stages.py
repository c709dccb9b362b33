"""The row products' tile shapes (two stages, three stages of B, quarters of a
short last round): which one runs depends on the rows per expert, on the length
of the product and on the number of tiles only, and all add in the same order, so
a token's results are the same bits whichever batch it sits in."""
import pytest
import torch

from paper_2609_36070_amd.layer import DeviceLayer
from paper_2609_36070_amd.workloads import Workload, make_inputs
from tests import dispatch
from tests.parity import say

pytestmark = pytest.mark.gpu

RUN = 100
TWO, THREE, QUARTERS = {"two"}, {"three"}, {"quarters"}


def shapes(w):
    """Tile shapes of the routed up/gate, dgrad and down (and dX) products and of
    the shared up/gate, with the routes of route_in_runs."""
    runs = w.T // RUN
    counts = [RUN * ((runs - e + w.E - 1) // w.E) for e in range(w.E)]
    tm, rows = sum(-(-c // 256) for c in counts), w.T
    return [dispatch.tile_shapes(tm * w.f // 128, w.d, rows, w.E), dispatch.tile_shapes(tm * w.f // 256, w.d, rows, w.E),
            dispatch.tile_shapes(tm * w.d // 256, w.f, rows, w.E)] + \
        ([dispatch.tile_shapes(-(-w.T // 256) * w.f_s // 128, w.d, w.T, 1)] if w.f_s else [])


def route_in_runs(T, E):
    """Runs of 100 tokens to each expert in turn."""
    return (torch.arange(T) // RUN % E).to(torch.int32)[:, None]


@pytest.mark.skipif(not dispatch.HAVE_CXX, reason="needs a host compiler")
@pytest.mark.parametrize("d,f,fs,E,sizes", [
    # products of 20 and 40 steps, then of 28 and 36: whole and ragged turns of
    # the six- and four-step loops
    (2560, 1280, 256, 2, {2600: (TWO, QUARTERS, TWO, QUARTERS), 2000: (THREE, QUARTERS, THREE, QUARTERS),
                          300: (QUARTERS,) * 4}),
    (1792, 2304, 0, 2, {2600: (TWO, TWO, TWO), 2000: (THREE, THREE, QUARTERS), 300: (QUARTERS,) * 3}),
    # more than a round of tiles, and the rest of it whole or in quarters
    (1280, 3328, 512, 5, {9500: (TWO | QUARTERS, TWO | QUARTERS, TWO, TWO), 6000: (TWO, TWO, TWO, TWO),
                          5000: (THREE | QUARTERS, THREE | QUARTERS, THREE, TWO), 3500: (THREE, THREE, THREE, QUARTERS),
                          200: (QUARTERS,) * 4}),
])
def test_shapes_bitwise(d, f, fs, E, sizes):
    big = Workload("shapes", T=max(sizes), d=d, E=E, k=1, f=f, f_s=fs, backward=True)
    say(f"[gpu] shapes d={d} f={f} f_s={fs} E={E} T={list(sizes)}")
    for T, want in sizes.items():
        assert tuple(shapes(big.scaled(T=T))) == tuple(want), (T, shapes(big.scaled(T=T)))
    inp = make_inputs(big, 5)
    layers = [DeviceLayer(big.scaled(T=T), dict(inp, X=inp["X"][:T], dY=inp["dY"][:T])) for T in sizes]
    for layer in layers:
        # the same routes and gate weights, whatever the batch
        layer.topk_idx.copy_(route_in_runs(layer.w.T, E))
        layer.topk_w.fill_(0.75)   # (1 would leave dZ zero)
        layer.plan()
        layer.forward()
        layer.backward()
    torch.cuda.synchronize()
    for layer in layers[1:]:
        T = layer.w.T
        assert torch.equal(layers[0].Y[:T], layer.Y), T
        assert torch.equal(layers[0].dX[:T], layer.dX), T
        assert torch.equal(layers[0].dZ[:T], layer.dZ), T

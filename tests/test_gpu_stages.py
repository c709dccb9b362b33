"""The row products with two and with three LDS stages of B: which one runs
depends on the rows per expert only, and both add in the same order, so a
token's results are the same bits whichever batch it sits in."""
import pytest
import torch

from paper_2609_36070_amd.layer import DeviceLayer
from paper_2609_36070_amd.workloads import Workload, make_inputs
from tests.parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,fs", [(256, 256, 256), (512, 768, 512), (768, 1280, 256)])
def test_two_and_three_stages_bitwise(d, f, fs):
    """K loops of 4 to 20 steps (and 8 to 40 in dX): whole and ragged turns of the
    six-step loop.  2500 tokens to 2 experts run two stages, their first 300
    three; the outputs of those tokens are equal bit for bit."""
    big = Workload("two", T=2500, d=d, E=2, k=1, f=f, f_s=fs, backward=True)
    say(f"[gpu] stages d={d} f={f} f_s={fs}")
    inp = make_inputs(big, 5)
    few = big.scaled(T=300)
    L = DeviceLayer(big, inp)
    S = DeviceLayer(few, dict(inp, X=inp["X"][:300], dY=inp["dY"][:300]))
    # the same routes: the two batch sizes sum their logits in different orders
    for layer in (L, S):
        layer.route()
    torch.cuda.synchronize()
    S.topk_idx.copy_(L.topk_idx[:300])
    S.topk_w.copy_(L.topk_w[:300])
    for layer in (L, S):
        layer.plan()
        layer.forward()
        layer.backward()
    torch.cuda.synchronize()
    assert torch.equal(L.Y[:300], S.Y)
    assert torch.equal(L.dX[:300], S.dX)

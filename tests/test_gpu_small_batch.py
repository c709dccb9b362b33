"""GPU parity of inference on small batches (the streaming expert kernels):
every output element against the oracle at the edges of their tiles.

The rule is: not kept for a backward, and T <= 16 (16-row tiles) or at most 64
routes per expert on average and a shared expert of bounded size (64-row
tiles).  Shapes lie on both sides of each
bound, with empty experts, experts of one row, of a whole tile and one row more.
"""
import pytest
import torch

from paper_2609_36070_amd.layer import DeviceLayer
from paper_2609_36070_amd.workloads import Workload, make_inputs
from tests import dispatch
from tests.parity import assert_close, to_np
from tests.test_gpu_small import forward_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [
    # 16-row tiles, one token; dense routing with a shared expert of another width
    Workload("one_dense", T=1, d=256, E=4, k=4, f=256, f_s=512, bias_std=0.5),
    Workload("sixteen", T=16, d=768, E=8, k=3, f=256),                # a whole 16-row tile at most
    Workload("seventeen", T=17, d=512, E=6, k=5, f=768, f_s=256, bias_std=1.0),   # first 64-row tiles
    Workload("one_per_expert", T=40, d=256, E=200, k=1, f=512),       # single rows, empty experts
    Workload("k16", T=50, d=1280, E=128, k=16, f=256, bias_std=0.5),
    Workload("dense_64", T=64, d=512, E=5, k=5, f=512, f_s=256),      # a whole 64-row tile per expert
    Workload("dense_65", T=65, d=512, E=5, k=5, f=512, f_s=256),      # past the bound: tile GEMMs
    Workload("dense_9", T=33, d=256, E=9, k=9, f=256),                # the sum over more than 8 experts
    Workload("skewed", T=250, d=256, E=16, k=4, f=256, bias_std=2.0),   # several 64-row tiles and empties
    # K of the up/gate products over two (unequal) and four workgroups
    Workload("split_2", T=5, d=2304, E=4, k=2, f=256, f_s=256, bias_std=0.5),
    Workload("split_4_dense", T=40, d=4352, E=3, k=3, f=256, f_s=512),
    Workload("mean_64", T=128, d=256, E=4, k=2, f=512, f_s=512),      # R = 64 E exactly
    Workload("mean_past", T=129, d=256, E=4, k=2, f=512, f_s=512),    # and past it
    Workload("shared_at", T=1024, d=256, E=64, k=1, f=256, f_s=1024),     # the shared expert's rows at their bound
    Workload("shared_past", T=1025, d=256, E=64, k=1, f=256, f_s=1024),   # and past it
], ids=lambda w: w.name)
def test_small_batch_parity(w):
    assert (dispatch.small_tiles(w) > 0) == (w.name not in ("dense_65", "mean_past", "shared_past"))
    forward_parity(w, seed=31)


@pytest.mark.parametrize("w,parts", [
    # dense routing past the small batches: the experts' products summed from
    # fp32 (in one round of tiles, in two), or the folded product (too much fp32
    # traffic for what it saves: 121 tiles of Y; more than half of the CUs: 132),
    # then the same with the activations kept
    (Workload("parts", T=1500, d=1024, E=4, k=4, f=512, f_s=512), True),
    (Workload("parts_rounds", T=1200, d=1024, E=16, k=16, f=256), True),
    (Workload("parts_one", T=600, d=512, E=1, k=1, f=512, f_s=256), True),
    (Workload("folded_121", T=2800, d=2816, E=2, k=2, f=256, f_s=512), False),
    (Workload("folded", T=2900, d=2816, E=2, k=2, f=256, f_s=512), False),
    (Workload("parts_train", T=130, d=512, E=9, k=9, f=256, backward=True), True),
    (Workload("folded_train", T=16700, d=512, E=2, k=2, f=256, f_s=256, backward=True), False),
], ids=lambda v: v.name if isinstance(v, Workload) else "")
def test_dense_down_products(w, parts):
    assert dispatch.dense_parts(w) == parts
    forward_parity(w, seed=32)


@pytest.mark.parametrize("w", [
    Workload("sparse", T=48, d=512, E=16, k=4, f=256, f_s=256, bias_std=1.0),
    Workload("dense", T=48, d=512, E=4, k=4, f=256, f_s=256),
], ids=lambda w: w.name)
def test_small_batch_against_tile_gemms(w):
    """The same layer keeping its activations runs the tile GEMMs: Y differs by
    summation order and the roundings it moves (one bf16 step of the largest
    value, 2^-8 relative, at H and at Y each)."""
    inp = make_inputs(w, 33)
    L = DeviceLayer(w, inp)
    L.step()
    y = L.Y.clone()
    inp["dY"] = inp["X"]
    K = DeviceLayer(w, inp, with_backward=True)
    K.route(); K.plan(); K.forward()
    torch.cuda.synchronize()
    assert_close("Y (small batch vs tiles)", to_np(y), to_np(K.Y), rel=2 ** -7)
    for _ in range(2):       # repeats bitwise, with the workspace overwritten between
        L.ws.fill_(255)
        L.step()
        torch.cuda.synchronize()
        assert torch.equal(L.Y, y)


@pytest.mark.parametrize("d", [512, 2304])
def test_small_batch_in_one_window_ring(d):
    """A ring holding every route runs a small batch as the one-pass forward
    does, K slices included: the same bits."""
    w = Workload("ring", T=30, d=d, E=8, k=2, f=256, f_s=256, bias_std=0.5)
    inp = make_inputs(w, 34)
    full, ring = DeviceLayer(w, inp), DeviceLayer(w, inp, ring_rows=w.T * w.k)
    full.step(), ring.step()
    torch.cuda.synchronize()
    assert torch.equal(full.Y, ring.Y)

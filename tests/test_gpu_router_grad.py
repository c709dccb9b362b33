"""GPU parity of the router's part of the backward (softmax backward, dW_r and
the router term of dX) at the edges of its expert groups, token tiles and
column blocks, every output element against the oracle."""
import pytest
import torch

from paper_2609_36070_amd.workloads import Workload
from tests.parity import assert_close, to_np
from tests.test_gpu_small import backward_parity, forward_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [
    # experts: one accumulator group, two, four, several passes; multiples of 8 or not
    Workload("e8", T=257, d=256, E=8, k=3, f=256, backward=True),
    Workload("e9", T=16, d=512, E=9, k=2, f=256, f_s=256, backward=True),
    Workload("e16", T=17, d=768, E=16, k=16 - 1, f=256, backward=True),
    Workload("e33", T=300, d=1280, E=33, k=8, f=256, bias_std=1.0, backward=True),
    Workload("e64", T=15, d=256, E=64, k=16, f=512, backward=True),
    Workload("e72", T=130, d=512, E=72, k=1, f=256, f_s=256, backward=True),
], ids=lambda w: w.name)
def test_router_gradient_edges(w):
    L, inp, _, idx_g, w_orc = forward_parity(w, seed=41)
    backward_parity(L, inp, w, idx_g, w_orc)
    # dW_r against the GPU's own dZ in float64: bf16 X times dZ split in two
    # bf16 parts (2^-16 of each dZ dropped), summed in fp32 over <= 300 tokens
    ref = inp["X"].astype("float64").T @ to_np(L.dZ).astype("float64")
    assert_close("dW_r (own dZ)", to_np(L.dW_r), ref, rel=5e-5)
    torch.cuda.synchronize()

"""What the forward does with its workspace: it writes inside the bytes it is
given, runs with the named regions alone, and with dense routing leaves the
per-route outputs' regions alone."""
import pytest
import torch

from oracle import moe_oracle as O
from paper_2609_36070_amd import binding as B
from paper_2609_36070_amd.layer import DeviceLayer
from paper_2609_36070_amd.workloads import Workload, make_inputs
from tests.parity import assert_close, check_route_and_plan, say, to_np, weights_dict

pytestmark = pytest.mark.gpu

CASES = [
    Workload("dense_small", T=40, d=512, E=5, k=5, f=512, f_s=256),          # fp32 products, 64-row tiles
    Workload("dense_slices", T=3, d=4352, E=3, k=3, f=256, f_s=512),         # and K slices before them
    Workload("dense_short", T=130, d=512, E=9, k=9, f=512, f_s=256),         # fp32 products, tile GEMMs
    Workload("sparse_slices", T=6, d=4096, E=12, k=2, f=256, f_s=256, bias_std=0.5),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
@pytest.mark.parametrize("fused", [False, True])
def test_forward_stays_in_its_workspace(w, fused):
    inp = make_inputs(w, 51)
    L = DeviceLayer(w, inp)
    off, nbytes = B.moe_workspace_region(L.shape, False, B.WS_YSH)
    regions = (off + max(nbytes, 1) + 255) // 256 * 256
    full = B.moe_workspace_bytes(L.shape, False)
    assert regions < full
    call = B.moe_forward_fused if fused else B.moe_forward
    for room in (regions, full):
        say(f"[gpu] {w.name} workspace {room} of {full}")
        L.ws = torch.full((full + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        L.route()
        L.plan()
        before = [L.ws_tensor(r, torch.uint8, (-1,)).clone() for r in (B.WS_YEXP, B.WS_YSH)]
        L.Y.fill_(7.0)
        call(L.shape, L.X, L.weights, L.topk_idx, L.topk_w, L.plan_bufs, L.Y, False, L.ws, ws_bytes=room)
        torch.cuda.synchronize()
        assert bool((L.ws[room:] == 0xA5).all()), "written past the workspace"
        if w.k == w.E:
            for r, b in zip((B.WS_YEXP, B.WS_YSH), before):
                assert torch.equal(L.ws_tensor(r, torch.uint8, (-1,)), b), "a per-route output was written"
        Zo, idx_g = check_route_and_plan(L, inp, w)
        fw = O.moe_forward(inp["X"], weights_dict(inp), idx_g, O.gate_weights(Zo, idx_g))
        assert_close("Y", to_np(L.Y), fw["Y"])
    with pytest.raises(B.MoeError):
        call(L.shape, L.X, L.weights, L.topk_idx, L.topk_w, L.plan_bufs, L.Y, False, L.ws, ws_bytes=regions - 1)

"""GPU checks of the one- and two-launch plans and of the one-launch router at
the edges of their ranges: the plan integer for integer against a stable sort,
the logits against float64, selection and weights from the GPU's own logits.
"""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2609_36070_amd import binding as B
from tests.parity import LOGIT_ABS_TOL, assert_close, say, to_np

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("T,k,E,bad", [
    (1, 1, 1, 0), (64, 1, 256, 0), (1024, 2, 7, 0), (683, 3, 33, 2),      # one launch, 1 and 2 groups
    (2049, 1, 200, 1), (1024, 8, 128, 0),                                 # one launch, up to 8 groups
    (8193, 1, 3, 1), (4096, 3, 256, 0), (5001, 16, 64, 5),                # two launches, ragged blocks
    (65536, 16, 20, 3), (65537, 16, 256, 4),                              # 2^20 routes and just past them
])
def test_plan_edges(T, k, E, bad):
    R = T * k
    say(f"[gpu] plan T={T} k={k} E={E} bad={bad}")
    rng = np.random.default_rng(R + E)
    p = rng.dirichlet(np.full(E, 0.3))                 # skewed, with empty experts
    idx = rng.choice(E, size=R, p=p).astype(np.int32)
    at = rng.choice(R, size=bad, replace=False)
    idx[at] = np.where(np.arange(bad) % 2, -1, E)      # ids outside the range are not placed
    ok = (idx >= 0) & (idx < E)
    order = np.argsort(np.where(ok, idx, E), kind="stable")[: ok.sum()]
    counts = np.bincount(idx[ok], minlength=E)
    pos = np.full(R, -1, np.int64)
    pos[order] = np.arange(ok.sum())
    sh = B.make_shape(T, 256, E, min(k, E), 256) if k <= E else B.make_shape(R, 256, E, 1, 256)
    ws = torch.full((B.moe_workspace_bytes(sh, False),), 255, dtype=torch.uint8, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    c, o, pm, rp = (torch.full((n,), -7, **i32) for n in (E, E + 1, R, R))
    B.moe_plan(sh, dev(idx), B.plan_bufs(c, o, pm, rp), ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_np(c), counts)
    assert np.array_equal(to_np(o), np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(to_np(pm)[: ok.sum()], order)
    assert np.array_equal(to_np(rp), pos)
    off, _ = B.moe_workspace_region(sh, False, B.WS_ERROR)
    assert int(ws[off:off + 4].view(torch.int32).item()) == (1 if bad else 0)


@pytest.mark.parametrize("T,d,E,k", [
    (1, 256, 8, 8), (17, 512, 12, 3), (2048, 768, 16, 4),          # 16 columns, one per lane
    (16, 4096, 24, 6), (33, 256, 32, 8),                           # two per lane, padded
    (50, 1280, 25, 5),                                             # odd: not aligned, the general router
    (100, 512, 48, 8), (5, 7168, 64, 16),                          # four per lane
    (300, 256, 96, 8), (2047, 512, 128, 16),                       # eight per lane
    (40, 768, 200, 10), (31, 256, 256, 1),                         # sixteen per lane
    (2049, 512, 32, 8), (1100, 512, 127, 8), (2100, 512, 128, 8),  # past its range: the other routers
    (33, 5120, 128, 8), (33, 5376, 128, 8), (9, 7168, 200, 4),     # long rows of many experts: its last and theirs
    (33, 4608, 72, 2), (33, 4864, 72, 2), (1280, 4608, 256, 4), (1281, 4608, 256, 4),
])
def test_router_edges(T, d, E, k):
    say(f"[gpu] router T={T} d={d} E={E} k={k}")
    rng = np.random.default_rng(T + d + E)
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16)
    X, W_r = bf(rng.standard_normal((T, d))), bf(rng.standard_normal((d, E)) / np.sqrt(d))
    bias = rng.standard_normal(E).astype(np.float32)
    sh = B.make_shape(T, d, E, k, 256)
    ws = torch.empty(B.moe_workspace_bytes(sh, False), dtype=torch.uint8, device="cuda")
    logits = torch.full((T, E), float("nan"), device="cuda")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), float("nan"), device="cuda")
    B.moe_route(sh, X.cuda(), W_r.cuda(), dev(bias), logits, idx, w, ws)
    torch.cuda.synchronize()
    Z = X.double().numpy() @ W_r.double().numpy() + bias
    got = to_np(logits)
    assert np.abs(got - Z).max() <= LOGIT_ABS_TOL
    assert np.array_equal(to_np(idx), O.topk_select(got, k))
    assert_close("weights", to_np(w), O.gate_weights(got.astype(np.float64), to_np(idx)), rel=1e-5)

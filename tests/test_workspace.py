"""Workspace sizes (host functions): a workspace made for a batch holds every
smaller one, with and without the backward, in one pass, as a ring and in MXFP8."""
import pytest

from paper_2609_36070_amd import binding as B

LAYERS = [
    # d, E, k, f, f_s: dense routing (short batches sum fp32 products), few and
    # many experts, K slices at one token and at many
    (7168, 8, 8, 2048, 2048), (256, 16, 16, 256, 0), (2816, 2, 2, 256, 512), (1024, 4, 4, 2048, 0),
    (4096, 64, 1, 2048, 2048), (4096, 32, 8, 1536, 0), (2048, 128, 8, 768, 0), (2304, 200, 1, 512, 1024),
    (256, 8, 2, 512, 0),
]
TOKENS = sorted(set(list(range(0, 70)) + [t + e for t in (128, 256, 512, 1000, 1024, 2048, 4096, 12800, 32768)
                                          for e in (-1, 0, 1)]))


@pytest.mark.parametrize("d,E,k,f,fs", LAYERS)
def test_sizes_never_fall_with_the_tokens(d, E, k, f, fs):
    def never_falls(name, size):
        got = [size(B.make_shape(t, d, E, k, f, fs)) for t in TOKENS]
        for a, b, t in zip(got, got[1:], TOKENS[1:]):
            assert 0 < a <= b, f"{name}: {a} bytes before {t} tokens, {b} there"

    for bwd in (0, 1):
        never_falls(f"one pass, backward {bwd}", lambda s: B.moe_workspace_bytes(s, bwd))
        for rows in (1, 700, 8192):
            never_falls(f"ring of {rows}, backward {bwd}", lambda s: B.moe_ring_workspace_bytes(s, rows, bwd))
    for mode in (0, 1, 2):
        never_falls(f"MXFP8, mode {mode}", lambda s: B.moe_mx_workspace_bytes(s, mode))


@pytest.mark.parametrize("d,E,k,f,fs", LAYERS)
def test_ring_sizes_never_fall_with_the_rows(d, E, k, f, fs):
    for t in (1, 16, 61, 300, 2000):
        s = B.make_shape(t, d, E, k, f, fs)
        rows = sorted({1, 16, 100, max(t * k - 1, 1), t * k, 4 * t * k})
        got = [B.moe_ring_workspace_bytes(s, r, 0) for r in rows]
        assert got[0] > 0 and got == sorted(got)


@pytest.mark.parametrize("d,E,k,f,fs", LAYERS)
def test_named_regions_hold_what_they_say(d, E, k, f, fs):
    """The regions follow each other without overlap, each of its documented size."""
    for t in (1, 16, 61, 1000):
        s = B.make_shape(t, d, E, k, f, fs)
        end = 0
        for which, n in ((B.WS_A, t * k * f), (B.WS_B, t * k * f), (B.WS_H, t * k * f), (B.WS_YEXP, t * k * d),
                         (B.WS_YSH, t * d)):
            off, nbytes = B.moe_workspace_region(s, False, which)
            assert nbytes == 2 * n and off >= end
            end = off + nbytes
        # MXFP8 starts right after the BF16 forward's regions
        assert B.moe_mx_workspace_bytes(s, 0) < end + t * d * 2 + t * k * f * 2 + t * d // 16 + t * k * f // 16 + 4096

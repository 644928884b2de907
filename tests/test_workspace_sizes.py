"""A workspace made for the largest batch of a layer takes every smaller one: its size never falls as the number of tokens grows, also
where another batch is split differently (the router's backward: a unit of 32 slices more per block is fewer blocks) or runs on other kernels (the expert
backward at slice width 96: one pass in small batches and again in large ones, two kernels between).  Questions to the library that need no device (it then counts 256 compute units)."""
import pytest

from paper_2510_04286_amd import binding as B

LAYERS = [(96, 224, 16, 2), (96, 384, 16, 2), (96, 384, 64, 1), (96, 768, 3, 1), (96, 1536, 16, 2), (96, 192, 9, 7), (48, 192, 16, 2), (48, 832, 2, 2),
          (24, 160, 3, 3), (64, 256, 32, 2), (128, 512, 64, 2), (192, 96, 4, 1), (64, 256, 8, 2, "f32"), (40, 100, 5, 3, "f32"), (192, 96, 4, 1, "f32")]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda v: "-".join(map(str, v)))
def test_the_backward_workspace_never_shrinks(layer):
    ds, He, E, k = layer[:4]
    dtype = layer[4] if len(layer) > 4 else "bf16"
    S = 4
    per = S * k
    edges = [u * 32 // per for u in (1, E, 2 * E, 2 * E + 1, 128, 192, 193, 255, 256, 257, 512, 513, 256 * 8, 256 * 10, 256 * 12, 256 * 16, 256 * 32)]
    tokens = sorted({t for e in edges for t in range(max(1, e - 3), e + 4)} | set(range(1, 12000, 37)))
    sizes = []
    for t in tokens:
        cfg = B.make_config(t, S * ds, S, k, E, He, dtype=dtype)
        assert B.slicemoe_backward_uses_mfma(cfg) == (1 if dtype == "bf16" else 0)
        sizes.append(B.slicemoe_backward_workspace_bytes(cfg))
    falls = [(a, b) for a, b, x, y in zip(tokens, tokens[1:], sizes, sizes[1:]) if y < x]
    assert not falls, falls[:5]

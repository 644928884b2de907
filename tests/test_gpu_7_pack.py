"""slicemoe_pack_weights against the fragment layout that csrc/pack.hip documents, rebuilt in numpy, bit for bit: widths
with and without zero padding of the K-steps and output tiles, one and two 32-expert tiles, a single hidden tile."""
import numpy as np
import pytest

from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs

pytestmark = pytest.mark.gpu

SHAPES = [(24, 40, 96), (48, 3, 32), (64, 32, 256), (96, 64, 64), (128, 1, 160)]


def frags_layer1(W, scale):
    """[nt][ks][lane][8] bf16 bits of W[K, N] * scale: lane (i, g), slot m holds W[16 ks + 8 g + m][32 nt + i]."""
    K, N = W.shape
    P = np.zeros(((K + 15) // 16 * 16, N), np.float32)
    P[:K] = W * scale
    P = P.reshape(-1, 2, 8, N // 32, 32)                      # ks, g, m, nt, i
    return wl.bf16_bits(P.transpose(3, 0, 1, 4, 2)).reshape(-1)   # nt, ks, g, i, m


def frags_layer2(W, scale, outer_first):
    K, N = W.shape
    P = np.zeros((K, (N + 31) // 32 * 32), np.float32)
    P[:, :N] = W
    P = np.clip(P * scale, -65504, 65504).astype(np.float16)
    P = P.reshape(K // 32, 2, 2, 2, 4, -1, 32)                # ht, s, m/4, g, m%4, nt, i
    P = P.transpose(5, 0, 1, 3, 6, 2, 4) if outer_first else P.transpose(0, 1, 5, 3, 6, 2, 4)
    return np.ascontiguousarray(P).view(np.uint16).reshape(-1)


def biases_f16(b, scale):
    q = np.clip(b * scale, -65504, 65504).astype(np.float16).reshape(-1, 4, 2, 4)   # ht, r/4, g, r%4
    return np.ascontiguousarray(q.transpose(0, 2, 1, 3)).view(np.uint16).reshape(-1)


def padded_f32(b):
    out = np.zeros((b.size + 31) // 32 * 32, np.float32)
    out[:b.size] = b
    return out.view(np.uint16)


@pytest.mark.parametrize("ds,E,He", SHAPES)
def test_packed_buffer_is_the_documented_layout(ds, E, He):
    from paper_2510_04286_amd import binding as B
    shape, _, w = make_inputs(wl.SliceMoEShape("pack", T=1, d=2 * ds, S=2, E=E, k=1, He=He))
    cfg = B.config_of(shape)
    got = B.pack(cfg, B.weights_to_device(w, "bf16"))["packed"].cpu().numpy()
    regions = [frags_layer1(w["Wr1"], 1.0), frags_layer2(w["Wr2"], 1.0, True), padded_f32(w["br1"]), padded_f32(w["br2"])]
    for e in range(E):
        regions += [frags_layer1(w["W1"][e], 0.25), frags_layer2(w["W2"][e], 4.0, False), biases_f16(w["b1"][e], 0.25),
                    padded_f32(w["b2"][e])]
    at = 0
    for n, want in enumerate(regions):   # every region starts on a 256-byte boundary
        want = want.view(np.uint8)
        assert np.array_equal(got[at:at + want.size], want), f"region {n}"
        at = (at + want.size + 255) // 256 * 256
    assert at == got.size


def test_matrices_of_more_than_two_gib():
    """2^28 fragments and more per matrix (64 experts of 2^20 + 32 hidden units): the last tiles of the last expert."""
    import torch
    from paper_2510_04286_amd import binding as B
    ds, E, He = 24, 64, 2 ** 20 + 32
    cfg = B.config_of(wl.SliceMoEShape("wide", T=1, d=2 * ds, S=2, E=E, k=1, He=He))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)

    def normal(*size):
        return torch.empty(size, dtype=torch.bfloat16, device="cuda:0").normal_(generator=gen)

    w = {"Wr1": normal(ds, 256), "br1": normal(256), "Wr2": normal(256, E), "br2": normal(E), "W1": normal(E, ds, He),
         "b1": normal(E, He), "W2": normal(E, He, ds), "b2": normal(E, ds)}
    got = B.pack(cfg, w)["packed"]
    n1, n2 = 32 * He * 2, 32 * He * 2   # bytes of an expert's W1 and W2 (both padded to 32)
    base = got.numel() - ((n1 + 255) // 256 * 256 + (n2 + 255) // 256 * 256 + (He * 2 + 255) // 256 * 256 + 256)
    tail = 2 * 64 * 16                  # two fragments of 64 lanes: the last hidden tile
    f1 = got[base + n1 - tail:base + n1].cpu().numpy()
    f2 = got[base + n1 + n2 - tail:base + n1 + n2].cpu().numpy()
    np.testing.assert_array_equal(f1, frags_layer1(w["W1"][-1, :, -32:].float().cpu().numpy(), 0.25).view(np.uint8))
    np.testing.assert_array_equal(f2, frags_layer2(w["W2"][-1, -32:].float().cpu().numpy(), 4.0, False).view(np.uint8))

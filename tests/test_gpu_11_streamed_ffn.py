"""The streamed expert kernels at their edges: row tiles (of 384, 256 and 128 rows at widths 128, 192 and 384, of 512 where a batch
of width 128 fills those better) that are full, one row short or one row over, experts without a row and with one, blocks with several row tiles
and several experts, the fewest hidden tiles that the pipelined kernel takes and the fewer that stay with the other, and k that is and is not a
power of two."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import TOL_BF16, make_inputs, rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ds,He,k,Ns,tile", [(128, 96, 2, 20000, 384), (128, 128, 3, 120000, 384), (192, 96, 3, 9001, 256), (192, 160, 2, 70000, 256),
                                             (384, 96, 2, 3000, 128), (384, 128, 1, 40000, 128),
                                             (128, 96, 1, 110000, 512), (128, 256, 2, 100000, 512),
                                             (128, 32, 2, 30000, 512), (128, 64, 3, 20000, 512), (192, 32, 2, 9001, 256), (192, 64, 3, 20000, 256),
                                             (384, 32, 2, 3000, 128), (384, 64, 1, 40000, 128)])
def test_row_tiles(ds, He, k, Ns, tile):
    import torch
    from paper_2510_04286_amd import binding as B
    E = 12
    s = wl.SliceMoEShape("tiles", T=Ns, d=ds, S=1, E=E, k=k, He=He)
    # slot 0 of a slice: experts 0, 2, 3, ... with 0, 1, tile - 1, tile, tile + 1, ... rows, the rest on expert 11; other slots: 8, 9
    idx = np.empty((Ns, k), np.int32)
    idx[:, 0] = 11
    at = 0
    for e, rows in zip((2, 3, 4, 5, 6, 7), (1, tile - 1, tile, tile + 1, 2 * tile + 33, 31)):
        idx[at:at + rows, 0] = e
        at += rows
    for j in range(1, k):
        idx[:, j] = 7 + j
    order = np.argsort(wl.uniform01(5, 0, 0, Ns))   # scattered over the batch
    idx = idx[order]
    pk = (0.25 + 0.5 * wl.uniform01(4, 0, 0, idx.size)).reshape(idx.shape)
    w = wl.make_weights(s)
    h = wl.make_h(s)
    d = oracle.dispatch(idx, E, -1)
    ref = oracle.expert_rows(h.reshape(-1, ds), idx, pk, d["perm"], s.Na, w["W1"], w["b1"], w["W2"], w["b2"])
    cfg = B.config_of(s)
    wd = B.pack(cfg, B.weights_to_device(w, s.dtype))

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    y = torch.full((s.Na + 1, ds), 123.0, dtype=B.y_dtype(cfg), device="cuda:0")
    B.slicemoe_expert_ffn(cfg, B.to_device(h, s.dtype), dev(pk.astype(np.float32).reshape(-1)), dev(d["offsets"]), dev(d["perm"]), wd, y[:-1])
    got = y.float().cpu().numpy()
    assert np.all(got[-1] == 123.0)   # nothing past the last row
    err = np.abs(got[:-1] - ref).max() / rms(ref)
    print(f"\n[width {ds} He {He}] max|err|/rms={err:.3e}")
    assert err <= TOL_BF16


@pytest.mark.parametrize("He,E,k,Ns", [(96, 12, 1, 110000), (256, 12, 2, 100000), (512, 64, 2, 50000)])
def test_width_128_the_other_kernel_gives_the_same_bits(He, E, k, Ns):
    """Batches that fill the 512-row tiles of ffn_streamed_kernel better than the pipelined kernel's 384 (one round of the chip instead of
    two, two instead of three): the first slices of such a batch have the bits that they have in one that the pipelined kernel takes."""
    import torch
    from paper_2510_04286_amd import binding as B
    s, _, w = make_inputs(wl.SliceMoEShape("rounds", T=4, d=128, S=1, E=E, k=k, He=He))
    wd = B.pack(B.config_of(s), B.weights_to_device(w, s.dtype))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    h = torch.randn((Ns, 128), generator=gen, device="cuda:0").to(torch.bfloat16)

    def layer(n):
        cfg = B.config_of(wl.SliceMoEShape("rounds", T=n, d=128, S=1, E=E, k=k, He=He))
        out, ws = torch.empty((n, 128), dtype=torch.bfloat16, device="cuda:0"), B.alloc_workspace(cfg)
        B.slicemoe_forward(cfg, h[:n], wd, out, ws)
        torch.cuda.synchronize()
        return out
    n = 70000 // k
    assert torch.equal(layer(Ns)[:n], layer(n))

"""The kernels for small batches (router and expert FFN, see split_tiles and ffn_is_small) at their edges: one slice, tiles
and units that end inside 32, one to four tiles per block, a block that has fewer, the largest batch they take and the
smallest that they do not, hidden widths below, at and above eight tiles, experts without a row, k from 1 to 8, a capacity
limit, logit noise.  Whole forward against the fp64 oracle with the bars of the forward tests, tables bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import TOL_BF16, make_inputs, rms, routing_agreement

pytestmark = pytest.mark.gpu


def shape(ds, He, E, k, Ns, S=1, cf=0.0):
    return wl.SliceMoEShape("small", T=Ns // S, d=S * ds, S=S, E=E, k=k, He=He, capacity_factor=cf)


CASES = {
    "one_slice": shape(64, 256, 32, 2, 1),
    "w64_31": shape(64, 256, 32, 2, 31),
    "w64_33": shape(64, 64, 7, 1, 33),
    "w64_3tiles": shape(64, 96, 5, 2, 1000, S=4),
    "w64_9tiles": shape(64, 288, 64, 2, 777),
    "w64_last_split_ffn": shape(64, 256, 32, 2, 6144, S=16),     # 1.5 units per CU
    "w64_first_other_ffn": shape(64, 256, 32, 2, 6160, S=16),
    # an expert of two hidden tiles in the pipelined kernel, whose second layer lags by a whole unit: blocks with one unit per
    # wavefront, with several, and with the rows of two experts
    "w24_first_other_ffn": shape(24, 96, 16, 2, 8208, S=16),       # 2 units per CU
    "w192_last_split_ffn": shape(192, 768, 16, 2, 8064, S=4),      # two rounds: 504 units and half a unit of each expert
    "w192_first_other_ffn": shape(192, 768, 16, 2, 8068, S=4),
    "w192_8192": shape(192, 768, 16, 2, 8192, S=4),
    "w192_8196": shape(192, 768, 16, 2, 8196, S=4),
    "w128_last_split_ffn": shape(128, 96, 16, 2, 12160, S=4),      # three rounds
    "w128_first_other_ffn": shape(128, 96, 16, 2, 12164, S=4),
    "w64_2tiles_other_ffn": shape(64, 64, 16, 2, 6400, S=4),
    "w64_2tiles_E64": shape(64, 64, 64, 3, 20000, S=4),
    "w64_2tiles_E5": shape(64, 64, 5, 2, 9000, S=4),
    "w64_4tiles_E64": shape(64, 128, 64, 3, 20000, S=4),
    "w64_two_tiles_a_block": shape(64, 128, 16, 3, 8193),
    "w64_last_split_router": shape(64, 128, 16, 2, 32768, S=16),  # four tiles per CU
    "w64_first_other_router": shape(64, 128, 16, 2, 32784, S=16),
    "w64_k8_capacity": shape(64, 256, 64, 8, 700, cf=0.7),
    "w64_E64_last_split_router": shape(64, 32, 64, 2, 16384, S=16),   # two tiles per CU with two 32-expert tiles
    "w24": shape(24, 96, 16, 2, 517),
    "w24_11tiles": shape(24, 352, 33, 2, 40),
    "w48": shape(48, 192, 16, 2, 300),
    "w96": shape(96, 384, 16, 3, 250),
    "w128": shape(128, 512, 64, 2, 200),
    "w128_17tiles": shape(128, 544, 9, 1, 65),
    "w192": shape(192, 768, 16, 2, 100),
    "w192_E40_1tile": shape(192, 32, 40, 2, 129),
    "w384": shape(384, 96, 5, 2, 33),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_batches(name):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(CASES[name])
    cfg = B.config_of(s)
    noisy = name in ("w64_33", "w96", "w64_E64_last_split_router")
    sigma = 0.3 if noisy else 0.0
    noise = wl.make_router_draws(s)[0] if noisy else None
    ref = oracle.forward_train(h, s.S, s.k, w, noise=noise, drop_u=None, capacity=s.capacity(), tau=1.0, sigma=sigma, rate=0.0)
    wd, hd = B.pack(cfg, B.weights_to_device(w, s.dtype)), B.to_device(h, s.dtype)
    ws = B.alloc_workspace(cfg)
    ws.fill_(0xFF)   # nothing is read unwritten
    out = torch.full_like(hd, 3.0)
    if noisy:
        B.slicemoe_forward_train(cfg, hd, wd, out, ws, temperature=1.0, noise_std=sigma, dropout_rate=0.0,
                                 noise=torch.from_numpy(noise).to("cuda:0"), drop_u=None, capacity_alpha=0.0)
    else:
        B.slicemoe_forward(cfg, hd, wd, out, ws)
    torch.cuda.synchronize()
    v = B.workspace_views(cfg, ws)
    idx = v["topk_idx"].cpu().numpy()
    mism, n_tie = routing_agreement(idx, ref["idx"], ref["logits"])
    inv = v["inv"].cpu().numpy().reshape(-1, s.k)
    # a near-tie moves one assignment, and under a capacity limit which later ones of the two experts are dropped
    bad = mism | np.any((inv >= 0) != (ref["inv"].reshape(-1, s.k) >= 0), axis=1)
    table = oracle.dispatch(idx, s.E, s.capacity())
    for n in ("counts_raw", "counts", "offsets", "inv"):
        np.testing.assert_array_equal(v[n].cpu().numpy().reshape(-1), np.asarray(table[n]).reshape(-1), err_msg=n)
    kept = int(table["offsets"][-1])
    np.testing.assert_array_equal(v["perm"].cpu().numpy()[:kept], table["perm"][:kept])
    diff = np.abs(out.float().cpu().numpy() - ref["h_out"]).reshape(-1, s.ds)
    err = diff[~bad].max() / rms(ref["h_out"])
    print(f"\n[{name}] near-ties {n_tie}, masked {int(bad.sum())}, max|err|/rms {err:.2e}")
    assert n_tie <= 1 and bad.sum() <= 4
    assert err <= TOL_BF16


@pytest.mark.parametrize("ds,He,E,k", [(24, 96, 16, 2), (48, 192, 40, 2), (64, 256, 32, 2), (64, 64, 64, 3), (64, 288, 16, 1),
                                       (96, 384, 16, 2), (96, 160, 33, 2), (128, 512, 64, 2), (192, 768, 16, 3), (192, 96, 40, 2),
                                       (128, 64, 12, 2), (192, 32, 40, 2)])
def test_a_slice_does_not_depend_on_its_batch(ds, He, E, k):
    """Dropless, a slice's selected experts, probabilities and output are the same bits whether it comes alone, in a batch small
    enough for the split kernels of the router, the experts or both, or in a large one: every sum has one order."""
    import torch
    from paper_2510_04286_amd import binding as B
    full = shape(ds, He, E, k, 40000, S=4)   # beyond both kernels' small batches
    s, _, w = make_inputs(shape(ds, He, E, k, 4, S=4))
    wd = B.pack(B.config_of(s), B.weights_to_device(w, s.dtype))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    h = torch.randn((full.T, full.d), generator=gen, device="cuda:0").to(torch.bfloat16)

    def layer(T):
        cfg = B.config_of(shape(ds, He, E, k, 4 * T, S=4))
        ws, out = B.alloc_workspace(cfg), torch.empty((T, full.d), dtype=torch.bfloat16, device="cuda:0")
        B.slicemoe_forward(cfg, h[:T], wd, out, ws)
        torch.cuda.synchronize()
        v = B.workspace_views(cfg, ws)
        return out, v["topk_idx"].reshape(-1, k).clone(), v["topk_p"].reshape(-1, k).clone()

    want = layer(full.T)
    for T in (1, 9, 250, 1500, 5000):
        got = layer(T)
        for name, a, b in zip(("h'", "topk_idx", "topk_p"), got, want):
            assert torch.equal(a, b[:a.shape[0]]), f"{name}, {T} tokens"

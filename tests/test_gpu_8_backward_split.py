"""The matrix-core backward at the edges of its split: rows per unit (32), hidden tiles per block (4 or 8, fewer,
or several groups of them), widths with zero-padded pieces, experts with no row, one row, or all of them, and the division
of assignment ids by k.  Every gradient against the fp64 oracle with the bars of test_gpu_4_backward.py, whose derivation
(one bf16 rounding of dL/dh, fp32 sums over operands of 16 or more significant bits) covers these kernels; the widths that
run on three-term operands (24, 48, 192) are held to a tenth of the weight-gradient bar."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs, rms, routing_agreement

pytestmark = pytest.mark.gpu

NAMES = ("Wr1", "br1", "Wr2", "br2", "W1", "b1", "W2", "b2")


def shape(ds, He, E, k, T, S=4, cf=0.0):
    return wl.SliceMoEShape("split", T=T, d=S * ds, S=S, E=E, k=k, He=He, capacity_factor=cf)


CASES = {
    "w24_3tiles": shape(24, 96, 16, 2, 129),
    "w24_5tiles": shape(24, 160, 4, 1, 40),             # five hidden tiles on eight wavefronts
    "w24_9tiles": shape(24, 288, 4, 2, 50),             # more than a block: rows and weights in kernels of their own
    "w48_6tiles": shape(48, 192, 16, 2, 100),
    "w48_1tile": shape(48, 32, 3, 3, 33),
    "w48_9tiles": shape(48, 288, 2, 2, 65),
    "w64_empty_experts": shape(64, 256, 64, 1, 3, S=2),  # six rows for 64 experts
    "w64_k5": shape(64, 256, 7, 5, 31),
    "w64_k6": shape(64, 128, 7, 6, 17),
    "w64_k7": shape(64, 64, 8, 7, 9),
    "w64_capacity_1": shape(64, 256, 8, 2, 16, cf=0.05),  # one or two rows per expert are kept
    "w64_one_row": shape(64, 256, 1, 1, 1, S=1),
    "w64_hot": shape(64, 256, 5, 1, 3001),               # one expert takes every row: its slots come from many blocks
    "w96_5tiles": shape(96, 160, 6, 2, 77),
    "w128_9tiles": shape(128, 288, 3, 2, 47),
    "w128_hot": shape(128, 64, 4, 2, 1500),
    "w192_2tiles": shape(192, 64, 8, 2, 65),
    "w192_5tiles": shape(192, 160, 3, 3, 22),
    # an expert's biases beyond the LDS of the rows kernel: the fp32 kernels (the router's part stays on the matrix cores)
    "w24_biases_beyond_lds": shape(24, 40000, 2, 1, 10, S=2),
    "w192_biases_beyond_lds": shape(192, 32000, 2, 1, 5, S=2),
    # two 32-expert tiles in the router's kernels; slices that end inside a 32-slice unit, one unit, several blocks of units
    "w24_E40": shape(24, 96, 40, 2, 331, S=3),
    "w48_E64": shape(48, 64, 64, 2, 8),
    "w64_E33": shape(64, 64, 33, 3, 7, S=3),
    "w192_E40": shape(192, 64, 40, 2, 30),
}


@pytest.mark.parametrize("name", list(CASES))
def test_backward_at_the_edges_of_the_split(name):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(CASES[name])
    if name.endswith("hot"):
        w["br2"] = wl.to_storage(np.where(np.arange(s.E) == s.E - 1, 8.0, w["br2"]), s.dtype)
    cfg = B.config_of(s)
    assert B.slicemoe_backward_uses_mfma(cfg) == (0 if name.endswith("beyond_lds") else 1)
    dout = wl.make_dout(s)
    ref_f = oracle.forward_train(h, s.S, s.k, w, noise=None, drop_u=None, capacity=s.capacity(), tau=1.0, sigma=0.0, rate=0.0)
    ref = oracle.backward(h, s.S, s.k, w, dout, ref_f["idx"], ref_f["inv"])
    wd, ws = B.pack(cfg, B.weights_to_device(w, s.dtype)), B.alloc_workspace(cfg)
    hd = B.to_device(h, s.dtype)
    out = torch.empty_like(hd)
    B.slicemoe_forward(cfg, hd, wd, out, ws)
    grads, d_h = B.alloc_weight_grads(cfg), torch.full_like(hd, 5.0)
    for t in grads.values():
        t.fill_(7.0)   # the call overwrites
    bws = torch.full((B.slicemoe_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaNs: nothing is read unwritten
    B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, s.dtype), d_h, grads, bws)
    torch.cuda.synchronize()
    views = B.workspace_views(cfg, ws)
    _, n_tie = routing_agreement(views["topk_idx"].cpu().numpy(), ref_f["idx"], ref_f["logits"])
    assert n_tie == 0, "this case was chosen to have no near-tie; pick another token count"
    np.testing.assert_array_equal(views["inv"].cpu().numpy(), ref_f["inv"])
    bound = 2.0 ** -8 * np.abs(ref["d_h"]) + 2e-4 * rms(ref["d_h"])
    excess = (np.abs(d_h.float().cpu().numpy() - ref["d_h"]) / bound).max()
    err = {n: np.abs(grads[n].cpu().numpy() - ref[n]).max() / max(rms(ref[n]), 1e-30) for n in NAMES}
    print(f"\n[{name}] dL/dh at {excess:.2f} of its bound; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert excess <= 1.0
    assert max(err.values()) <= 5e-4, err
    if s.ds in (24, 48, 192):
        assert max(err[n] for n in ("W1", "b1", "W2", "b2")) <= 5e-5, err


@pytest.mark.parametrize("ds,He,T,E,draws", [(24, 96, 512, 16, False), (48, 192, 1024, 16, False), (192, 768, 512, 16, False),
                                              (48, 192, 600, 40, True), (192, 768, 400, 40, True)])
def test_gradients_of_the_three_term_widths_are_fp32_exact(ds, He, T, E, draws):
    """Widths 24, 48 and 192 keep every operand at 24 bits: the relative 2-norm error of each weight gradient against the fp64
    oracle stays below 2^-21 = 4.8e-7, four roundings to fp32 of every summand (probability, dL/dp, dL/dg, dL/du) and of the
    sums over them.  Operands of 22 bits, or an order of the matrix instructions' sums that is biased, do not meet it (8.5e-7)."""
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(shape(ds, He, E, 2, T, S=768 // ds))
    cfg = B.config_of(s)
    dout = wl.make_dout(s)
    noise, drop_u = wl.make_router_draws(s) if draws else (None, None)
    tau, sigma, rate = (0.8, 0.1, 0.2) if draws else (1.0, 0.0, 0.0)
    wd, ws, hd = B.pack(cfg, B.weights_to_device(w, s.dtype)), B.alloc_workspace(cfg), B.to_device(h, s.dtype)
    train = {"temperature": tau, "noise_std": sigma, "dropout_rate": rate, "capacity_alpha": 0.0,
             "noise": torch.from_numpy(noise).to("cuda:0") if draws else None,
             "drop_u": torch.from_numpy(drop_u).to("cuda:0") if draws else None}
    out = torch.empty_like(hd)
    B.slicemoe_forward_train(cfg, hd, wd, out, ws, **train)
    grads, d_h = B.alloc_weight_grads(cfg), torch.empty_like(hd)
    bws = torch.empty(B.slicemoe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, s.dtype), d_h, grads, bws, train=train)
    torch.cuda.synchronize()
    views = B.workspace_views(cfg, ws)
    kw = {"tau": tau, "noise": noise, "sigma": sigma, "drop_u": drop_u, "rate": rate}
    ref = oracle.backward(h, s.S, s.k, w, dout, views["topk_idx"].cpu().numpy(), views["inv"].cpu().numpy(), **kw)
    err = {n: np.linalg.norm(grads[n].cpu().numpy().astype(np.float64) - ref[n]) / np.linalg.norm(ref[n]) for n in NAMES}
    print("\n" + " ".join(f"{n} {e:.2e}" for n, e in err.items()))
    assert max(err.values()) <= 2.0 ** -21, err

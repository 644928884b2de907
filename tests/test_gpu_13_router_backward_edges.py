"""The router's backward at the edges of its tiles of 32 slices, through the kernel that gives dL/dg and dL/dh together (widths 24, 48 and 64,
96 with up to 32 experts) and the pair beside it (96 with more): one slice, tiles one slice short and one over, the last block without a
tile, expert counts that are no multiple of 4 or 32 (noise rows that start unaligned), one to eight selections (two are requested ahead),
capacity drops (assignments without a row), dropout that leaves one or no selection, and the capacity loss.  Against the fp64 oracle with the bars
of the backward tests: dL/dh one bf16 rounding (2^-8 of the element) plus 2e-4 of the RMS, weight gradients 5e-4 of the RMS."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs, rms, routing_agreement

pytestmark = pytest.mark.gpu

CASES = {   # width, E, k, T, S, capacity factor, tau, sigma, rate, alpha
    "24_one_slice": (24, 5, 1, 1, 1, 0.0, 1.0, 0.2, 0.0, 0.0),
    "24_E33_k3": (24, 33, 3, 31, 1, 0.0, 0.8, 0.1, 0.3, 0.0),
    "24_E64_k8": (24, 64, 8, 33, 3, 0.0, 1.0, 0.0, 0.9, 40.0),
    "48_E7_k3_drops": (48, 7, 3, 65, 1, 0.6, 1.0, 0.1, 0.0, 0.0),
    "48_E35_k2": (48, 35, 2, 103, 3, 0.0, 1.5, 0.2, 0.2, 0.0),
    "64_E3_k2": (64, 3, 2, 63, 1, 0.0, 1.0, 0.3, 0.2, 40.0),
    "64_E40_k5_drops": (64, 40, 5, 43, 3, 0.7, 1.0, 0.0, 0.5, 0.0),
    "64_E1": (64, 1, 1, 97, 1, 0.0, 1.0, 0.1, 0.2, 0.0),
    "64_many_tiles": (64, 6, 3, 8231, 1, 0.9, 1.0, 0.1, 0.2, 0.0),
    "96_E30_k3": (96, 30, 3, 61, 2, 0.0, 0.8, 0.1, 0.4, 40.0),
    "96_E34_k2": (96, 34, 2, 95, 1, 0.8, 1.0, 0.1, 0.2, 40.0),
    # the capacity loss's sums take four assignments a load: fewer than that, one left over, and more than its blocks take in one round
    "64_cap_1": (64, 5, 1, 1, 1, 0.0, 1.0, 0.2, 0.0, 40.0),
    "64_cap_3": (64, 2, 1, 3, 1, 0.0, 1.0, 0.2, 0.0, 40.0),
    "64_cap_2049": (64, 7, 1, 683, 3, 0.0, 1.0, 0.2, 0.2, 400.0),
    "24_cap_131073": (24, 9, 3, 43691, 1, 0.0, 1.0, 0.0, 0.2, 4000.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gradients(name):
    import torch
    from paper_2510_04286_amd import binding as B
    ds, E, k, T, S, cf, tau, sigma, rate, alpha = CASES[name]
    shape, h, w = make_inputs(wl.SliceMoEShape(name, T=T, d=S * ds, S=S, E=E, k=k, He=64, capacity_factor=cf))
    cfg = B.config_of(shape)
    assert B.slicemoe_backward_uses_mfma(cfg) == 1
    dout, (noise, drop_u) = wl.make_dout(shape), wl.make_router_draws(shape)
    okw = dict(tau=tau, sigma=sigma, rate=rate)
    ref_f = oracle.forward_train(h, S, k, w, noise=noise, drop_u=drop_u, capacity=shape.capacity(), **okw)
    capg = oracle.capacity_surrogate(ref_f["idx"], ref_f["pk"], E, alpha)["grad"] if alpha else None
    ref = oracle.backward(h, S, k, w, dout, ref_f["idx"], ref_f["inv"], noise=noise, drop_u=drop_u, capg=capg, **okw)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    wd, ws, hd = B.pack(cfg, B.weights_to_device(w, shape.dtype)), B.alloc_workspace(cfg), B.to_device(h, shape.dtype)
    tkw = dict(temperature=tau, noise_std=sigma, dropout_rate=rate, noise=dev(noise), drop_u=dev(drop_u))
    B.slicemoe_forward_train(cfg, hd, wd, torch.empty_like(hd), ws, **tkw)
    grads, d_h = B.alloc_weight_grads(cfg), torch.full_like(hd, 5.0)
    for t in grads.values():
        t.fill_(7.0)   # the call overwrites
    bws = torch.full((B.slicemoe_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaNs: nothing is read unwritten
    B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, shape.dtype), d_h, grads, bws, train=dict(tkw, capacity_alpha=alpha))
    torch.cuda.synchronize()
    views = B.workspace_views(cfg, ws)
    _, n_tie = routing_agreement(views["topk_idx"].cpu().numpy(), ref_f["idx"], ref_f["logits"])
    assert n_tie == 0, "this case was chosen to have no near-tie; pick another token count"
    np.testing.assert_array_equal(views["inv"].cpu().numpy(), ref_f["inv"])
    bound = 2.0 ** -8 * np.abs(ref["d_h"]) + 2e-4 * rms(ref["d_h"])
    worst = (np.abs(d_h.float().cpu().numpy() - ref["d_h"]) / bound).max()
    err = {}
    for n, t in grads.items():
        scale = rms(ref[n])
        e = np.abs(t.cpu().numpy() - ref[n]).max()
        err[n] = e / scale if scale > 0 else e
    print(f"\n[{name}] dL/dh {worst:.2f} of its bound; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert worst <= 1.0
    assert max(err.values()) <= 5e-4, err

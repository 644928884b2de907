"""The fp32 kernels (fp32 storage, and every shape the bf16 matrix-core kernels do not take) at the edges of their tiles:
rows and slices that end inside a unit of 32, slice widths that are no multiple of 4 or 32 or exceed one chunk of columns
(64, 128), hidden widths below a tile and above one group of 256, router widths below 256, one to 64 experts, k up to 8, one
expert with every row.  Forward and every gradient against the fp64 oracle.  Bars: those of the forward and backward
tests (1e-4 of the RMS for fp32 storage; for bf16 storage the one rounding of the result, 2^-8 relative per element, plus
2e-4 RMS, and for h' the fp16 rows on top; 5e-4 of the RMS for the fp32 weight gradients): the arithmetic is fp32 throughout, so only
the order of sums of at most a few thousand terms differs."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import TOL_F32, make_inputs, rms, routing_agreement

pytestmark = pytest.mark.gpu

NAMES = ("Wr1", "br1", "Wr2", "br2", "W1", "b1", "W2", "b2")


def shape(ds, He, E, k, T, Hr, dtype="f32", S=3, cf=0.0):
    return wl.SliceMoEShape("generic", T=T, d=S * ds, S=S, E=E, k=k, He=He, dtype=dtype, capacity_factor=cf, Hr=Hr)


CASES = {
    "one_of_each": shape(1, 1, 1, 1, 1, 1, S=1),
    "ds5": shape(5, 3, 2, 2, 11, 7),
    "ds32": shape(32, 64, 8, 2, 33, 256),
    "ds33": shape(33, 37, 5, 3, 43, 100),
    "ds64_E64": shape(64, 256, 64, 2, 90, 256),            # Wr2 beyond the LDS
    "ds65_two_groups": shape(65, 300, 9, 2, 37, 256),
    "ds128": shape(128, 33, 4, 2, 50, 64),
    "ds132_k8": shape(132, 40, 33, 8, 21, 64),
    # five to seven output tiles on eight wavefronts: some have none.  A hidden width of a few units makes the product short
    "ds160_five_tiles": shape(160, 2, 3, 2, 41, 64),
    "ds192_six_tiles": shape(192, 4, 3, 2, 41, 64),
    "ds224_seven_tiles": shape(224, 2, 3, 2, 41, 64),
    "bf16_ds192_six_tiles": shape(192, 8, 4, 2, 70, 64, "bf16"),
    "ds257_wide": shape(257, 270, 3, 2, 21, 130, S=2),
    "hot": shape(48, 72, 4, 1, 900, 128),
    "capacity": shape(64, 128, 8, 2, 200, 256, cf=0.6),
    "bf16_ds40": shape(40, 50, 6, 2, 61, 128, "bf16"),
    "bf16_ds384": shape(384, 96, 5, 2, 27, 256, "bf16", S=2),
    "bf16_ds64_Hr64": shape(64, 96, 7, 3, 45, 64, "bf16"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_generic_layer_and_gradients(name):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(CASES[name])
    if name == "hot":
        w["br2"] = wl.to_storage(np.where(np.arange(s.E) == 1, 8.0, w["br2"]), s.dtype)
    cfg = B.config_of(s, flags=B.SLICEMOE_FLAG_FORCE_GENERIC)
    dout = wl.make_dout(s)
    ref_f = oracle.forward_train(h, s.S, s.k, w, noise=None, drop_u=None, capacity=s.capacity(), tau=1.0, sigma=0.0, rate=0.0)
    ref = oracle.backward(h, s.S, s.k, w, dout, ref_f["idx"], ref_f["inv"])
    wd, ws = B.weights_to_device(w, s.dtype), B.alloc_workspace(cfg)
    hd = B.to_device(h, s.dtype)
    out = torch.full_like(hd, 3.0)
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

    def excess(got, want, extra):
        scale = rms(want)
        bound = np.full_like(want, TOL_F32 * scale) if s.dtype == "f32" else 2.0 ** -8 * np.abs(want) + extra * scale
        return (np.abs(got.float().cpu().numpy() - want) / bound).max()

    worst = {"h'": excess(out, ref_f["h_out"], 2e-3), "dL/dh": excess(d_h, ref["d_h"], 2e-4)}
    err = {n: np.abs(grads[n].cpu().numpy() - ref[n]).max() / max(rms(ref[n]), 1e-30) if rms(ref[n]) > 0 else
           np.abs(grads[n].cpu().numpy()).max() for n in NAMES}
    print(f"\n[{name}] of their bounds: {worst}; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert max(worst.values()) <= 1.0, worst
    assert max(err.values()) <= 5e-4, err

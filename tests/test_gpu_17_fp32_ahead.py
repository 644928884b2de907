"""The fp32 kernels' split and the instances that request weights ahead.  How the expert backward hands its units of 32 rows to the blocks: one unit per block up to as many units as there are
compute units, two from the next one on (the blocks of the second half then have none), experts without rows, a single row, and
one expert with every row.  And the instances that request weights a batch ahead (32 and 64 columns, whole quads): hidden widths that
leave wavefronts without hidden units, without a part of dL/dx, or with a second group of 256.  And the router instance that does so
(256 hidden units, whole chunks of 64 columns, whole octets of experts): one chunk and two, one and two tiles of experts, one to four
assignments of which a capacity limit drops some, several units per block.  Every gradient against the fp64 oracle on the routing that the forward call left behind.  Bars: those of the fp32 edge
tests (1e-4 of the RMS for dL/dh; 5e-4 of the RMS for the weight gradients): only the order of fp32 sums of at most 9000 terms differs."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import TOL_F32, make_inputs, rms, routing_agreement

pytestmark = pytest.mark.gpu

NAMES = ("Wr1", "br1", "Wr2", "br2", "W1", "b1", "W2", "b2")


def shape(T, E, k, S=4, ds=16, He=32, Hr=32, cf=0.0):
    return wl.SliceMoEShape("split", T=T, d=S * ds, S=S, E=E, k=k, He=He, dtype="f32", Hr=Hr, capacity_factor=cf)


CASES = {   # the expert that the router's bias prefers, if any: then units are as many as its rows need
    "one_row": (shape(1, 3, 1, S=1), None),
    "one_unit_each": (shape(12, 8, 2), None),
    "units_255": (shape(2040, 2, 1), 1),
    "units_256": (shape(2048, 2, 1), 1),
    "units_257": (shape(2049, 2, 1), 0),
    "two_groups_of_hidden_units": (shape(70, 5, 2, He=290), None),
    "w32_one_tile": (shape(50, 3, 2, ds=32, He=32), None),
    "w32_seven_tiles": (shape(50, 3, 2, ds=32, He=224), None),
    "w64_three_tiles": (shape(50, 3, 2, ds=64, He=96), None),
    "w64_two_groups": (shape(50, 3, 2, ds=64, He=288), None),
    "w64_units_per_block": (shape(2100, 2, 1, ds=64, He=64), 1),
    "router_one_expert_tile": (shape(11, 8, 1, ds=64, Hr=256), None),
    "router_two_expert_tiles": (shape(40, 40, 4, ds=128, Hr=256, cf=0.7), None),
    "router_units_per_block": (shape(2100, 16, 3, ds=64, Hr=256), None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gradients_at_the_edges(name):
    import torch
    from paper_2510_04286_amd import binding as B
    case, hot = CASES[name]
    s, h, w = make_inputs(case)
    if hot is not None:
        w["br2"] = wl.to_storage(np.where(np.arange(s.E) == hot, 50.0, w["br2"]), s.dtype)
    cfg = B.config_of(s)
    dout = wl.make_dout(s)
    wd, ws, hd = B.weights_to_device(w, s.dtype), B.alloc_workspace(cfg), B.to_device(h, s.dtype)
    B.slicemoe_forward(cfg, hd, wd, torch.empty_like(hd), ws)
    views = B.workspace_views(cfg, ws)
    idx, inv = views["topk_idx"].cpu().numpy(), views["inv"].cpu().numpy()
    if hot is not None:
        assert (idx == hot).all()
    ref = oracle.backward(h, s.S, s.k, w, dout, idx, inv)
    grads, d_h = B.alloc_weight_grads(cfg), torch.full_like(hd, 5.0)
    for t in grads.values():
        t.fill_(7.0)   # the call overwrites
    bws = torch.full((B.slicemoe_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaNs: nothing is read unwritten
    for _ in range(2):   # the second call finds the first one's values in the workspace
        B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, s.dtype), d_h, grads, bws)
    torch.cuda.synchronize()
    err = {n: np.abs(grads[n].cpu().numpy() - ref[n]).max() / (rms(ref[n]) or 1.0) for n in NAMES}
    err_h = np.abs(d_h.cpu().numpy() - ref["d_h"]).max() / rms(ref["d_h"])
    print(f"\n[{name}] dL/dh {err_h:.1e}; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert err_h <= TOL_F32
    assert max(err.values()) <= 5e-4, err


FORWARD = {   # the expert kernel that requests ahead: 32 and 64 columns, hidden widths of one tile, some, all wavefronts' and two groups
    "w32_one_tile": shape(50, 3, 2, ds=32, He=32),
    "w32_seven_tiles": shape(21, 5, 3, ds=32, He=224, cf=0.6),
    "w64_three_tiles": shape(50, 3, 2, ds=64, He=96),
    "w64_two_groups": shape(50, 3, 2, ds=64, He=288),
    "w64_one_row": shape(1, 2, 1, S=1, ds=64, He=256),
    # the router's second layer in LDS: columns in quads; rows, since columns would be 720 bytes too many (464 without the
    # histogram's counts); rows of an odd width
    "router_columns": shape(9, 39, 3, ds=492, Hr=128),
    "router_rows_fit_columns_do_not": shape(9, 39, 3, ds=496, Hr=256),
    "router_rows": shape(9, 17, 3, ds=20, Hr=129),
}


@pytest.mark.parametrize("name", list(FORWARD))
def test_forward_at_the_edges(name):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(FORWARD[name])
    cfg = B.config_of(s)
    ref = oracle.forward_train(h, s.S, s.k, w, noise=None, drop_u=None, capacity=s.capacity(), tau=1.0, sigma=0.0, rate=0.0)
    wd, ws, hd = B.weights_to_device(w, s.dtype), B.alloc_workspace(cfg), B.to_device(h, s.dtype)
    out = torch.full_like(hd, 3.0)
    B.slicemoe_forward(cfg, hd, wd, out, ws)
    torch.cuda.synchronize()
    _, n_tie = routing_agreement(B.workspace_views(cfg, ws)["topk_idx"].cpu().numpy(), ref["idx"], ref["logits"])
    assert n_tie == 0, "this case was chosen to have no near-tie; pick another token count"
    err = np.abs(out.cpu().numpy() - ref["h_out"]).max() / rms(ref["h_out"])
    print(f"\n[{name}] h' {err:.1e}")
    assert err <= TOL_F32

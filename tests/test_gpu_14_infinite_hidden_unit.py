"""A router hidden unit that is infinite (a diverged step): the slice's logits are no numbers, and its dL/dg and dL/dh say so, whatever
kernels recompute them.  The slice is the last one and a capacity limit drops both of its assignments, so nothing but the router's own
recomputation can bring the NaN in; every other slice's gradient stays a number."""
import numpy as np
import pytest

from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ds,E", [(24, 16), (48, 40), (64, 16), (64, 40), (96, 16), (96, 40), (128, 16), (128, 64), (192, 16), (80, 16)])
def test_gradients_are_not_numbers(ds, E):
    import torch
    from paper_2510_04286_amd import binding as B
    Ns = 70
    shape, h, w = make_inputs(wl.SliceMoEShape("inf", T=Ns, d=ds, S=1, E=E, k=2, He=64, capacity_factor=0.2 * E / 2))   # 20% of the rows each
    h = h.copy()
    h[:, 0] = 0.0
    h[-1] = 0.0
    h[-1, 0] = 1.0e38
    w = {n: np.array(a, copy=True) for n, a in w.items()}
    w["Wr1"][0] = 0.0
    w["Wr1"][0, 5] = 64.0      # feature 0, which only the last slice has, reaches this unit alone and takes it beyond the largest fp32
    w["Wr2"][5] = -1.0         # logits: +inf for experts 0 and 1, -inf for the others
    w["Wr2"][5, :2] = 1.0
    w["br2"][:] = 0.0
    w["br2"][:2] = 16.0        # the experts of every slice: full long before the last one
    cfg = B.config_of(shape)
    wd, hd, ws = B.pack(cfg, B.weights_to_device(w, shape.dtype)), B.to_device(h, shape.dtype), B.alloc_workspace(cfg)
    dout = B.to_device(wl.make_dout(shape), shape.dtype)
    B.slicemoe_forward(cfg, hd, wd, torch.empty_like(hd), ws)
    v = B.workspace_views(cfg, ws)
    assert sorted(v["topk_idx"].reshape(-1, 2)[-1].tolist()) == [0, 1] and v["inv"].reshape(-1, 2)[-1].tolist() == [-1, -1]
    d_h, grads = torch.zeros_like(hd), B.alloc_weight_grads(cfg)
    bws = torch.zeros(B.slicemoe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    B.slicemoe_backward(cfg, hd, wd, ws, dout, d_h, grads, bws)
    torch.cuda.synchronize()
    assert torch.isnan(grads["br2"]).all()
    assert torch.isnan(d_h[-1]).any()
    assert torch.isfinite(d_h[:-1]).all()
    for n in ("W1", "b1", "W2", "b2"):   # the experts never saw the slice
        assert torch.isfinite(grads[n]).all(), n

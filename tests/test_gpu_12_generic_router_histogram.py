"""The generic router leaves the per-chunk histogram (eight slices a chunk) that the dispatch's scatter sums: the dispatch of a forward
call against the oracle's dispatch of the same selections, entry by entry, at the last batch that takes this route and the first that
does not (16 384 slices of 16 experts, 8192 of 17 to 32, 4096 of 64), at a last block of one slice, at rows that end before their padding, with one
expert, with eight selections a slice, with a capacity and from both storage types.  Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs

pytestmark = pytest.mark.gpu

CASES = {   # T, E, k, dtype, capacity factor
    "one_slice": (1, 3, 2, "f32", 0.0),
    "one_expert": (17, 1, 1, "f32", 0.0),
    "k8": (1025, 33, 8, "bf16", 0.0),
    "last_of_16": (16384, 16, 2, "f32", 0.0),
    "beyond_16": (16385, 16, 2, "f32", 0.0),
    "last_of_17": (8192, 17, 3, "f32", 0.0),
    "beyond_17": (8193, 17, 3, "bf16", 0.0),
    "last_of_64": (4096, 64, 1, "f32", 1.1),
    "beyond_64": (4097, 64, 1, "f32", 1.1),
    "capacity": (777, 8, 2, "f32", 0.7),
}


@pytest.mark.parametrize("name", list(CASES))
def test_forward_dispatches_the_generic_routers_selections(name):
    import torch
    from paper_2510_04286_amd import binding as B
    T, E, k, dtype, cf = CASES[name]
    s = wl.SliceMoEShape("hist", T=T, d=4, S=1, E=E, k=k, He=4, dtype=dtype, capacity_factor=cf, Hr=8)
    _, h, w = make_inputs(s)
    cfg = B.config_of(s, flags=B.SLICEMOE_FLAG_FORCE_GENERIC)
    ws = B.alloc_workspace(cfg)
    ws.fill_(0xFF)   # nothing is read unwritten
    hd = B.to_device(h, s.dtype)
    B.slicemoe_forward(cfg, hd, B.weights_to_device(w, s.dtype), torch.empty_like(hd), ws)
    torch.cuda.synchronize()
    v = {n: t.cpu().numpy() for n, t in B.workspace_views(cfg, ws).items() if n != "y"}
    want = oracle.dispatch(v["topk_idx"], E, s.capacity())
    assert np.bincount(v["topk_idx"].ravel(), minlength=E).max() > 0
    for n in ("counts_raw", "counts", "offsets", "inv"):
        np.testing.assert_array_equal(v[n], want[n], err_msg=n)
    kept = want["offsets"][-1]
    np.testing.assert_array_equal(v["perm"][:kept], want["perm"][:kept])

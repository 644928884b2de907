"""The expert backward where every pre-activation is far below zero, z = -5 +- 0.15: the activation and its derivative are small there
(1e-6, 1e-5) and keep their own precision, they are not what is left of two numbers next to one.  One expert and one assignment per slice, so that
its probability is 1 and z = x W1 + b1.  Against the fp64 oracle, relative 2-norm.

Bar, of dW2 (sums of the activation) and of dW1 and db1 (sums of the derivative): the relative 2-norm of the error that the coefficients of
csrc/gelu_grad.h leave in exact arithmetic at the case's own z, computed here; two roundings of the exponent, up to 24, of
2^-24 each and of its power of two; an error of z of 2^-21 (sums around 5 in fp32) times the logarithmic derivative, below 6; and
2^-17 where the second products take operands of 16 significant bits.  The summands' errors are independent of the upstream gradient's sign, so
that the sum's is theirs; twice that for the sample."""
import math
import os
import re

import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04286_amd", "csrc", "gelu_grad.h")


def fit_errors(x):
    """In exact arithmetic, at every x: 2 Phi(-x), twice the derivative of GELU at -x, and the error of both."""
    txt = open(HEADER).read()
    p = float(re.search(r"kGeluGradP = ([0-9.e+-]+)f", txt).group(1))
    c = [float(v.rstrip("f")) for v in re.search(r"kGeluGradN\[\d+\] = \{([^}]*)\}", txt).group(1).split(", ")]
    e = np.exp(-x * x / 2)
    q = np.array([math.erfc(v / math.sqrt(2.0)) for v in x])
    return q, q - math.sqrt(2.0 / math.pi) * x * e, np.abs(e * (1.0 - x * np.polyval(c, 1.0 / (1.0 + p * x))) - q)


def test_the_coefficients_give_what_their_header_says():
    """8.6e-9 of 2 Phi(-x) at the most; relative to it 1.2e-5 up to x = 4, 3.3e-2 up to 11 (1e-28), and 2.7e-4 of the derivative, whose
    zero is at 0.75."""
    x = np.linspace(0.0, 13.0, 13001)
    q, r, err = fit_errors(x)
    assert err.max() <= 8.7e-9 and err[x < 0.5].max() <= 5.2e-9
    assert (err / q)[x <= 4].max() <= 1.2e-5 and (err / q)[x <= 11].max() <= 3.3e-2
    assert (err / np.abs(r))[(x >= 2) & (x <= 11)].max() <= 2.8e-4


@pytest.mark.gpu
@pytest.mark.parametrize("ds,He,T", [(24, 96, 300), (48, 96, 300), (64, 96, 300), (64, 288, 300), (96, 96, 300), (96, 384, 9000), (128, 96, 300), (192, 96, 300)])
def test_gradients_far_below_zero(ds, He, T):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(wl.SliceMoEShape("tail", T=T, d=ds, S=1, E=1, k=1, He=He))
    w = dict(w, b1=np.full_like(w["b1"], -5.0), W1=w["W1"] * 0.25)
    cfg = B.config_of(s)
    assert B.slicemoe_backward_uses_mfma(cfg) == 1
    dout = wl.make_dout(s)
    hd, ws = B.to_device(h, s.dtype), B.alloc_workspace(cfg)
    wd = B.pack(cfg, B.weights_to_device(w, s.dtype))
    B.slicemoe_forward(cfg, hd, wd, torch.empty_like(hd), ws)
    v = B.workspace_views(cfg, ws)
    ref = oracle.backward(h, s.S, s.k, w, dout, v["topk_idx"].cpu().numpy(), v["inv"].cpu().numpy())
    grads, d_h = B.alloc_weight_grads(cfg), torch.empty_like(hd)
    bws = torch.empty(B.slicemoe_backward_workspace_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, s.dtype), d_h, grads, bws)
    torch.cuda.synchronize()
    x = -(h.astype(np.float64) @ w["W1"][0] + w["b1"][0]).reshape(-1)[:200000]
    assert 4.2 < x.min() and x.max() < 5.8
    q, r, fit = fit_errors(x)
    other = 24 * 2.0 ** -23 + 2.0 ** -23 + 6 * 2.0 ** -21 + (0.0 if ds in (24, 48, 192) else 2.0 ** -17)
    bar_w2, bar_w1 = 2 * (np.linalg.norm(x * fit) / np.linalg.norm(x * q) + other), 2 * (np.linalg.norm(fit) / np.linalg.norm(r) + other)
    bar = {"W2": bar_w2, "W1": bar_w1, "b1": bar_w1}
    err = {n: float(np.linalg.norm(grads[n].cpu().numpy() - ref[n]) / np.linalg.norm(ref[n])) for n in bar}
    print(f"\n[width {ds}, He {He}] " + " ".join(f"{n} {err[n]:.1e} of {bar[n]:.1e}" for n in bar))
    assert all(err[n] <= bar[n] for n in bar), err

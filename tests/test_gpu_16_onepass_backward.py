"""The one-pass expert backward (slice widths 24, 48 and 96) where its split can go wrong: hidden tiles that fill a pass of the block's
wavefronts exactly, leave some idle, or need several passes (dL/dx and dL/dp of the passes before are read back and added to),
one row, a ragged last unit, several units per block, every k, a capacity limit, an expert that takes all rows.  Against the fp32
kernels, which every shape has (SLICEMOE_FLAG_FORCE_GENERIC), on the same routing; and on both sides of every line of the choice between this
kernel and the two others at width 96 (csrc/onepass_split.h says which side a case is on) and of the two ways to split the units, against 64 bits.

Bars.  Both sides sum in fp32; the operands of the one-pass kernel's second products have 24 significant bits at 24 and 48, 16 at 96 (two
bf16 terms), so a summand differs by at most 2^-17 of itself at 96 and by fp32 rounding at the others, and a gradient, a sum
of them that does not cancel below its RMS, by 2e-4 (96) or 5e-5 of that RMS; dL/dh is rounded to bf16 on both sides: one unit in the
last place, 2^-7 relative, plus the same share of the RMS."""
import numpy as np
import pytest

import oracle
from paper_2510_04286_amd import workload as wl
from tests.common import make_inputs, rms
from tests.test_onepass_split import split

pytestmark = pytest.mark.gpu

NAMES = ("Wr1", "br1", "Wr2", "br2", "W1", "b1", "W2", "b2")


def shape(ds, He, E, k, T, S=4, cf=0.0):
    return wl.SliceMoEShape("onepass", T=T, d=S * ds, S=S, E=E, k=k, He=He, capacity_factor=cf)


CASES = {
    "w24_1_pass_full": shape(24, 128, 4, 2, 65),      # eight tiles of 16 on eight wavefronts
    "w24_16_wavefronts": shape(24, 160, 3, 3, 41),    # ten tiles on sixteen
    "w24_16_wavefronts_full": shape(24, 256, 5, 2, 70),
    "w24_2_passes": shape(24, 288, 4, 2, 53),         # eighteen: ten and eight
    "w24_5_passes": shape(24, 1056, 2, 1, 90),        # sixty-six: fourteen four times, ten
    "w24_half_of_the_shares": shape(24, 96, 6, 2, 240, S=32),   # 480 units and six experts on 480 blocks: shares of two
    "w24_one_row": shape(24, 32, 1, 1, 1, S=1),
    "w24_k8": shape(24, 96, 9, 8, 30),
    "w48_1_pass_full": shape(48, 192, 5, 2, 100),     # twelve tiles on twelve wavefronts
    "w48_2_passes": shape(48, 224, 7, 5, 33),         # fourteen: eight and six
    "w48_5_passes": shape(48, 832, 2, 2, 40),         # fifty-two: twelve, twelve, twelve, twelve, four
    "w48_capacity": shape(48, 192, 8, 2, 64, cf=0.4),
    "w48_units_per_block": shape(48, 64, 2, 2, 3000, S=8),
    "w96_1_pass_full": shape(96, 192, 9, 7, 29),
    "w96_2_passes_one_unit": shape(96, 384, 16, 2, 200, S=8),
    "w96_4_passes_one_unit": shape(96, 768, 3, 1, 77),
    "w96_2_passes_many_units": shape(96, 224, 5, 4, 2700, S=8),   # 2700 units: ten and more per block
    "w96_hot": shape(96, 160, 4, 1, 3000, S=4),
}


@pytest.mark.parametrize("name", list(CASES))
def test_one_pass_backward_equals_the_fp32_kernels(name):
    import torch
    from paper_2510_04286_amd import binding as B
    s, h, w = make_inputs(CASES[name])
    if name.endswith("hot"):
        w["br2"] = wl.to_storage(np.where(np.arange(s.E) == s.E - 1, 8.0, w["br2"]), s.dtype)
    dout = B.to_device(wl.make_dout(s), s.dtype)
    hd = B.to_device(h, s.dtype)
    cfg = B.config_of(s)
    wd, ws, out = B.pack(cfg, B.weights_to_device(w, s.dtype)), B.alloc_workspace(cfg), torch.empty_like(hd)
    B.slicemoe_forward(cfg, hd, wd, out, ws)
    got = []
    for flags in (0, B.SLICEMOE_FLAG_FORCE_GENERIC):
        c = B.config_of(s, flags=flags)
        assert B.slicemoe_backward_uses_mfma(c) == (0 if flags else 1)
        grads, d_h = B.alloc_weight_grads(c), torch.full_like(hd, 5.0)
        for t in grads.values():
            t.fill_(7.0)   # the call overwrites
        bws = torch.full((B.slicemoe_backward_workspace_bytes(c),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaNs: nothing is read unwritten
        for _ in range(2):   # the second call finds the first one's values in the workspace
            B.slicemoe_backward(c, hd, wd, ws, dout, d_h, grads, bws)
        torch.cuda.synchronize()
        got.append({n: t.cpu().numpy().astype(np.float64) for n, t in grads.items()} | {"d_h": d_h.float().cpu().numpy().astype(np.float64)})
    bar = 2e-4 if s.ds == 96 else 5e-5
    err = {n: np.abs(got[0][n] - got[1][n]).max() / max(rms(got[1][n]), 1e-30) for n in NAMES}
    excess = (np.abs(got[0]["d_h"] - got[1]["d_h"]) / (2.0 ** -7 * np.abs(got[1]["d_h"]) + bar * rms(got[1]["d_h"]))).max()
    print(f"\n[{name}] dL/dh at {excess:.2f} of its bound; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert excess <= 1.0
    assert max(err[n] for n in ("W1", "b1", "W2", "b2")) <= bar, err
    assert max(err.values()) <= 5e-4, err


TRAIN = dict(tau=0.8, sigma=0.1, rate=0.2)
EDGES = {   # (shape, whether the one pass takes it at 256 compute units)
    "w24_16_wavefronts": (shape(24, 224, 5, 2, 60), True),
    "w48_capacity": (shape(48, 288, 6, 2, 80, cf=0.7), True),
    # two units per expert and fewer: a block for every unit; one unit more
    "w24_8_units": (shape(24, 96, 4, 2, 128, S=1), True),
    "w24_9_units": (shape(24, 96, 4, 2, 129, S=1), True),
    "w48_64_experts_few_rows": (shape(48, 224, 64, 2, 33, S=2), True),
    "w96_64_experts_a_row_each": (shape(96, 384, 64, 2, 9, S=4), True),
    "w96_8_units": (shape(96, 224, 4, 2, 128, S=1), True),
    "w96_9_units": (shape(96, 224, 4, 2, 129, S=1), True),
    "w96_2_passes_256_units": (shape(96, 224, 7, 1, 8192, S=1), True),
    "w96_2_passes_257_units": (shape(96, 224, 7, 1, 8193, S=1), False),
    "w96_2_passes_2559_units": (shape(96, 224, 5, 2, 40944, S=1), False),
    "w96_2_passes_2560_units": (shape(96, 224, 5, 2, 40945, S=1), True),
    "w96_3_passes_256_units": (shape(96, 416, 4, 1, 8192, S=1), True),
    "w96_3_passes_257_units": (shape(96, 416, 4, 1, 8193, S=1), False),
    "w96_4_passes_192_units": (shape(96, 672, 3, 3, 512, S=4, cf=1.0), True),
    "w96_4_passes_224_units": (shape(96, 672, 3, 1, 7168, S=1), True),
    "w96_4_passes_225_units": (shape(96, 672, 3, 1, 7169, S=1), False),
    "w96_4_passes_16_experts_193_units": (shape(96, 672, 16, 1, 6145, S=1), False),
    "w96_4_passes_prime_193_units": (shape(96, 608, 3, 1, 6145, S=1), True),
    "w96_5_passes": (shape(96, 800, 3, 2, 100, S=1), False),   # (k = 2: with one assignment the dropout makes every probability one)
}


@pytest.mark.parametrize("name", list(EDGES))
def test_both_sides_of_the_choice_against_64_bits(name):
    """Noise, dropout and the capacity loss, on the routing and the probabilities that the forward left behind.  The bars of the test above; of the router's
    gradients only the small cases are compared, a larger one has hidden units so close to zero that the two sides gate them differently."""
    import torch
    from paper_2510_04286_amd import binding as B
    case, onepass = EDGES[name]
    s, h, w = make_inputs(case)
    units, cus = (s.Na + 31) // 32, torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or split().chosen(s.ds, s.He, s.E, units, cus) == onepass
    cfg = B.config_of(s)
    assert B.slicemoe_backward_uses_mfma(cfg) == 1
    noise, drop_u = wl.make_router_draws(s)
    dout, alpha = wl.make_dout(s), 0.3 * s.Ns
    train = dict(temperature=TRAIN["tau"], noise_std=TRAIN["sigma"], dropout_rate=TRAIN["rate"], noise=torch.from_numpy(noise).to("cuda:0"),
                 drop_u=torch.from_numpy(drop_u).to("cuda:0"))
    hd, ws = B.to_device(h, s.dtype), B.alloc_workspace(cfg)
    wd = B.pack(cfg, B.weights_to_device(w, s.dtype))
    B.slicemoe_forward_train(cfg, hd, wd, torch.empty_like(hd), ws, **train)
    grads, d_h = B.alloc_weight_grads(cfg), torch.empty_like(hd)
    bws = torch.full((B.slicemoe_backward_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaNs: nothing is read unwritten
    B.slicemoe_backward(cfg, hd, wd, ws, B.to_device(dout, s.dtype), d_h, grads, bws, train=dict(train, capacity_alpha=alpha))
    torch.cuda.synchronize()
    v = {n: t.cpu().numpy() for n, t in B.workspace_views(cfg, ws).items() if n in ("topk_idx", "topk_p", "inv")}
    capg = oracle.capacity_surrogate(v["topk_idx"], v["topk_p"].astype(np.float64), s.E, alpha)["grad"]
    ref = oracle.backward(h, s.S, s.k, w, dout, v["topk_idx"], v["inv"], noise=noise, drop_u=drop_u, capg=capg, **TRAIN)
    small = s.Ns <= 1000
    bar = 2e-4 if s.ds == 96 else 5e-5
    err = {n: np.abs(grads[n].cpu().numpy() - ref[n]).max() / rms(ref[n]) for n in (NAMES if small else ("W1", "b1", "W2", "b2"))}
    print(f"\n[{name}] {units} units; " + " ".join(f"{n} {e:.1e}" for n, e in err.items()))
    assert max(err[n] for n in ("W1", "b1", "W2", "b2")) <= bar, err
    assert max(err.values()) <= 5e-4, err
    if small:
        got = d_h.float().cpu().numpy().astype(np.float64)
        excess = (np.abs(got - ref["d_h"]) / (2.0 ** -7 * np.abs(ref["d_h"]) + 2e-4 * rms(ref["d_h"]))).max()
        assert excess <= 1.0

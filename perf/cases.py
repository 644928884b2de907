"""The work that a program using this library has it do, as a set of measurable cases.

A case is one call (or one training step) of the SliceMoE layer through the entry points of
`paper_2510_04286_amd.binding`, at the sizes of `paper_2510_04286_amd.workload`: the benchmark layers, the paper's own
layer (d = 768, 16 experts) over its slice counts, and the fp32 layer.  Two modes:

    forward   inference: weights packed once when they were loaded, workspace kept; one slicemoe_forward
    train     one step's share of this layer: the weights have just been updated, so they are packed again, then the
              forward with the training-time router and the backward with every weight gradient

A case's fields: mode, layer (a key of workload.CONFIGS), T (tokens), k (experts per slice), dtype ("bf16" | "f32":
storage), capacity (capacity factor, 0 = dropless), skew (how unevenly the router favours the experts, see `prepare`),
and for training tau, sigma, rate, alpha (softmax temperature, logit-noise standard deviation, dropout rate,
capacity-loss weight).
"""
import math
from dataclasses import replace

import torch

from paper_2510_04286_amd import binding as B
from paper_2510_04286_amd import workload as wl

INFER = {"mode": "forward", "k": 2, "dtype": "bf16", "capacity": 0.0, "skew": 0.0}
TRAIN = {"mode": "train", "k": 2, "dtype": "bf16", "capacity": 0.0, "skew": 0.0, "tau": 1.0, "sigma": 0.1, "rate": 0.2,
         "alpha": 0.0}


def listed():
    return [
        # one decoding step of a batch of 32 sequences: a few hundred slices, launch latency
        {"name": "forward_decode", **INFER, "layer": "headline", "T": 32},
        # a language-model layer's batch: 4096 tokens, LayerNorm-scaled
        {"name": "forward_lm", **INFER, "layer": "lm", "T": 4096},
        # prefill at the benchmark's headline size
        {"name": "forward_headline", **INFER, "layer": "headline", "T": 16384},
        # a ragged batch under a capacity limit with a router that favours a few experts: rows are dropped
        {"name": "forward_capacity", **INFER, "layer": "headline", "T": 12289, "capacity": 1.25, "skew": 0.15},
        # the largest layer and batch of the benchmark
        {"name": "forward_large", **INFER, "layer": "large", "T": 65536},
        # the paper's layer cut into four slices (wide rows), an odd batch, three experts per slice
        {"name": "forward_paper_S4", **INFER, "layer": "paper_S4_k2", "T": 5001, "k": 3},
        # fp32 storage: the precise layer
        {"name": "forward_f32", **INFER, "layer": "tiny", "T": 512, "dtype": "f32"},
        # a training step at the headline size, with logit noise and cross-slice dropout
        {"name": "train_headline", **TRAIN, "layer": "headline", "T": 16384},
        # the paper's own training: eight slices, dropout 0.2, the capacity loss's gradient, an odd batch
        {"name": "train_paper", **TRAIN, "layer": "paper", "T": 8191, "sigma": 0.0, "alpha": 1.0},
        # its slice-count ablation at the narrow end: sixteen slices
        {"name": "train_paper_S16", **TRAIN, "layer": "paper_S16_k2", "T": 2048, "sigma": 0.0},
        # a training step of the largest layer on one micro-batch
        {"name": "train_large", **TRAIN, "layer": "large", "T": 16384},
        # fp32 storage, both directions
        {"name": "train_f32", **TRAIN, "layer": "tiny", "T": 1000, "dtype": "f32"},
    ]


# Token counts from a decoding step to a full batch, per mode and layer.  The upper ends keep every draw below the
# cost of the largest listed case.
RANGES = {
    "forward": {"headline": (1, 65536), "lm": (1, 65536), "large": (1, 32768), "paper": (1, 65536), "paper_S2_k2": (1, 16384),
                "paper_S4_k2": (1, 32768), "paper_S16_k2": (1, 65536), "paper_S32_k2": (1, 65536), "tiny": (1, 4096)},
    "train": {"headline": (64, 32768), "lm": (64, 32768), "large": (64, 8192), "paper": (64, 32768), "paper_S2_k2": (32, 1024),
              "paper_S4_k2": (32, 2048), "paper_S16_k2": (64, 4096), "paper_S32_k2": (64, 2048), "tiny": (32, 4096)},
}
WEIGHTS = {"headline": 5, "lm": 3, "large": 3, "paper": 3, "paper_S2_k2": 1, "paper_S4_k2": 1, "paper_S16_k2": 1,
           "paper_S32_k2": 1, "tiny": 3}


def draw(rng):
    mode = "forward" if rng.random() < 0.5 else "train"
    layers = sorted(RANGES[mode])
    layer = rng.choices(layers, [WEIGHTS[n] for n in layers])[0]
    lo, hi = RANGES[mode][layer]
    case = dict(INFER if mode == "forward" else TRAIN)
    case["layer"] = layer
    case["T"] = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    case["k"] = rng.choices([1, 2, 3], [1, 4, 1])[0]
    if case["k"] == 3:   # half as much expert work again
        case["T"] = max(lo, case["T"] * 2 // 3)
    case["dtype"] = "f32" if layer == "tiny" else "bf16"
    if rng.random() < 0.25:
        case["capacity"] = rng.choice([1.0, 1.25, 2.0])
        case["skew"] = rng.choice([0.0, 0.15])
    if mode == "train":
        case["tau"] = rng.choice([0.8, 1.0, 1.5])
        case["sigma"] = rng.choice([0.0, 0.1])
        case["rate"] = rng.choice([0.0, 0.2])
        case["alpha"] = rng.choice([0.0, 1.0])
    return case


def _shape(case):
    return replace(wl.CONFIGS[case["layer"]], T=case["T"], k=case["k"], dtype=case["dtype"], capacity_factor=case["capacity"])


def prepare(case, seed):
    """Hidden states ~ N(0, 1) (LayerNorm-scaled for the layers that are), Kaiming-uniform weights, standard-normal
    upstream gradients, the router's draws; with skew s the router's bias of expert e is lowered by s log(e + 1)."""
    shape = _shape(case)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32

    def normal(*size):
        return torch.randn(size, generator=gen, device=dev)

    def uniform(fan_in, *size):
        return ((2.0 * torch.rand(size, generator=gen, device=dev) - 1.0) / math.sqrt(fan_in)).to(dt)

    h = normal(shape.T, shape.d)
    if shape.layernorm:
        h = torch.nn.functional.layer_norm(h, (shape.d,))
    h = h.to(dt)
    ds, Hr, E, He = shape.ds, shape.Hr, shape.E, shape.He
    w = {"Wr1": uniform(ds, ds, Hr), "br1": uniform(ds, Hr), "Wr2": uniform(Hr, Hr, E), "br2": uniform(Hr, E),
         "W1": uniform(ds, E, ds, He), "b1": uniform(ds, E, He), "W2": uniform(He, E, He, ds), "b2": uniform(He, E, ds)}
    if case["skew"] > 0:
        ranks = torch.arange(1, E + 1, device=dev, dtype=torch.float32)
        w["br2"] = (w["br2"].float() - case["skew"] * ranks.log()).to(dt)

    cfg = B.config_of(shape)
    state = {"cfg": cfg, "h": h, "out": torch.empty_like(h), "ws": B.alloc_workspace(cfg), "w": B.pack(cfg, w)}
    state["stats"] = B.workspace_views(cfg, state["ws"])["stats"]
    if case["mode"] == "train":
        noise = normal(shape.Ns, E) if case["sigma"] > 0 else None
        drop_u = torch.rand((shape.Ns, shape.k), generator=gen, device=dev) if case["rate"] > 0 else None
        state["train"] = {"temperature": case["tau"], "noise_std": case["sigma"], "dropout_rate": case["rate"], "noise": noise,
                          "drop_u": drop_u, "capacity_alpha": case["alpha"]}
        state["d_out"] = normal(shape.T, shape.d).to(dt)
        state["d_h"] = torch.empty_like(h)
        state["grads"] = B.alloc_weight_grads(cfg)
        state["bws"] = torch.empty(B.slicemoe_backward_workspace_bytes(cfg), dtype=torch.uint8, device=dev)
    return state


def run(state):
    cfg, h, w, out, ws = state["cfg"], state["h"], state["w"], state["out"], state["ws"]
    if "train" not in state:
        B.slicemoe_forward(cfg, h, w, out, ws)
        return {"h_out": out, "stats": state["stats"]}
    if "packed" in w:   # the optimizer has changed the weights since the last step
        B.slicemoe_pack_weights(cfg, w, w["packed"])
    B.slicemoe_forward_train(cfg, h, w, out, ws, **state["train"])
    B.slicemoe_backward(cfg, h, w, ws, state["d_out"], state["d_h"], state["grads"], state["bws"], train=state["train"])
    return {"h_out": out, "stats": state["stats"], "d_h": state["d_h"], **state["grads"]}


def work(case):
    """Inputs read once, outputs written once; contractions over the assignments that are kept."""
    s = _shape(case)
    ds, Hr, E, He = s.ds, s.Hr, s.E, s.He
    el = 2 if s.dtype == "bf16" else 4
    # under a capacity limit: the share of the assignments that the skewed router keeps at factor 1.25 (measured)
    kept = s.Na * (1.0 if case["capacity"] <= 0 else 0.46)
    weights = ds * Hr + Hr + Hr * E + E + E * (2 * ds * He + He + ds)
    nbytes = 2 * s.T * s.d * el + weights * el
    flops = s.Ns * 2 * (ds * Hr + Hr * E) + kept * 4 * ds * He
    if case["mode"] == "train":
        nbytes += 2 * s.T * s.d * el + weights * 4
        nbytes += s.Ns * E * 4 if case["sigma"] > 0 else 0
        nbytes += s.Na * 4 if case["rate"] > 0 else 0
        # dL/d(hidden) and dL/dx of both networks, and both layers' weight gradients
        flops += s.Ns * 8 * (ds * Hr + Hr * E) + kept * 8 * ds * He
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """Against the layer in 64-bit arithmetic (same routing) the bf16 layer measures 2.2e-3 (h', dL/dh: one bf16 rounding
    and the fp16 activation), the fp32 layer 4e-7."""
    return {"rel": 8e-3 if case["dtype"] == "bf16" else 1e-5}

"""The work that users of this framework have it do, as measurable cases: training steps (forward and backward)
and evaluation passes (forward only) of one GPU's MoE layer through `MoELayer`.

A case names a layer shape (T tokens, d_model, d_ff, E experts, top-k), the capacity factor, the element type and
activation, how skewed the gate is, whether tokens carry Random-Token-Selection keys, and the training options that
the paper uses (balancing loss, gate jitter, expert dropout, grouped selection).  Weights, the layer with its
buffers and the routing bias are what a program keeps between passes; tokens, keys and upstream gradients are its
inputs.  Everything is made from the seed on the GPU.
"""
import functools
import math

import torch

from paper_2109_10465_amd import binding as B
from paper_2109_10465_amd import inputs as I
from paper_2109_10465_amd.layer import MoELayer

_DTYPES = {"f32": (B.F32, torch.float32), "bf16": (B.BF16, torch.bfloat16)}
_ACTS = {"relu": B.RELU, "gelu": B.GELU}
_DEFAULTS = {"mode": "train", "dtype": "bf16", "act": "gelu", "k": 2, "cf": 1.0, "w_std": 0.02, "skew": "none",
             "skew_param": 0.0, "keys": True, "groups": 1, "aux_coef": 0.0, "jitter_eps": 0.0, "drop_p": 0.0}


def _case(**over):
    return {**_DEFAULTS, **over}


def listed():
    return [
        # The tiny layer of the unit tests and of debugging runs: launches and latency are all there is.
        _case(name="train_f32_tiny", dtype="f32", act="relu", T=256, d=64, f=256, E=4, k=1),
        # fp32 training on a batch that fits no tile: position priority instead of keys, one hot expert.
        _case(name="train_f32_ragged", dtype="f32", T=777, d=136, f=328, E=5, cf=1.25, skew="hot0", skew_param=0.5,
              keys=False),
        # fp32 training at an ordinary size, one expert drawing 30 % of the tokens.
        _case(name="train_f32_top2", dtype="f32", T=4096, d=512, f=2048, E=8, cf=1.25, skew="hot0", skew_param=0.3),
        # A small bf16 micro-batch of a small model.
        _case(name="train_bf16_small", act="relu", T=512, d=512, f=2048, E=8, k=1),
        # bf16 training on sizes that are no multiple of any tile, popular and unpopular experts.
        _case(name="train_bf16_ragged", T=5003, d=776, f=3080, E=6, cf=1.25, skew="zipf", skew_param=1.1),
        # Fine-tuning with everything on: balancing loss, jitter, expert dropout, selection inside groups.
        _case(name="finetune_bf16_options", T=8192, d=768, f=3072, E=16, groups=8, aux_coef=0.01, jitter_eps=0.01,
              drop_p=0.4),
        # The headline training step: 16 sequences of 1024 tokens, 32 experts, balanced gate.
        _case(name="train_bf16_top2_e32", T=16384, d=1024, f=4096, E=32),
        # Many experts, top-1, Zipf-skewed: most experts are nearly empty, some overflow.
        _case(name="train_bf16_top1_e128", T=32768, d=1024, f=4096, E=128, k=1, skew="zipf", skew_param=1.1),
        # The largest: a big per-GPU share of wide experts, nothing dropped.
        _case(name="train_bf16_large", T=65536, d=2048, f=8192, E=16, cf=2.0, w_std=0.01),
        # Evaluation over a full validation batch (capacity factor 2.0, utilisation counted).
        _case(name="eval_bf16_top2_e32", mode="eval", T=16384, d=1024, f=4096, E=32, cf=2.0),
        # Evaluation of one short batch: an odd number of sentences' last tokens, every expert nearly empty.
        _case(name="eval_bf16_few_tokens", mode="eval", T=61, d=1024, f=4096, E=32, cf=2.0),
        # Evaluation of a ragged last batch with many experts.
        _case(name="eval_bf16_top1_e128", mode="eval", T=1511, d=1024, f=4096, E=128, k=1, cf=2.0, skew="zipf",
              skew_param=1.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_mult8(rng, lo, hi):
    return max(8, 8 * int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 8)))


def draw(rng):
    """One more case of the same ranges: fp32 training of small layers, bf16 training from micro-batches to the large
    share, bf16 evaluation from a few tokens to a full batch."""
    while True:
        kind = rng.choice(("train_f32", "train_bf16", "train_bf16", "eval_bf16"))
        c = _case(k=rng.choice((1, 2)), act=rng.choice(("gelu", "gelu", "relu")), cf=rng.choice((1.0, 1.25, 2.0)))
        if kind == "train_f32":
            c.update(dtype="f32", T=_log_int(rng, 256, 4096), d=_log_mult8(rng, 64, 512), E=_log_int(rng, 4, 16))
        elif kind == "train_bf16":
            c.update(T=_log_int(rng, 512, 65536), d=_log_mult8(rng, 512, 2048), E=_log_int(rng, 6, 128))
        else:
            c.update(mode="eval", cf=2.0, T=_log_int(rng, 61, 16384), d=_log_mult8(rng, 512, 2048), E=_log_int(rng, 8, 128))
        c["f"] = 8 * int(round(c["d"] * rng.uniform(2.4, 4.0) / 8))
        skew = rng.choice(("none", "hot0", "zipf"))
        if skew != "none":
            c.update(skew=skew, skew_param=rng.uniform(0.3, 0.5) if skew == "hot0" else 1.1)
        c["keys"] = rng.random() < 0.75
        if kind == "train_bf16" and rng.random() < 0.3:        # the fine-tuning options, groups where T allows them
            c.update(aux_coef=0.01, jitter_eps=0.01, drop_p=0.4)
            if rng.random() < 0.5 and c["T"] >= 1024:
                c["groups"] = rng.choice((2, 4))
                c["T"] -= c["T"] % (256 * c["groups"])
        # no more work, weights or buffers than the largest listed cases have
        if (_kept_rows(c) * c["d"] * c["f"] <= 1.2e5 * 2048 * 8192 and c["E"] * c["d"] * c["f"] <= 128 * 1024 * 4096
                and c["E"] * _capacity(c) * c["f"] <= 16 * 16384 * 8192):
            return c


def _capacity(c):
    """Slots per expert, rounded up so that every group gets the same number."""
    cap = max(1, math.ceil(c["k"] * c["cf"] * c["T"] / c["E"]))
    return -(-cap // c["groups"]) * c["groups"]


@functools.lru_cache(maxsize=64)
def _bias(E, d, w_std, skew, param, seed):
    w = I.small("case", 1, d, 8, E, 1, 1, w_std=w_std, skew=skew, skew_param=param)
    return I.gate_bias(w, seed)


def prepare(case, seed):
    c = case
    dtype, tdt = _DTYPES[c["dtype"]]
    T, d, f, E = c["T"], c["d"], c["f"], c["E"]
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    train = c["mode"] == "train"

    def normal(*shape, std=1.0, dt=tdt):
        t = torch.randn(*shape, generator=g, device=dev, dtype=torch.float32)
        return (t.mul_(std) if std != 1.0 else t).to(dt)

    def stack(rows, cols):      # expert by expert: the fp32 draws of all experts at once need not fit beside the rest
        t = torch.empty(E, rows, cols, device=dev, dtype=tdt)
        for e in range(E):
            t[e] = normal(rows, cols, std=c["w_std"])
        return t

    bias = _bias(E, d, c["w_std"], c["skew"], c["skew_param"], 0)
    state = {
        "x": normal(T, d), "Wg": normal(d, E, std=c["w_std"], dt=torch.float32),
        "bias": None if bias is None else torch.from_numpy(bias).to(dev),
        "W1": stack(d, f), "W2": stack(f, d),
        "keys": torch.rand(T, generator=g, device=dev) if c["keys"] else None,
        "dy": normal(T, d) if train else None,
        "seed": seed,
        "layer": MoELayer(T, d, f, E, c["k"], _capacity(c), dtype, _ACTS[c["act"]], device="cuda:0",
                          aux_coef=c["aux_coef"], forward_only=not train, groups=c["groups"],
                          jitter_eps=c["jitter_eps"], drop_p=c["drop_p"]),
    }
    return state


def run(state):
    s, layer = state, state["layer"]
    y = layer.forward(s["x"], s["Wg"], s["bias"], s["W1"], s["W2"], s["keys"], seed=s["seed"])
    if layer.forward_only:
        return {"y": y, "expert_demand": layer.expert_demand}
    dx, dWg, dW1, dW2 = layer.backward(s["dy"])
    out = {"y": y, "dx": dx, "dWg": dWg, "dW1": dW1, "dW2": dW2}
    if layer.aux_coef != 0.0:
        out["aux_loss"] = layer.aux_loss
    return out


def _demand(c):
    """Expected candidates per expert, from the gate's skew."""
    E, T = c["E"], c["T"]
    if c["skew"] == "hot0":
        q = [c["skew_param"]] + [(1.0 - c["skew_param"]) / (E - 1)] * (E - 1)
    elif c["skew"] == "zipf":
        q = [(r + 1.0) ** -c["skew_param"] for r in range(E)]
        q = [v / sum(q) for v in q]
    else:
        q = [1.0 / E] * E
    if c["k"] == 1:
        return [T * v for v in q]
    odds = sum(v / (1.0 - v) for v in q)
    return [T * (v + v * (odds - v / (1.0 - v))) for v in q]


def _kept_rows(c):
    """Expected rows in use over all experts: the mean of min(demand, capacity), demand taken as normal."""
    C, rows = float(_capacity(c)), 0.0
    for mu in _demand(c):
        sd = math.sqrt(max(mu, 1e-9))
        a = (C - mu) / sd
        rows += C - (C - mu) * 0.5 * (1.0 + math.erf(a / math.sqrt(2.0))) - sd * math.exp(-0.5 * min(a * a, 1400.0)) / math.sqrt(2.0 * math.pi)
    return max(1.0, rows)


def work(case):
    """Bytes: tokens in and out, the weights of the experts that get rows, and in training every weight gradient
    (fp32, written for every expert).  Flops: two products per kept row forward, four more backward, and the gate's."""
    c = case
    T, d, f, E, s = c["T"], c["d"], c["f"], c["E"], 2 if c["dtype"] == "bf16" else 4
    touched = sum(1.0 - math.exp(-mu) for mu in _demand(c))
    n = 2 * T * d * s + 2 * touched * d * f * s + 4 * d * E + (4 * T if c["keys"] else 0)
    products, gates = 2, 1
    if c["mode"] == "train":
        n += 2 * T * d * s + 8 * E * d * f + 4 * d * E
        products, gates = 6, 3
    return {"bytes": n, "flops": 2.0 * products * _kept_rows(c) * d * f + 2.0 * gates * T * d * E}


def tolerance(case):
    """Every output of the listed cases compared with the same layer in 64 bits on the same routing: fp32 outputs are
    1.8e-7 .. 9.4e-7 away from it, bf16 outputs 2.3e-3 .. 3.7e-3 (they are rounded to 8 bits, and so are the hidden
    activation, its derivative and the per-expert rows on the way)."""
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 5e-6}

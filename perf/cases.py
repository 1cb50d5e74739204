"""What a user of this package has it do, as cases that can be timed.

A case is one pass of a serving or evaluation program through the public entry
points (paper_2308_15030_amd.binding): decode steps, prompts of every size,
expert swaps, in bf16 and in fp32, at the MoE-layer shapes of the repository's
workloads (workloads.CONFIGS) and between them.  `prepare` makes what such a
program holds before the call -- loaded layers and hidden states -- and `run`
is the pass itself.

Kinds of pass
  forward   one smoe_forward per stacked layer (bf16): prefill or a decode step
  calls     the five per-step calls per stacked layer: the only form fp32 layers
            have, and what a program uses that looks between the steps
  period    decode steps of two update periods, each followed by the update of
            the resident set on the device (smoe_update_on_device)
  swap      experts loaded into slots with smoe_set_resident, then a decode
            step; twice, the second time other experts into the same slots

The hidden states of stacked layers are drawn independently: in a model,
attention and dense blocks stand between two MoE layers.  They come from the
mixture that workloads.py describes (Gaussian clusters with Zipf frequencies),
made on the GPU here so that it takes milliseconds.
"""
from __future__ import annotations

import math

import torch

from paper_2308_15030_amd import binding as b

_SIGMA, _ZIPF, _W_STD = 0.5, 1.1, 0.02


def _case(**kw):
    c = dict(kind="forward", dtype="bf16", E=64, K=16, d_model=768, d_ff=3072, T=32, layers=1, gate="full",
             residual=True, spare=0, steps=1, loads=0, bank="device")
    c.update(kw)
    return c


def listed():
    return [
        # the tiny fp32 layer (workload c1): five calls on a few hundred kilobytes, all latency
        _case(name="tiny-fp32", kind="calls", dtype="f32", E=8, K=2, d_model=64, d_ff=256, T=256, residual=False),
        # interactive decoding of a single sequence through the six MoE layers of Switch-base-64
        _case(name="decode-1", T=1, layers=6),
        # a half-filled decode batch, a tighter memory budget, renormalised gates, a spare slot for later swaps
        _case(name="decode-13", T=13, K=10, layers=6, gate="renorm", spare=1),
        # the decode workload (c4): 32 sequences, resident set updated every 16 steps
        _case(name="decode-32-updates", kind="period", T=32, steps=16, residual=False),
        # the paper's own setting, experts in external memory: swaps from a pinned host bank between steps
        _case(name="decode-32-swaps-pinned", kind="swap", T=32, loads=2, bank="pinned"),
        # a short prompt, or a large decode batch, on a 32-expert model
        _case(name="prompt-100", E=32, K=8, T=100, layers=6),
        # a prefill chunk of odd length
        _case(name="chunk-777", T=777, layers=2, gate="renorm"),
        # widths and counts that fit no tile: odd expert count, d_model and d_ff no multiples of 64
        _case(name="ragged-1213", E=33, K=11, d_model=416, d_ff=1696, T=1213, layers=2, residual=False),
        # Switch-base-8 prefill (c2) through the separate calls
        _case(name="base8-calls-4096", kind="calls", E=8, K=4, T=4096),
        # the headline workload (c3): Switch-base-64 prefill, six layers
        _case(name="base64-prefill-4096", T=4096, layers=6),
        # Switch-large-128 prefill (c5), four of its layers
        _case(name="large128-prefill-16384", E=128, K=32, d_model=1024, d_ff=4096, T=16384, layers=4),
        # evaluation in fp32 at the Switch-base width
        _case(name="base8-fp32-512", kind="calls", dtype="f32", E=8, K=4, T=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "calls", "fp32", "period", "swap"])
    E = rng.choice([8, 16, 24, 32, 33, 64, 64, 100, 128])
    K = min(32, _log_int(rng, 2, max(2, E // 2)))
    d, f = rng.choice([(768, 3072), (768, 3072), (1024, 4096), (768, 2048), (512, 2048),
                       (32 * rng.randint(8, 32), 32 * rng.randint(24, 128))])
    c = _case(E=E, K=K, d_model=d, d_ff=f, gate=rng.choice(["full", "renorm"]), residual=rng.random() < 0.7,
              spare=rng.choice([0, 0, 1]))
    if kind == "decode":
        c.update(T=_log_int(rng, 1, 32), layers=rng.randint(1, 6))
    elif kind == "prefill":
        T = _log_int(rng, 33, 16384)
        c.update(T=T, layers=rng.randint(1, 6 if T <= 4096 else 2))
    elif kind == "calls":
        c.update(kind="calls", T=_log_int(rng, 1, 8192), layers=rng.randint(1, 2))
    elif kind == "fp32":
        d = 4 * _log_int(rng, 16, 192)
        c.update(kind="calls", dtype="f32", d_model=d, d_ff=4 * d - 4 * rng.randint(0, 5), T=_log_int(rng, 1, 1024),
                 E=min(E, 32), K=min(K, 8))
    elif kind == "period":
        c.update(kind="period", T=_log_int(rng, 1, 32), steps=rng.choice([4, 8, 16]))
    else:
        c.update(kind="swap", T=_log_int(rng, 1, 32), loads=rng.randint(1, min(4, K)),
                 bank=rng.choice(["device", "pinned"]), E=max(E, 16), K=min(K, 16))
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _act(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _mixture(c, g, dev):
    """Cluster centres and frequencies of the layer stack's hidden states."""
    n = max(16, c["E"] // 2)
    mu = torch.randn(n, c["d_model"], device=dev, generator=g)
    p = torch.arange(1, n + 1, device=dev, dtype=torch.float32).pow(-_ZIPF)
    return mu, p / p.sum()


def _states(c, mu, cur, g):
    x = mu[cur]
    return (x + _SIGMA * torch.randn(x.shape, device=x.device, generator=g)).to(_act(c))


def _experts(c, n, g, dev):
    d, f = c["d_model"], c["d_ff"]
    w = [torch.randn(n, *s, device=dev, generator=g, dtype=_act(c)).mul_(_W_STD) for s in ((d, f), (f, d))]
    return w[0], w[1]


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    L, T, E, K, d, act = c["layers"], c["T"], c["E"], c["K"], c["d_model"], _act(c)
    mu, p = _mixture(c, g, dev)
    nx = {"period": 2 * c["steps"], "swap": 2}.get(c["kind"], L)        # hidden states of one pass
    if c["kind"] == "period":      # sequences hold a cluster and leave it now and then; two periods of a drifting stream
        rows = []
        for s in range(nx):
            fresh = torch.multinomial(p, T, replacement=True, generator=g)
            if s % c["steps"] == 0:
                cur = fresh
            else:
                cur = torch.where(torch.rand(T, device=dev, generator=g) < 1 / 32, fresh, cur)
            rows.append(cur)
        cur = torch.stack(rows)
    else:
        cur = torch.multinomial(p, nx * T, replacement=True, generator=g).view(nx, T)
    x = _states(c, mu, cur, g)
    out = torch.empty_like(x)
    # per-token and per-expert results of every layer (or of the last step), one tensor per kind
    i32, f32 = torch.int32, torch.float32
    shapes = {"orig_expert": (i32, T), "orig_gate": (f32, T), "slot": (i32, T), "gate": (f32, T), "xnorm": (f32, T),
              "count": (i32, E), "gsum": (f32, E), "score": (f32, E), "perm": (i32, T), "inv_perm": (i32, T),
              "offsets": (i32, K + 1)}
    results = {k: torch.zeros(L, n, dtype=t, device=dev) for k, (t, n) in shapes.items()}
    layers, bank = [], None
    for i in range(L):
        router = _W_STD * torch.randn(E, d, device=dev, generator=g)
        held = E if c["kind"] == "period" else K
        w1, w2 = _experts(c, held, g, dev)
        lay = b.Layer(E, K, d, c["d_ff"], T, b.SMOE_BF16 if act == torch.bfloat16 else b.SMOE_F32,
                      b.SMOE_GATE_RENORM if c["gate"] == "renorm" else b.SMOE_GATE_FULL, router_w=router,
                      device=dev, spare_slots=c["spare"])
        lay.expert_norm[:held].copy_(lay.expert_norm_of(w1, w2))
        for s in range(K):
            lay.set_resident(s, s, w1[s], w2[s])
        for k, v in results.items():
            setattr(lay, k, v[i])
        layers.append(lay)
        if c["kind"] == "period":
            bank = (w1, w2)
    loads = []
    if c["kind"] == "swap":        # two sets of newcomers for the first slots: experts K.., then the first occupants again
        n = c["loads"]
        w1, w2 = _experts(c, 2 * n, g, dev)
        if c["bank"] == "pinned":
            h1, h2 = (torch.empty(w.shape, dtype=w.dtype, pin_memory=True).copy_(w) for w in (w1, w2))
            w1, w2 = h1, h2
        newcomers = [e for e in range(K, E)][:n]
        loads = [[(s, newcomers[s], w1[s], w2[s]) for s in range(len(newcomers))],
                 [(s, s, w1[n + s], w2[n + s]) for s in range(len(newcomers))]]
    xs, outs = list(x.unbind(0)), list(out.unbind(0))
    return {"case": c, "layers": layers, "x": xs, "outs": outs, "res": xs if c["residual"] else [None] * nx, "bank": bank,
            "loads": loads, "returned": dict(results, out=out)}


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(state):
    c, T = state["case"], state["case"]["T"]
    xs, outs, res = state["x"], state["outs"], state["res"]
    if c["kind"] == "forward":
        for lay, x, o, r in zip(state["layers"], xs, outs, res):
            lay.forward_fused(x, T, accumulate=0, residual=r, out=o)
    elif c["kind"] == "calls":
        for lay, x, o, r in zip(state["layers"], xs, outs, res):
            lay.forward(x, T, accumulate=0, residual=r, out=o)
    elif c["kind"] == "period":
        lay, n = state["layers"][0], c["steps"]
        for s in range(2 * n):
            lay.forward_fused(xs[s], T, accumulate=int(s % n != 0), residual=res[s], out=outs[s])
            if s % n == n - 1:
                lay.update_on_device(*state["bank"])
    else:
        lay = state["layers"][0]
        for s in range(2):
            for slot, expert, w1, w2 in state["loads"][s]:
                lay.set_resident(slot, expert, w1, w2)
            lay.forward_fused(xs[s], T, accumulate=s, residual=res[s], out=outs[s])
    return state["returned"]


def work(case):
    """Every slot that can have a token streams its expert's two matrices once per layer or step; a swapped expert is
    read from the bank and written to its slot; x, residual and out once each; the router once."""
    c = case
    T, E, K, d, f = c["T"], c["E"], c["K"], c["d_model"], c["d_ff"]
    size = 2 if c["dtype"] == "bf16" else 4
    active = K * (1.0 - (1.0 - 1.0 / K) ** T)              # slots with at least one of T tokens, if they are spread evenly
    one = 2 * d * f * size
    passes = {"period": 2 * c["steps"], "swap": 2}.get(c["kind"], c["layers"])
    per = active * one + (2 + bool(c["residual"])) * T * d * size + 4 * E * d + 40 * T
    swapped = 2 * min(c["loads"], E - K) if c["kind"] == "swap" else 0
    return {"bytes": passes * per + swapped * 2 * one, "flops": passes * (4.0 * T * d * f + 2.0 * T * d * E)}


def tolerance(case):
    """Whole numbers are exact.  bf16: the hidden activations and the output are each rounded to 8 bits of mantissa, and
    another order of the sums moves some of those roundings by one unit; fp32: sums of at most a few thousand terms."""
    return {"rel": 5e-3, "max": 0.03} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-4}

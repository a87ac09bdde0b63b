"""The work a user of this library has it do, as cases to be timed: forwards of MoTE layers from one
token to long prompts, a whole block, and what training and conversion call beside them (ternary and
round-to-nearest packing, the load-balancing statistic, straight-through gradients).

Widths, expert counts and loads are those of workloads.py and of the tests; weights and inputs are
drawn on the device from the seed with the distributions of workloads.py.  A case is a dict of plain
values; `kind` says which entry point it calls.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2506_14435_amd as M

# (d_model, d_ff, std of the shared expert's weights) of the configurations in workloads.py: tiny, and the
# 0.5B / 1.5B / 3B / 7B widths
WIDTHS = ((256, 512, 0.02), (896, 4864, 0.012), (1536, 8960, 0.012), (2048, 11008, 0.015), (3584, 18944, 0.01))
SIGMA_SHARED = {d: s for d, _, s in WIDTHS}
SIGMA_LATENT = 0.02


def _layer(name, d, f, e, k, t, bits=0, load="even", distinct=0, kind="layer"):
    """bits: 0 for the bf16 shared expert, 8 / 4 for its RTN codes.  load: how the router spreads tokens
    ("even", "zipf", or "subset": only `distinct` experts can be selected)."""
    return dict(name=name, kind=kind, d=d, f=f, e=e, k=k, t=t, bits=bits, load=load, distinct=distinct)


def listed():
    return [
        # one short request to a small layer: nothing but launches and latency
        _layer("tiny_T64", 256, 512, 4, 2, 64),
        # token-by-token generation for one user: two experts and the shared expert are streamed
        _layer("decode_3b_T1", 2048, 11008, 16, 2, 1, load="subset", distinct=2),
        # the same for a full decode batch: every expert is streamed
        _layer("decode_3b_T64", 2048, 11008, 16, 2, 64, load="subset", distinct=16),
        # a few users on a memory-limited server: INT4 shared expert (Section 4.3)
        _layer("decode_3b_T4_int4", 2048, 11008, 16, 2, 4, bits=4, load="subset", distinct=4),
        # a chunk of a prompt, of no round length: experts see some 60 rows each
        _layer("chunk_3b_T500", 2048, 11008, 16, 2, 500),
        # a 2048-token sequence through the small model's layer (outlier channels in x)
        _layer("prefill_0.5b_T2048", 896, 4864, 8, 2, 2048),
        # one sequence through the paper's own layer as a block: RMSNorm in front, residual behind, top-1 of four
        _layer("block_3b_top1_T2048", 2048, 11008, 4, 1, 2048, kind="block"),
        # a batch of prompts
        _layer("prefill_3b_T8192", 2048, 11008, 16, 2, 8192),
        # the largest: a big batch through the widest layer, experts loaded unevenly (about 10x)
        _layer("prefill_7b_zipf_T16384", 3584, 18944, 16, 2, 16384, load="zipf"),
        # training: the latent fp32 weights of one expert matrix are ternarised anew in every step
        dict(name="pack_3b_f32", kind="pack", n_out=11008, n_in=2048, dtype="f32", binary=False),
        # training: router with the load-balancing statistic over a batch of four sequences
        dict(name="balance_3b_T8192", kind="balance", d=2048, e=16, k=2, t=8192),
        # training: gradients of the gate matrices of all experts for the same batch
        dict(name="ste_3b_R16384", kind="ste", rows=16384, n_out=11008, n_in=2048, e=16, load="even"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("layer",) * 8 + ("block",) * 2 + ("pack", "pack", "rtn_pack", "balance", "ste", "ste"))
    d, f, _ = rng.choice(WIDTHS)
    f -= 128 * rng.randrange(0, f // 1024 + 1)      # hidden widths are any multiple of 128
    if kind in ("pack", "rtn_pack"):
        n_out, n_in = (f, d) if rng.random() < 0.67 else (d, f)
        if kind == "pack":
            return dict(kind=kind, n_out=n_out, n_in=n_in, dtype=rng.choice(("f32", "f32", "bf16")),
                        binary=rng.random() < 0.2)
        return dict(kind=kind, n_out=n_out, n_in=n_in, bits=rng.choice((8, 4)))
    e = rng.choice((4, 8, 16, 16, 64))
    if kind == "balance":
        return dict(kind=kind, d=d, e=e, k=rng.choice((1, 2, 2, min(e, 8))), t=_log_int(rng, 256, 16384))
    if kind == "ste":
        n_out, n_in = (f, d) if rng.random() < 0.67 else (d, f)
        rows = _log_int(rng, 64, 16384 if d < 3584 else 8192)
        return dict(kind=kind, rows=rows, n_out=n_out, n_in=n_in, e=min(e, 16), load=rng.choice(("even", "zipf")))
    if d > 2048:
        e = min(e, 16)
    t = _log_int(rng, 1, 16384 if d < 3584 else 8192)
    load = rng.choice(("even", "even", "zipf", "subset"))
    case = _layer(None, d, f, e, rng.choice((1, 2, 2)), t, bits=rng.choice((0, 0, 0, 8, 4)), load=load,
                  distinct=rng.randrange(2, e + 1) if load == "subset" else 0, kind=kind)
    del case["name"]
    return case


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(g, *shape, std=1.0):
    return torch.randn(*shape, device="cuda", generator=g) * std


def _zipf_bias(e, rs):
    """The skewed load of workloads.py: -0.45 * 1.2 * ln(rank), ranks dealt to the experts at random."""
    return (-0.45 * 1.2 * np.log(1.0 + rs.permutation(e))).astype(np.float32)


def _hidden(g, t, d):
    x = _randn(g, t, d)
    if d == 896:      # the 0.5B configuration: four outlier channels, twenty times as large
        x[:, torch.randperm(d, device="cuda", generator=g)[:4]] *= 20.0
    return x.to(torch.bfloat16)


def _router(g, d, e):
    return _randn(g, d, e, std=d ** -0.5).to(torch.bfloat16)


def _prepare_layer(c, seed):
    g, rs = _gen(seed), np.random.RandomState(seed % (1 << 32))
    d, f, e = c["d"], c["f"], c["e"]
    bias = None
    if c["load"] != "even":
        if c["load"] == "zipf":
            b = _zipf_bias(e, rs)
        else:
            b = np.zeros(e, np.float32)
            b[rs.permutation(e)[:c["distinct"]]] = 30.0
        bias = torch.from_numpy(b).cuda()
    shared, scales = [], None
    for shape in ((f, d), (f, d), (d, f)):
        shared.append(_randn(g, *shape, std=SIGMA_SHARED[d]).to(torch.bfloat16))
    if c["bits"]:
        packed = [M.mote_pack_rtn(w, c["bits"]) for w in shared]
        shared, scales = [p for p, _ in packed], tuple(s for _, s in packed)
    wt = [torch.empty(e, d * f // 16, dtype=torch.int32, device="cuda") for _ in range(3)]
    alpha = torch.empty(3, e, 1, dtype=torch.float32, device="cuda")
    for ex in range(e):
        for m in range(3):
            shape = (f, d) if m < 2 else (d, f)
            M.mote_pack_ternary(_randn(g, *shape, std=SIGMA_LATENT), packed=wt[m][ex], alpha=alpha[m, ex])
    layer = M.MoteLayer(_router(g, d, e), *shared, *wt, alpha[:, :, 0].t().contiguous(), c["k"], router_bias=bias,
                        shared_bits=c["bits"], shared_scales=scales)
    layer.workspace(c["t"])
    state = dict(kind=c["kind"], layer=layer, x=_hidden(g, c["t"], d))
    if c["kind"] == "block":
        state["x"] = (state["x"].float() * 3.0 + 0.25).to(torch.bfloat16)     # a hidden state before its norm
        state["gamma"] = (1.0 + _randn(g, d, std=0.1)).to(torch.bfloat16)
    return state


def _prepare_ste(c, seed):
    g, rs = _gen(seed), np.random.RandomState(seed % (1 << 32))
    n, k, e, r = c["n_out"], c["n_in"], c["e"], c["rows"]
    share = np.exp(_zipf_bias(e, rs)) if c["load"] == "zipf" else np.ones(e)
    counts = rs.multinomial(r, share / share.sum())
    packed = torch.empty(e, n * k // 16, dtype=torch.int32, device="cuda")
    alpha = torch.empty(e, 1, dtype=torch.float32, device="cuda")
    for ex in range(e):
        M.mote_pack_ternary(_randn(g, n, k, std=SIGMA_LATENT), packed=packed[ex], alpha=alpha[ex])
    need = M.load_library().mote_ste_backward_workspace_bytes(r, n, k, e)
    return dict(kind="ste", dy=_randn(g, r, n).to(torch.bfloat16), offsets=[0] + np.cumsum(counts).tolist(),
                packed=packed, alpha=alpha, n_out=n, n_in=k,
                q=torch.randint(-127, 128, (r, k), device="cuda", generator=g, dtype=torch.int8),
                beta=torch.rand(r, device="cuda", generator=g) * 4 + 1,
                workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in ("layer", "block"):
        return _prepare_layer(c, seed)
    if kind == "ste":
        return _prepare_ste(c, seed)
    g = _gen(seed)
    if kind == "balance":
        return dict(kind=kind, x=_hidden(g, c["t"], c["d"]), w_router=_router(g, c["d"], c["e"]), k=c["k"])
    if kind == "rtn_pack":
        w = _randn(g, c["n_out"], c["n_in"], std=SIGMA_LATENT).to(torch.bfloat16)
        return dict(kind=kind, w=w, bits=c["bits"])
    w = _randn(g, c["n_out"], c["n_in"], std=SIGMA_LATENT)
    return dict(kind=kind, w=w.to(torch.bfloat16) if c["dtype"] == "bf16" else w, binary=c["binary"])


def run(state):
    s, kind = state, state["kind"]
    if kind == "layer":
        return M.mote_layer_forward(s["layer"], s["x"])
    if kind == "block":
        return M.mote_block_forward(s["layer"], s["x"], s["gamma"])
    if kind == "ste":
        return M.mote_ste_linear_backward(s["dy"], s["offsets"], s["packed"], s["alpha"], 1, s["q"], s["beta"],
                                          s["n_out"], s["n_in"], workspace=s["workspace"])
    if kind == "balance":
        return M.mote_router_balance(s["x"], s["w_router"], s["k"])
    if kind == "rtn_pack":
        return M.mote_pack_rtn(s["w"], s["bits"])
    return M.mote_pack_ternary(s["w"], binary=s["binary"])


def work(case):
    c, kind = case, case["kind"]
    if kind in ("layer", "block"):
        t, d, f, e, k = c["t"], c["d"], c["f"], c["e"], c["k"]
        active = min(c["distinct"] or e, t * k)
        weights = active * 3 * d * f / 4 + 3 * d * f * (c["bits"] or 16) / 8 + 2 * d * e
        return dict(bytes=weights + 4 * t * d, flops=6.0 * t * d * f * (k + 1))
    if kind == "ste":
        r, n, k, e = c["rows"], c["n_out"], c["n_in"], c["e"]
        return dict(bytes=2 * r * n + r * k + e * n * k / 4 + 4 * r * k + 4 * e * n * k, flops=4.0 * r * n * k)
    if kind == "balance":
        t, d, e = c["t"], c["d"], c["e"]
        return dict(bytes=2 * t * d + 2 * d * e + 4 * t * e + 8 * t * c["k"], flops=2.0 * t * d * e)
    n = c["n_out"] * c["n_in"]
    if kind == "rtn_pack":
        return dict(bytes=2 * n + n * c["bits"] / 8 + 4 * c["n_out"], flops=2.0 * n)
    return dict(bytes=n * (2 if c["dtype"] == "bf16" else 4) + n / 4, flops=3.0 * n)


def tolerance(case):
    """About four times the largest difference seen over the ranges above."""
    kind = case["kind"]
    if kind in ("pack", "rtn_pack"):
        return "exact"        # codes and scales are defined to the bit
    if kind == "balance":     # fp32 roundings of fp64 values: 2.6e-8 and 6.0e-8 against fp64
        return {"rel": 1e-7, "max": 2.4e-7}
    if kind == "ste":         # fp32 sums of exact products: 1.6e-7 and 1.6e-6 against fp64
        return {"rel": 6e-7, "max": 6.4e-6}
    # bf16 outputs, and bf16 / int8 hidden values that may round the other way: 3.3e-4 and one unit in the
    # last place (7.8e-3) with the channels of x and of the hidden layer in another order
    return {"rel": 1.3e-3, "max": 3.1e-2}

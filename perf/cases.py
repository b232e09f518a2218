"""Performance cases of the MoE layer on one GPU, through the package's public entry points.

Five kinds of case, each a piece of work that a program using this package has it do:

  layer     one MoE-layer forward (routing, grouping, schedule, expert FFNs, combine): a decode step
            when T is small, a prefill when it is large
  share     an expert-parallel rank's pre-routed share, some experts fetched from pinned host memory
  dispatch  routing, grouping with the row gather, the schedule and the combine of a rank whose
            experts run elsewhere
  pack      one layer's parameters brought into the kernels' layout (loading a model)

All inputs are drawn on the GPU from the seed alone: activations N(0,1), matrices N(0,1/fan_in), and
a router bias (or expert ids) that gives the experts Zipf-distributed loads.
"""
import math

import torch

from paper_2506_12417_amd import binding as B
from paper_2506_12417_amd.layer import XCDS, MoELayer, PreRoutedShare, default_q_tokens

DEV = "cuda:0"


# ------------------------------------------------------------------------------------- the cases
def listed():
    switch = dict(kind="layer", d=768, F=3072, E=128, k=1, act="relu", dtype="bf16", renorm=0, shared_F=0, zipf=1.0)
    fine = dict(kind="layer", d=2048, F=1408, E=60, k=4, act="swiglu", dtype="bf16", renorm=0, shared_F=5632, zipf=1.2)
    large = dict(kind="layer", d=4096, F=14336, E=8, k=2, act="swiglu", dtype="bf16", renorm=1, shared_F=0, zipf=2.0)
    return [
        # the fp32 layer at its smallest configuration: launches and latencies
        dict(name="f32_tiny", kind="layer", T=256, d=64, F=128, E=8, k=2, act="relu", dtype="f32", renorm=1, shared_F=0, zipf=1.5),
        # an fp32 layer of ordinary size, for programs that check or train against full precision
        dict(name="f32_layer", kind="layer", T=1501, d=768, F=2048, E=16, k=2, act="swiglu", dtype="f32", renorm=1, shared_F=0, zipf=1.0),
        # decode steps: a few sequences, one token each; the weights of the chosen experts are the work
        dict(switch, name="switch_decode", T=8),
        dict(fine, name="fine_decode", T=33),
        dict(large, name="large_decode", T=3),
        # one short batch: nearly every expert active with a handful of rows
        dict(switch, name="switch_short", T=1000),
        # prefill at the benchmark's sizes
        dict(switch, name="switch_prefill", T=16384),
        dict(fine, name="fine_prefill", T=8192),
        dict(large, name="large_prefill", T=8192),
        # a rank's share with half of its experts in host memory, at the benchmark's size
        dict(name="share_host_experts", kind="share", T=32768, d=768, F=3072, n_local=16, n_foreign=16, n_slots=16, foreign=0.30, zipf=1.5),
        # grouping for experts that live elsewhere: many experts, many assignments, a ragged width
        dict(name="dispatch", kind="dispatch", T=20011, d=1032, E=256, k=8, renorm=1, zipf=0.6),
        # loading one layer's experts and router
        dict(name="pack_layer", kind="pack", n=60, d=2048, F=1408, act="swiglu", dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["switch", "fine", "large", "any", "any", "f32", "f32", "share", "dispatch", "pack"])
    if kind == "switch":
        return dict(kind="layer", T=_log_int(rng, 1, 16384), d=768, F=3072, E=128, k=1, act="relu", dtype="bf16", renorm=0,
                    shared_F=0, zipf=round(rng.uniform(0.0, 1.5), 2))
    if kind == "fine":
        return dict(kind="layer", T=_log_int(rng, 1, 8192), d=2048, F=1408, E=60, k=4, act="swiglu", dtype="bf16", renorm=0,
                    shared_F=5632, zipf=round(rng.uniform(0.0, 1.5), 2))
    if kind == "large":
        return dict(kind="layer", T=_log_int(rng, 1, 8192), d=4096, F=14336, E=8, k=2, act="swiglu", dtype="bf16", renorm=1,
                    shared_F=0, zipf=round(rng.uniform(0.0, 2.0), 2))
    if kind == "any":       # widths, expert counts and activations in between
        E = rng.choice([4, 8, 16, 24, 48, 64, 100])
        return dict(kind="layer", T=_log_int(rng, 1, 8192), d=64 * _log_int(rng, 4, 40), F=64 * _log_int(rng, 8, 64), E=E,
                    k=rng.randint(1, min(E, 4)), act=rng.choice(["relu", "swiglu"]), dtype="bf16", renorm=rng.randint(0, 1),
                    shared_F=0, zipf=round(rng.uniform(0.0, 1.5), 2))
    if kind == "f32":
        E = rng.choice([4, 8, 16, 32])
        return dict(kind="layer", T=_log_int(rng, 1, 2048), d=8 * _log_int(rng, 8, 128), F=32 * _log_int(rng, 4, 64), E=E,
                    k=rng.randint(1, 2), act=rng.choice(["relu", "swiglu"]), dtype="f32", renorm=rng.randint(0, 1),
                    shared_F=0, zipf=round(rng.uniform(0.0, 1.5), 2))
    if kind == "share":
        slots = rng.randint(1, 16)
        return dict(kind="share", T=_log_int(rng, 256, 32768), d=768, F=3072, n_local=rng.randint(1, 16),
                    n_foreign=rng.randint(1, 16), n_slots=slots, foreign=round(rng.uniform(0.1, 0.5), 2),
                    zipf=round(rng.uniform(0.0, 1.5), 2))
    if kind == "dispatch":
        return dict(kind="dispatch", T=_log_int(rng, 16, 20000), d=8 * _log_int(rng, 16, 256), E=rng.randint(8, 256),
                    k=rng.randint(1, 8), renorm=rng.randint(0, 1), zipf=round(rng.uniform(0.0, 1.2), 2))
    return dict(kind="pack", n=_log_int(rng, 1, 60), d=64 * _log_int(rng, 4, 32), F=64 * _log_int(rng, 4, 44),
                act=rng.choice(["relu", "swiglu"]), dtype=rng.choice(["bf16", "bf16", "f32"]))


# ------------------------------------------------------------------------------------ the inputs
def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 64 + stream)


def _normal(shape, std, dtype, seed, stream):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=_gen(seed, stream))


def _shares(E, s, seed):
    """Zipf(s) load shares over an order of the experts that the seed decides."""
    p = torch.arange(1, E + 1, dtype=torch.float64).pow(-s)
    order = torch.randperm(E, generator=torch.Generator().manual_seed(int(seed)))
    out = torch.empty(E, dtype=torch.float64)
    out[order] = p / p.sum()
    return out


def _bias(E, s, seed):
    """A router bias under which tokens with N(0,1) logits choose their first expert by _shares."""
    want = _shares(E, s, seed).to(DEV)
    z = torch.randn((16384, E), device=DEV, generator=_gen(seed, 9))
    b = want.log()
    for _ in range(16):
        got = torch.bincount((z + b.float()).argmax(1), minlength=E).double() / z.shape[0]
        b = b + 0.3 * (want.log() - got.clamp_min(0.25 / z.shape[0]).log())
        b = b - b.max()
    return b.float()


def _matrices(n, d, F, act, dtype, seed, stream):
    """Expert matrices in the paper's orientation: [n, inputs, outputs]."""
    names = (("W1", d, F), ("W2", F, d)) if act == "relu" else (("Wg", d, F), ("Wu", d, F), ("Wd", F, d))
    return {name: _normal((n, i, o), i ** -0.5, dtype, seed, stream + j) for j, (name, i, o) in enumerate(names)}


def _inputs(case, seed):
    dt, kind = _dtype(case), case["kind"]
    if kind == "pack":
        return {"w": _matrices(case["n"], case["d"], case["F"], case["act"], dt, seed, 20),
                "W_g": _normal((case["d"], case["n"]), case["d"] ** -0.5, dt, seed, 2)}
    x = _normal((case["T"], case["d"]), 1.0, dt, seed, 1)
    if kind == "share":
        E = case["n_local"] + case["n_foreign"]
        p = torch.cat([_shares(case["n_local"], case["zipf"], seed) * (1.0 - case["foreign"]),
                       _shares(case["n_foreign"], case["zipf"], seed + 1) * case["foreign"]])
        ids = torch.multinomial(p.to(DEV), case["T"], replacement=True, generator=_gen(seed, 3)).to(torch.int32)
        return {"x": x, "ids": ids, "w": _matrices(E, case["d"], case["F"], "relu", dt, seed, 20)}
    got = {"x": x, "W_g": _normal((case["d"], case["E"]), case["d"] ** -0.5, dt, seed, 2), "b": _bias(case["E"], case["zipf"], seed)}
    if kind == "dispatch":
        got["y_perm"] = _normal((case["T"] * case["k"], case["d"]), 1.0, torch.float32, seed, 4)
        return got
    got["w"] = _matrices(case["E"], case["d"], case["F"], case["act"], dt, seed, 20)
    if case["shared_F"]:
        got["shared"] = _matrices(1, case["d"], case["shared_F"], "swiglu", dt, seed, 30)
    return got


def _bits(t):
    """A host copy as the layer's loaders take it: float32, or bfloat16 bit patterns."""
    return t.cpu().numpy() if t.dtype == torch.float32 else t.view(torch.int16).cpu().numpy().view("uint16")


def _pack_group(group, w, first=0):
    """Expert matrices into a group's packed storage, all experts in one call per matrix."""
    n = w[next(iter(w))].shape[0]
    if "W1" in w:
        B.moe_pack_weights(w["W1"], None, n, group.d, group.F, group.dt, group.w_in[first])
    else:
        B.moe_pack_weights(w["Wg"], w["Wu"], n, group.d, group.F, group.dt, group.w_in[first])
    B.moe_pack_w_out(w["W2"] if "W1" in w else w["Wd"], n, group.F, group.d, group.dt, group.w_out[first])


class _Share:
    """A share and the device slots that it owns."""

    def __init__(self, share, x, ids):
        self.share, self.x, self.ids = share, x, ids

    def __del__(self):
        self.share.close()


def prepare(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    dt = B.MOE_F32 if case.get("dtype") == "f32" else B.MOE_BF16
    if kind == "layer":
        layer = MoELayer(case["T"], case["d"], case["F"], case["E"], case["k"], case["act"], case["dtype"], case["renorm"],
                         shared_F=case["shared_F"], device=DEV)
        layer.load_router(_bits(inp["W_g"]), inp["b"].cpu().numpy())
        _pack_group(layer.experts, inp["w"])
        if case["shared_F"]:
            _pack_group(layer.shared, inp["shared"])
        return {"kind": kind, "layer": layer, "x": inp["x"]}
    if kind == "share":
        nl, nf = case["n_local"], case["n_foreign"]
        share = PreRoutedShare(case["T"], case["d"], case["F"], nl + nf, nl, case["n_slots"], device=DEV)
        _pack_group(share.local, {n: m[:nl] for n, m in inp["w"].items()})
        for e in range(nl, nl + nf):
            share.load_expert(e, {n: _bits(m[e]) for n, m in inp["w"].items()})
        return {"kind": kind, "state": _Share(share, inp["x"], inp["ids"])}
    if kind == "dispatch":
        T, d, E, k = case["T"], case["d"], case["E"], case["k"]
        A, i32 = T * k, torch.int32
        tile_m = B.moe_ffn_pick_tile_m(dt, A, E)
        cap = B.moe_plan_capacity(A, E, tile_m, XCDS)
        ws = B.moe_workspace_bytes(B.MOE_OP_PERMUTE, T, d, 0, E, k, dt)
        new = lambda shape, t: torch.empty(shape, dtype=t, device=DEV)  # noqa: E731
        return dict(inp, kind=kind, case=dict(case), dt=dt, tile_m=tile_m, cap=cap, ws=new(max(ws, 16), torch.uint8), ws_bytes=ws,
                    expert_idx=new((T, k), i32), gate_w=new((T, k), torch.float32), counts=new(E, i32), offsets=new(E + 1, i32),
                    perm=new(A, i32), inv_perm=new(A, i32), x_perm=new((A, d), inp["x"].dtype), tiles=new((cap, 4), i32),
                    plan_hdr=new(B.MOE_PLAN_HDR_INTS, i32), sched=new((E, XCDS), i32), y=new((T, d), torch.float32),
                    q=default_q_tokens(dt))
    n, d, F, t = case["n"], case["d"], case["F"], _dtype(case)
    rows = F if case["act"] == "relu" else 2 * F
    return dict(inp, kind=kind, case=dict(case), dt=dt, w_in=torch.empty((n, rows, d), dtype=t, device=DEV),
                w_out=torch.empty((n, d, F), dtype=t, device=DEV), W_gt=torch.empty((n, d), dtype=t, device=DEV),
                norm2=torch.empty(n, dtype=torch.float32, device=DEV))


# -------------------------------------------------------------------------------------- one pass
def run(state):
    s, kind = state, state["kind"]
    if kind == "layer":
        y = s["layer"].forward(s["x"])
        return {"y": y, "expert_idx": s["layer"].expert_idx, "gate_w": s["layer"].gate_w}
    if kind == "share":
        st = s["state"]
        return {"y": st.share.forward(st.x, st.ids)}
    if kind == "dispatch":
        c = s["case"]
        T, d, E, k, dt = c["T"], c["d"], c["E"], c["k"], s["dt"]
        B.moe_route_topk(s["x"], s["W_g"], s["b"], T, d, E, k, c["renorm"], dt, s["expert_idx"], s["gate_w"])
        B.moe_permute(s["x"], s["expert_idx"], T, d, E, k, dt, s["counts"], s["offsets"], s["perm"], s["inv_perm"], s["x_perm"],
                      s["ws"], s["ws_bytes"])
        B.moe_plan_tiles(s["counts"], s["offsets"], E, T * k, s["tile_m"], XCDS, s["q"], B.MOE_PLAN_HARMOENY, s["tiles"], s["cap"],
                         s["plan_hdr"], s["sched"])
        B.moe_unpermute_combine(s["y_perm"], s["inv_perm"], s["gate_w"], None, T, d, k, s["y"])
        return {n: s[n] for n in ("expert_idx", "gate_w", "counts", "offsets", "perm", "inv_perm", "x_perm", "sched", "y")}
    c, w = s["case"], s["w"]
    n, d, F, dt = c["n"], c["d"], c["F"], s["dt"]
    if c["act"] == "relu":
        B.moe_pack_weights(w["W1"], None, n, d, F, dt, s["w_in"])
        B.moe_pack_w_out(w["W2"], n, F, d, dt, s["w_out"])
    else:
        B.moe_pack_weights(w["Wg"], w["Wu"], n, d, F, dt, s["w_in"])
        B.moe_pack_w_out(w["Wd"], n, F, d, dt, s["w_out"])
    B.moe_pack_router(s["W_g"], d, n, dt, s["W_gt"], s["norm2"])
    # (16-bit w_out holds IEEE half patterns)
    w_out = s["w_out"] if dt == B.MOE_F32 else s["w_out"].view(torch.float16)
    return {"w_in": s["w_in"], "w_out": w_out, "W_gt": s["W_gt"], "norm2": s["norm2"]}


# ------------------------------------------------------------------------- what a pass must cost
def _active(E, s, picks):
    """Experts with at least one of `picks` draws from Zipf(s) shares."""
    p = [(i + 1.0) ** -s for i in range(E)]
    return sum(1.0 - (1.0 - v / sum(p)) ** picks for v in p)


def work(case):
    kind = case["kind"]
    es = 4 if case.get("dtype") == "f32" else 2
    d = case["d"]
    if kind == "pack":
        one = case["n"] * d * case["F"] * (2 if case["act"] == "relu" else 3) + d * case["n"]
        return {"bytes": 2 * one * es + 4 * case["n"], "flops": 0}
    if kind == "dispatch":
        T, E, k = case["T"], case["E"], case["k"]
        A = T * k
        return {"bytes": T * d * es + d * E * es + 4 * E + 8 * A          # routing: x, W_g, b -> ids, gates
                + 8 * A + 8 * E + A * d * es + 4 * E * XCDS               # perm, inv_perm, counts, offsets, x_perm, schedule
                + A * d * 4 + T * d * 4,                                  # combine
                "flops": 2 * T * d * E + 2 * A * d}
    T, F = case["T"], case["F"]
    if kind == "share":
        n = _active(case["n_local"], case["zipf"], T * (1 - case["foreign"])) + case["n_foreign"]
        return {"bytes": T * d * 2 + T * 4 + n * 2 * d * F * 2 + T * d * 4, "flops": 4 * T * d * F}
    E, k, mats = case["E"], case["k"], 2 if case["act"] == "relu" else 3
    b = T * d * es + d * E * es + 4 * E + T * k * 8 + T * d * 4 + _active(E, case["zipf"], T * k) * mats * d * F * es
    f = 2 * T * d * E + 2 * T * k * d * F * mats
    if case["shared_F"]:
        b += 3 * d * case["shared_F"] * es
        f += 6 * T * d * case["shared_F"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Measured between run() and exact(), times four or more: bf16 layers round their hidden activations
    once to 11 bits (2.1e-4 over all sizes); fp32 layers and everything else sum in fp32 (up to 1.1e-6).
    Integers and copies are exact everywhere (the selection is decided in 64 bits)."""
    if case["kind"] == "pack":      # copies and one rounding to half; norm2 is a sum in fp32
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "dispatch" or case.get("dtype") == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-3}


# --------------------------------------------------------------------- the same in 64 bits, plainly
def _route_exact(case, inp):
    logits = inp["x"].double() @ inp["W_g"].double() + inp["b"].double()
    _, idx = torch.topk(logits, case["k"], dim=1)
    gate = torch.softmax(logits, 1).gather(1, idx)
    return idx, gate / gate.sum(1, keepdim=True) if case["renorm"] else gate


def _ffn_exact(x, w, e):
    if "W1" in w:
        return (x @ w["W1"][e].double()).clamp_min(0.0) @ w["W2"][e].double()
    return (torch.nn.functional.silu(x @ w["Wg"][e].double()) * (x @ w["Wu"][e].double())) @ w["Wd"][e].double()


def _experts_exact(x, idx, gate, w):
    y = torch.zeros(x.shape, dtype=torch.float64, device=DEV)
    for e in range(w[next(iter(w))].shape[0]):
        t, j = (idx == e).nonzero(as_tuple=True)
        if t.numel():
            y.index_add_(0, t, _ffn_exact(x[t].double(), w, e) * gate[t, j][:, None])
    return y


def exact(case, seed):
    inp, kind = _inputs(case, seed), case["kind"]
    if kind == "share":
        ids = inp["ids"].long()[:, None]
        return {"y": _experts_exact(inp["x"], ids, torch.ones(ids.shape, dtype=torch.float64, device=DEV), inp["w"])}
    if kind == "pack":
        w = inp["w"]
        first, last = (w["W1"], w["W2"]) if case["act"] == "relu" else (w["Wg"], w["Wd"])
        order = torch.arange(32, device=DEV)
        if case["dtype"] == "bf16":        # packed row 16 h + j of a block of 32 holds output 2 j + h
            order = torch.cat([order[0::2], order[1::2]])

        def rows(m):                       # [n, inputs, outputs] -> [n, blocks, 32, inputs]
            t = m.transpose(1, 2)
            return t.reshape(t.shape[0], t.shape[1] // 32, 32, t.shape[2])[:, :, order]

        w_in = rows(first)
        if case["act"] == "swiglu":
            w_in = torch.stack([w_in, rows(w["Wu"])], 2)
        n = case["n"]
        return {"w_in": w_in.reshape(n, -1, case["d"]), "w_out": rows(last).reshape(n, case["d"], case["F"]).to(
            torch.float32 if case["dtype"] == "f32" else torch.float16), "W_gt": inp["W_g"].t().contiguous(), "norm2": None}
    idx, gate = _route_exact(case, inp)
    if kind == "layer":
        y = _experts_exact(inp["x"], idx, gate, inp["w"])
        if case["shared_F"]:
            y += _ffn_exact(inp["x"].double(), inp["shared"], 0)
        return {"y": y, "expert_idx": idx.int(), "gate_w": gate}
    flat = idx.reshape(-1)
    perm = torch.argsort(flat, stable=True)
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(perm.numel(), device=DEV)
    counts = torch.bincount(flat, minlength=case["E"])
    offsets = torch.cat([torch.zeros(1, dtype=counts.dtype, device=DEV), counts.cumsum(0)])
    y = torch.zeros(inp["x"].shape, dtype=torch.float64, device=DEV)
    for j in range(case["k"]):
        y += gate[:, j, None] * inp["y_perm"][inv.reshape(-1, case["k"])[:, j]].double()
    return {"expert_idx": idx.int(), "gate_w": gate, "counts": counts.int(), "offsets": offsets.int(), "perm": perm.int(),
            "inv_perm": inv.int(), "x_perm": inp["x"][perm // case["k"]], "sched": None, "y": y}

"""Workloads of the library, as programs that use it call them: MoE layers of GPT-MoE shapes (prefill, decode, bf16,
fp32, top-1, top-2, all experts or a share of them resident) and the offline side (affinity statistics of a routing
trace, transfers, multi-hop affinity, scores of candidate placements).

``listed()`` names the workloads that stand for each range, ``draw(rng)`` gives further ones of the same ranges.  A case is
a dict of plain values with a ``kind``:

  layer      one MoE layer through ``MoELayerRun.step``; ``fused`` selects the index-only dispatch with the fused
             expert FFN, otherwise the four separate calls.  ``routing``:
               gate     the layer's own gate decides (experts that are not resident drop their tokens)
               skewed   Zipf-distributed experts supplied by the caller (a trace-driven run)
               local    the tokens one GPU holds after the exchange: global ids, all of resident experts
  step       the benchmark's step: such a layer and the affinity statistic of the routing trace it belongs to
  statistics, transfers, multihop   one pass over a routing trace [L,N] with E experts
  scores     locality of B candidate placements from the counts of a trace
"""
from __future__ import annotations

import math

import torch

from paper_2401_08383_amd import binding as B
from paper_2401_08383_amd.pipeline import AffinityRun, MoELayerRun

DEV = "cuda"
MAX_FLOPS = 1.1e12         # the largest listed layer: 16384 tokens x 2048 x 8192
MAX_WEIGHT_BYTES = 17.2e9  # the widest listed layer: 64 experts of 4096 x 16384


def _layer(T, d, f, E, k=1, E_local=None, dtype="bf16", act="erf", fused=True, routing="gate"):
    return dict(kind="layer", T=T, d=d, f=f, E=E, E_local=E if E_local is None else E_local, k=k, renorm=k > 1,
                dtype=dtype, act=act, fused=fused, routing=routing)


def listed():
    return [
        # the smallest call of a serving loop: one sequence, one new token, one layer of the 350M-shaped model
        dict(name="decode_one_token", **_layer(1, 1024, 4096, 8)),
        # a decode batch of odd size through the XL-shaped model: most experts get one to four tokens
        dict(name="decode_batch", **_layer(61, 2048, 8192, 32)),
        # the widest layer, top-2 decode: every one of the 64 experts' weights (17 GB) is read once
        dict(name="decode_top2_wide", **_layer(256, 4096, 16384, 64, k=2)),
        # the benchmark step: 8192-token prefill of the 350M-shaped layer and its 12-layer trace statistic
        dict(name="prefill_step_350m", **dict(_layer(8192, 1024, 4096, 8), kind="step"), L=12, N=8192, trace_E=8, G=4),
        # a short prompt of odd length, top-2 with renormalised weights, through the four separate calls
        dict(name="prefill_short_top2", **_layer(1531, 1024, 4096, 16, k=2, act="tanh", fused=False)),
        # prefill of the XL-shaped layer with trace-driven, skewed routing over 32 experts
        dict(name="prefill_xl_skewed", **_layer(16384, 2048, 8192, 32, routing="skewed")),
        # one GPU's share of an expert-parallel layer: 8 of 64 experts resident, 32768 tokens after the exchange
        dict(name="prefill_share_8_of_64", **_layer(32768, 1024, 4096, 64, E_local=8, routing="local")),
        # the small fp32 layer used where results are compared in full precision
        dict(name="layer_f32", **_layer(512, 64, 256, 8, dtype="f32")),
        # offline: everything the placement program needs from a 24-layer trace of a million tokens
        dict(name="trace_statistics", kind="statistics", L=24, N=1 << 20, E=64, G=8),
        # offline: transfers of vanilla and coherent expert parallelism on a trace of odd length
        dict(name="trace_transfers", kind="transfers", L=24, N=999983, E=64, G=8),
        # offline: affinity of every layer to all later ones
        dict(name="trace_multihop", kind="multihop", L=24, N=1 << 20, E=64, G=8),
        # offline: one generation of candidate placements of a search
        dict(name="placement_scores", kind="scores", L=24, N=1 << 20, E=64, G=8, B=4096),
    ]


# ---------------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(_log(rng, lo, hi)))))


def _draw_layer(rng):
    while True:
        T = _log_int(rng, 1, 32768)
        d = 64 * _log_int(rng, 8, 64)
        f = d * 4 if rng.random() < 0.75 else 64 * _log_int(rng, d // 32, d // 16)
        E = _log_int(rng, 4, 64)
        k = rng.choice((1, 1, 2))
        E_local = E if rng.random() < 0.7 else max(1, E // rng.choice((2, 4, 8)))
        routing = "local" if E_local < E and rng.random() < 0.5 else rng.choice(("gate", "gate", "skewed"))
        c = _layer(T, d, f, E, k, E_local, act=rng.choice(("erf", "erf", "tanh")), fused=rng.random() < 0.75, routing=routing)
        if E_local * d * f * 4 <= MAX_WEIGHT_BYTES and 4.0 * T * k * d * f <= MAX_FLOPS:
            return c


def draw(rng):
    u = rng.random()
    if u < 0.60:
        return _draw_layer(rng)
    if u < 0.70:
        return _layer(_log_int(rng, 16, 4096), 4 * _log_int(rng, 8, 64), 4 * _log_int(rng, 32, 256), _log_int(rng, 2, 16),
                      rng.choice((1, 2)), dtype="f32", fused=rng.random() < 0.75)
    G = rng.choice((2, 4, 8))
    E = G * rng.randint(1, 64 // G) if rng.random() < 0.5 else 8 * rng.randint(1, 8)
    c = dict(kind=rng.choice(("statistics", "statistics", "transfers", "multihop", "scores")), L=rng.randint(2, 24),
             N=_log_int(rng, 1000, 1 << 20), E=E, G=G)
    if c["kind"] == "scores":
        c["B"] = _log_int(rng, 16, 4096)
    return c


# ---------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(shape, std, dtype, g):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)


def _zipf_ids(shape, E, g):
    """Expert ids whose frequencies follow 1/rank^1.1 over a random order of the experts."""
    p = 1.0 / torch.arange(1, E + 1, dtype=torch.float64, device=DEV) ** 1.1
    edges = torch.cumsum(p / p.sum(), 0).float()
    rank = torch.searchsorted(edges, torch.rand(shape, device=DEV, generator=g)).clamp_(max=E - 1)
    return torch.randperm(E, device=DEV, generator=g)[rank].int()


def _layer_state(c, seed):
    g = _gen(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    T, d, f, E, E_local, k = (c[n] for n in ("T", "d", "f", "E", "E_local", "k"))
    x = _normal((T, d), 1.0, dt, g)
    w_gate = _normal((E, d), 1.0 / math.sqrt(d), dt, g)  # logits ~ N(0,1)
    w1 = _normal((E_local, f, d), 0.02, dt, g)
    w2 = _normal((E_local, d, f), 0.02, dt, g)
    expert_map, idx = None, None
    resident = torch.sort(torch.randperm(E, device=DEV, generator=g)[:E_local]).values
    if E_local < E:
        expert_map = torch.full((E,), -1, dtype=torch.int32, device=DEV)
        expert_map[resident] = torch.arange(E_local, dtype=torch.int32, device=DEV)
    if c["routing"] == "local":
        idx = resident[torch.randint(0, E_local, (T, k), device=DEV, generator=g)].int()
    elif c["routing"] == "skewed":
        idx = _zipf_ids((T, k), E, g)
    if idx is not None and k == 2 and E > 1:  # the two experts of a token differ (where more than one is to be had)
        if c["routing"] == "local":
            if E_local > 1:
                place = expert_map[idx.long()]
                other = (place[:, 0] + 1 + place[:, 1] % (E_local - 1)) % E_local
                idx[:, 1] = resident[other.long()].int()
        else:
            idx[:, 1] = torch.where(idx[:, 1] == idx[:, 0], (idx[:, 0] + 1) % E, idx[:, 1])
    act = B.EXF_ACT_GELU_ERF if c["act"] == "erf" else B.EXF_ACT_GELU_TANH
    return MoELayerRun(x, w_gate, w1, w2, k, renormalize=c["renorm"], expert_map=expert_map, topk_idx=idx, act=act, fused=c["fused"])


def _trace(L, N, E, seed):
    """[L,N]: layer 0 uniform; later a permutation of the previous expert with probability 0.7, else uniform."""
    g = _gen(seed)
    t = torch.empty((L, N), dtype=torch.int32, device=DEV)
    t[0] = torch.randint(0, E, (N,), device=DEV, generator=g, dtype=torch.int32)
    for l in range(1, L):
        perm = torch.randperm(E, device=DEV, generator=g).int()
        other = torch.randint(0, E, (N,), device=DEV, generator=g, dtype=torch.int32)
        t[l] = torch.where(torch.rand(N, device=DEV, generator=g) < 0.7, perm[t[l - 1].long()], other)
    return t


def _placements(count, L, E, G, seed):
    """[count,L,E]: per layer a random permutation of the experts cut into G equal parts."""
    order = torch.rand((count, L, E), device=DEV, generator=_gen(seed)).argsort(dim=2)
    return (order // (E // G)).int()


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "layer":
        return dict(kind=kind, layer=_layer_state(c, seed))
    if kind == "step":
        trace = _trace(c["L"], c["N"], c["trace_E"], seed + (1 << 20))
        placement = _placements(1, c["L"], c["trace_E"], c["G"], seed + (1 << 21))[0]
        return dict(kind=kind, layer=_layer_state(c, seed), stats=AffinityRun(trace, placement, c["trace_E"], c["G"]))
    L, N, E, G = c["L"], c["N"], c["E"], c["G"]
    trace = _trace(L, N, E, seed)
    if kind == "scores":
        counts = B.affinity_histogram(trace, E)["counts"]
        maps = _placements(c["B"], L, E, G, seed + 1)
        return dict(kind=kind, counts=counts, maps=maps, out=torch.empty((c["B"], L - 1), dtype=torch.int64, device=DEV))
    if kind == "multihop":
        return dict(kind=kind, trace=trace, E=E, ws=_workspace(B.lib().affinity_multihop_workspace_bytes(L, N, E)))
    placement = _placements(1, L, E, G, seed + 1)[0]
    if kind == "statistics":
        return dict(kind=kind, stats=AffinityRun(trace, placement, E, G))
    home = torch.randint(0, G, (N,), device=DEV, generator=_gen(seed + 2), dtype=torch.int32)
    return dict(kind=kind, trace=trace, placement=placement, home=home, G=G,
                ws=_workspace(B.lib().routing_transfers_workspace_bytes(L, N)))


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


# ---------------------------------------------------------------------------------------------- one pass
def _layer_pass(layer):
    layer.step()
    return dict(out=layer.out, topk_idx=layer.topk_idx, topk_w=layer.topk_w)


def _stats_pass(stats):
    stats.step()
    return dict(counts=stats.counts, loads=stats.loads, cond_prob=stats.cond_prob, n_invalid=stats.n_invalid,
                local_per_pair=stats.local_per_pair)


def run(state):
    kind = state["kind"]
    if kind == "layer":
        return _layer_pass(state["layer"])
    if kind == "step":
        out = _layer_pass(state["layer"])
        out.update(_stats_pass(state["stats"]))
        return out
    if kind == "statistics":
        return _stats_pass(state["stats"])
    if kind == "transfers":
        local, away = B.routing_transfers(state["trace"], state["placement"], state["home"], state["G"], workspace=state["ws"])
        return dict(local=local, away=away)
    if kind == "multihop":
        return B.affinity_multihop(state["trace"], state["E"], workspace=state["ws"])
    return B.placement_locality_from_counts(state["counts"], state["maps"], out=state["out"])


# ---------------------------------------------------------------------------------------------- what a pass cannot do without
def _layer_work(c):
    T, d, f, E, E_local, k = (c[n] for n in ("T", "d", "f", "E", "E_local", "k"))
    s = 2 if c["dtype"] == "bf16" else 4
    kept = T * k * (E_local / E if c["routing"] != "local" else 1.0)
    touched = E_local * (1.0 - (1.0 - 1.0 / E_local) ** kept)  # experts with at least one token, expected
    return dict(bytes=2.0 * T * d * s + E * d * s + 2.0 * touched * d * f * s + 8.0 * T * k,
                flops=2.0 * T * d * E + 4.0 * kept * d * f)


def _trace_work(kind, L, N, E, B_=0):
    tables = {"statistics": (L - 1) * E * E * 12.0 + L * E * 8.0, "multihop": L * (L - 1) / 2 * E * E * 12.0, "transfers": 4.0 * N}
    if kind == "scores":
        return dict(bytes=(L - 1) * E * E * 8.0 + B_ * (L * E * 4.0 + (L - 1) * 8.0), flops=1.0 * B_ * (L - 1) * E * E)
    return dict(bytes=4.0 * L * N + tables[kind], flops=0.0)


def work(case):
    c = case
    if c["kind"] == "layer":
        return _layer_work(c)
    if c["kind"] == "step":
        a, b = _layer_work(c), _trace_work("statistics", c["L"], c["N"], c["trace_E"])
        return dict(bytes=a["bytes"] + b["bytes"], flops=a["flops"] + b["flops"])
    return _trace_work(c["kind"], c["L"], c["N"], c["E"], c.get("B", 0))


def tolerance(case):
    if case["kind"] in ("layer", "step"):
        if case["dtype"] == "f32":
            return dict(rel=1e-5, max=1e-3, differ=2e-3)
        # bf16 hidden activations and outputs; `differ`: two experts whose fp32 logits are a rounding apart
        return dict(rel=1e-2, max=5e-2, differ=2e-3)
    if case["kind"] in ("statistics", "multihop"):
        return dict(rel=1e-6, max=1e-5)  # the counts are exact, the probabilities one division
    return "exact"

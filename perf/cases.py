"""The work that users of the routed low-rank linear layer have it do, as measurable cases.

A case is a dict of plain values; `kind` says which calls one pass makes:
  decode   one decode step of a decoder block (q/k/v, o, gate/up, down) or of its MLP, over plans made once per batch; more
           than 32 sequences go through the calls that take any number
  step     one prefill step of a single routed layer: pool, cache probe, buckets and plan, aggregation, forward
  block    prefill of the seven projections of a decoder block, q/k/v and gate/up horizontally fused
  grouped  a ragged batch of clustered prompts through the pattern cache and the three MLP layers, one plan for all
  routed   routing without a cache: pool and route, buckets, aggregation, forward (fp32 layers)
  ranks    the rank-granular form: one score per rank, gather of single ranks, forward
  train    one router training step: route, aggregation, routed output, loss and gradient
Sizes are the repository's workloads (LLaMA-7B-shaped layers, 4096 / 11008) or generic ones of the same proportions.
"""
from __future__ import annotations

import random

import torch

import paper_2605_08568_amd as pa
import synth_inputs as si

DEV = "cuda"
TAU = 0.9


def listed():
    return [
        # interactive use: one user, one token at a time, a whole decoder block, replayed from a HIP graph as servers do
        {"name": "decode_block_1seq", "kind": "decode", "part": "block", "hidden": 4096, "inter": 11008, "seqs": 1,
         "patterns": 1, "replay": True},
        # a small server: a dozen sequences that do not fill the matrix instruction, eager calls
        {"name": "decode_block_12seq", "kind": "decode", "part": "block", "hidden": 4096, "inter": 11008, "seqs": 12,
         "patterns": 3, "replay": False},
        # the benchmark's decode workload: MLP of 32 sequences with four patterns
        {"name": "decode_mlp_32seq", "kind": "decode", "part": "mlp", "hidden": 4096, "inter": 11008, "seqs": 32,
         "patterns": 4, "replay": True},
        # a loaded server: more sequences than one panel, an odd number of them
        {"name": "decode_mlp_150seq", "kind": "decode", "part": "mlp", "hidden": 4096, "inter": 11008, "seqs": 150,
         "patterns": 6, "replay": False},
        # time to first token of one short question
        {"name": "step_1x77", "kind": "step", "n": 4096, "m": 4096, "R": 2048, "G": 16, "k": 8, "prompts": 1,
         "shortest": 77, "longest": 77, "shared": 0, "cold": False},
        # the benchmark's headline workload: eight prompts of 512 tokens, the cache knows all of them
        {"name": "step_8x512", "kind": "step", "n": 4096, "m": 4096, "R": 2048, "G": 16, "k": 8, "prompts": 8,
         "shortest": 512, "longest": 512, "shared": 0, "cold": False},
        # a ragged batch on a cleared cache: every prompt is routed, appended and aggregated, two groups shared by all
        {"name": "step_20_ragged_cold", "kind": "step", "n": 4096, "m": 4096, "R": 2048, "G": 16, "k": 8, "prompts": 20,
         "shortest": 20, "longest": 701, "shared": 2, "cold": True},
        # one long prompt through every projection of a block
        {"name": "block_1x2048", "kind": "block", "hidden": 4096, "inter": 11008, "prompts": 1, "shortest": 2048,
         "longest": 2048},
        # the cache stress workload: 256 ragged prompts of 16 clusters, the largest call
        {"name": "grouped_256_ragged", "kind": "grouped", "hidden": 4096, "inter": 11008, "prompts": 256, "clusters": 16,
         "shortest": 32, "longest": 2048},
        # the small fp32 configuration
        {"name": "routed_fp32_4x64", "kind": "routed", "n": 1024, "m": 1024, "R": 256, "G": 8, "k": 4, "prompts": 4,
         "shortest": 64, "longest": 64},
        # every rank its own expert, as the method is written
        {"name": "ranks_8x512", "kind": "ranks", "n": 4096, "m": 4096, "R": 2048, "K": 1024, "prompts": 8,
         "shortest": 512, "longest": 512},
        # training the router on one batch
        {"name": "train_8x512", "kind": "train", "n": 4096, "m": 4096, "R": 2048, "G": 16, "k": 8, "prompts": 8,
         "shortest": 512, "longest": 512},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _prompts(rng, most_prompts, most_tokens):
    """Number and length range of a batch's prompts, at most most_tokens tokens in all."""
    p = _log_int(rng, 1, most_prompts)
    longest = _log_int(rng, 16, max(16, min(4096, most_tokens // p)))
    shortest = longest if rng.random() < 0.4 else _log_int(rng, max(1, longest // 16), longest)
    return {"prompts": p, "shortest": shortest, "longest": longest}


def draw(rng):
    kind = rng.choice(["decode"] * 4 + ["step"] * 3 + ["block", "grouped", "routed", "ranks", "train"])
    hidden, inter = rng.choice([(1024, 2816), (2048, 5632), (4096, 11008), (4096, 11008)])
    if kind == "decode":
        seqs = _log_int(rng, 1, 192)
        return {"kind": kind, "part": rng.choice(["block", "mlp"]), "hidden": hidden, "inter": inter, "seqs": seqs,
                "patterns": rng.randint(1, min(8, seqs)), "replay": rng.random() < 0.5}
    if kind == "block":
        return {"kind": kind, "hidden": hidden, "inter": inter, **_prompts(rng, 4, 4096)}
    if kind == "grouped":
        p = _log_int(rng, 16, 256)
        longest = _log_int(rng, 64, 1024)
        return {"kind": kind, "hidden": hidden, "inter": inter, "prompts": p, "clusters": rng.randint(2, 16),
                "shortest": _log_int(rng, 8, longest), "longest": longest}
    if kind == "routed":
        n, m = rng.choice([256, 520, 1024, 1032, 2048]), rng.choice([256, 516, 1024, 2048])
        G = rng.choice([4, 8, 10])
        return {"kind": kind, "n": n, "m": m, "R": G * rng.choice([8, 20, 25]), "G": G, "k": rng.randint(1, G // 2),
                **_prompts(rng, 8, 1024)}
    n, m = rng.choice([(1024, 1024), (2048, 5632), (4096, 4096), (4096, 4096), (4096, 11008)])
    if kind == "ranks":
        R = rng.choice([512, 1024, 2048]) if n > 1024 else 512
        return {"kind": kind, "n": n, "m": m, "R": R, "K": 32 * rng.randint(R // 128, R // 48), **_prompts(rng, 8, 4096)}
    gs, G = rng.choice([64, 96, 128]), rng.choice([8, 16])
    if n == 1024:
        gs = 64
    if kind == "train":
        return {"kind": kind, "n": n, "m": m, "R": gs * G, "G": G, "k": rng.randint(2, G // 2), **_prompts(rng, 8, 4096)}
    k = rng.randint(2, G // 2)
    return {"kind": kind, "n": n, "m": m, "R": gs * G, "G": G, "k": k, **_prompts(rng, 24, 8192),
            "shared": rng.choice([0, 0, 1]), "cold": rng.random() < 0.4}


# ---------------------------------------------------------------------------------------------------- inputs
def _lengths(case):
    """The prompt lengths of a case: fixed by the case, so that its work is."""
    r = random.Random(case["prompts"] * 1000003 + case["shortest"] * 1009 + case["longest"])
    return [r.randint(case["shortest"], case["longest"]) for _ in range(case["prompts"])]


def _offsets(case):
    return torch.from_numpy(si.offsets_from_lengths(_lengths(case))).to(DEV)


def _tokens(gen, rows, width, dtype=torch.bfloat16):
    return torch.randn((rows, width), device=DEV, generator=gen, dtype=torch.float32).to(dtype)


def _router(gen, L, G, d):
    return torch.randn((L, G, d), device=DEV, generator=gen) / d ** 0.5


def _factors(gen, n, m, G, gs, gs_padded, dtype):
    """Row-major Vt [R][n], Ut [R][m]: rows of unit length, sigma_i = (i+1)^-0.5 in Ut, groups padded with zero ranks."""
    R = G * gs
    Vt = torch.randn((R, n), device=DEV, generator=gen) / n ** 0.5
    Ut = torch.randn((R, m), device=DEV, generator=gen) / m ** 0.5
    Ut *= (torch.arange(R, device=DEV, dtype=torch.float32) + 1.0).rsqrt()[:, None]
    if gs_padded != gs:
        pad = (0, 0, 0, gs_padded - gs)
        Vt = torch.nn.functional.pad(Vt.view(G, gs, n), pad).reshape(G * gs_padded, n)
        Ut = torch.nn.functional.pad(Ut.view(G, gs, m), pad).reshape(G * gs_padded, m)
    return Vt.to(dtype), Ut.to(dtype)


def _layer(gen, n, m, G, gs, gs_padded=None, keep_rowmajor=False):
    gp = gs_padded or gs
    Vt, Ut = _factors(gen, n, m, G, gs, gp, torch.bfloat16)
    rm = pa.Layer(Vt, Ut, n, m, G * gp, G, pa.PARSE_ROWMAJOR)
    mm = pa.layer_to_mfma16(rm)
    return (mm, rm) if keep_rowmajor else mm


def _subsets(gen, count, G, k):
    """count random k-subsets of G groups, ids ascending (int32 [count][k])."""
    score = torch.rand((count, G), device=DEV, generator=gen)
    return score.topk(k, dim=1).indices.sort(dim=1).values.to(torch.int32).contiguous()


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _empty(rows, cols, dtype=torch.bfloat16):
    return torch.empty((rows, cols), dtype=dtype, device=DEV)


# the layers of a decoder block: (fused calls, each a list of (n, m)); groups of real and of stored ranks
def _projections(case):
    h, i = case["hidden"], case["inter"]
    if case["kind"] == "grouped" or case.get("part") == "mlp":      # R = 20 groups; 128 ranks at 4096 x 11008
        gs = max(32, int(128 * h / 4096) // 32 * 32)
        return 20, 10, [[(h, i, gs, gs), (h, i, gs, gs)], [(i, h, gs, gs)]]
    def proj(n, m):                                                  # 0.6 of the dense parameter count in 16 groups
        gs = si.config3_ranks(n, m, 16)[1]
        return n, m, gs, (gs + 31) // 32 * 32
    return 16, 8, [[proj(h, h)] * 3, [proj(h, h)], [proj(h, i)] * 2, [proj(i, h)]]


def prepare(case, seed):
    torch.manual_seed(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return globals()["_prepare_" + case["kind"]](dict(case), gen)


def run(state):
    return state["pass"](state)


# ---------------------------------------------------------------------------------------------------- decode
def _prepare_decode(case, gen):
    G, k, calls = _projections(case)
    B, npat = case["seqs"], case["patterns"]
    pid = (torch.arange(B, device=DEV) % npat).to(torch.int32)
    st = {"pass": _run_decode, "pid": pid, "calls": [], "graph": None}
    xs = {w: _tokens(gen, B, w) for w in sorted({p[0] for c in calls for p in c})}
    for c in calls:
        layers = [_layer(gen, n, m, G, gs, gp) for n, m, gs, gp in c]
        pats = [pa.Patterns(k, npat, subsets=_subsets(gen, npat, G, k)) for _ in c]
        call = {"layers": layers, "pats": pats, "x": xs[c[0][0]], "ys": [_empty(B, p[1]) for p in c],
                "plan": pa.decode_plan(layers, pats, pid) if B <= 32 else None}
        need = pa.lowrank_decode_planned_workspace_bytes(layers) if B <= 32 else pa.lowrank_decode_multi_workspace_bytes(layers)
        call["ws"] = _bytes(need)
        st["calls"].append(call)
    if case["replay"]:
        _decode_calls(st)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            _decode_calls(st)
        st["graph"] = g
    return st


def _decode_calls(st):
    for c in st["calls"]:
        if c["plan"] is not None:
            pa.lowrank_decode_planned(c["layers"], c["x"], c["plan"], c["ys"], c["ws"])
        else:
            pa.lowrank_decode_multi(c["layers"], c["pats"], c["x"], st["pid"], c["ys"], c["ws"])


def _run_decode(st):
    if st["graph"] is not None:
        st["graph"].replay()
    else:
        _decode_calls(st)
    return [y for c in st["calls"] for y in c["ys"]]


# ---------------------------------------------------------------------------------------------------- prefill step of one layer
def _prepare_step(case, gen):
    n, m, G, k, P, sh = case["n"], case["m"], case["G"], case["k"], case["prompts"], case["shared"]
    gs = case["R"] // G
    off = _offsets(case)
    rows = sum(_lengths(case))
    slots = max(32, P)
    st = {"pass": _run_step, "case": case, "off": off, "rows": rows, "slots": slots, "X": _tokens(gen, rows, n),
          "layer": _layer(gen, n, m, G, gs), "Wr": _router(gen, 1, G, n), "cache": pa.Cache(slots, n, 1, k, max(P, 8))}
    st["cache"].set_shared(sh)
    own = (k - sh) * gs
    st["Vs"], st["Us"] = torch.empty((slots, own, n), dtype=torch.bfloat16, device=DEV), torch.empty((slots, own, m), dtype=torch.bfloat16, device=DEV)
    head = (None, None)
    if sh:
        head = pa.pack_experts(st["layer"], torch.arange(sh, dtype=torch.int32, device=DEV))
    st["pats"] = pa.Patterns(k, slots, st["Vs"], st["Us"], Vt_shared=head[0], Ut_shared=head[1], n_shared=sh)
    i32 = lambda c: torch.empty(c, dtype=torch.int32, device=DEV)  # noqa: E731
    st["emb"], st["sim"] = _empty(P, n, torch.float32), torch.empty(P, dtype=torch.float32, device=DEV)
    st["entry"], st["hit"], st["sub"] = i32(P), torch.empty(P, dtype=torch.uint8, device=DEV), i32((P, 1, k))
    st["bucket"] = (i32(P), i32(P), i32(P + 1), i32(1), i32(P))
    st["ws_route"] = _bytes(pa.route_workspace_bytes(rows, P, n))
    st["plan"] = _bytes(pa.prefill_plan_bytes(rows, P, slots))
    st["ws"] = _bytes(pa.lowrank_prefill_planned_workspace_bytes(st["layer"], rows, P, k, slots))
    st["Y"] = _empty(rows, m)
    _run_step(st)                       # the cache and the aggregated blocks of a program that has been running
    return st


def _run_step(st):
    c = st["case"]
    k, sh = c["k"], c["shared"]
    if c["cold"]:
        st["cache"].clear()
    pa.pool(st["X"], st["off"], st["emb"], st["ws_route"])
    st["cache"].lookup_or_route(st["emb"], TAU, st["Wr"], st["entry"], st["hit"], st["sim"], st["sub"])
    pa.bucket_and_plan(st["sub"], k, k, st["off"], st["entry"], st["rows"], st["slots"], st["bucket"], st["plan"])
    pa.pack_new_entries(st["layer"], st["sub"].view(-1)[sh:], k, k - sh, st["entry"], st["hit"], st["Vs"], st["Us"])
    pa.lowrank_prefill_planned(st["layer"], st["pats"], st["X"], st["off"], st["entry"], st["plan"], st["Y"], st["ws"])
    return [st["Y"], st["entry"], st["hit"], st["sub"], st["sim"], st["bucket"][0], st["bucket"][1]]


# ---------------------------------------------------------------------------------------------------- prefill of a decoder block
def _prepare_block(case, gen):
    G, k, calls = _projections(case)
    P = case["prompts"]
    rows = sum(_lengths(case))
    st = {"pass": _run_block, "off": _offsets(case), "pid": torch.arange(P, dtype=torch.int32, device=DEV), "calls": []}
    xs = {w: _tokens(gen, rows, w) for w in sorted({p[0] for c in calls for p in c})}
    for c in calls:
        layers = [_layer(gen, n, m, G, gs, gp) for n, m, gs, gp in c]
        pats = []
        for l in layers:
            Vs, Us = pa.pack_patterns(l, _subsets(gen, P, G, k), k, k, None, None, P)
            pats.append(pa.Patterns(k, P, Vs, Us))
        need = (pa.lowrank_prefill_multi_workspace_bytes(layers, pats, rows) if len(c) > 1
                else pa.lowrank_workspace_bytes(pa.PARSE_PREFILL, layers[0], rows, k, P, P))
        st["calls"].append({"layers": layers, "pats": pats, "x": xs[c[0][0]], "ys": [_empty(rows, p[1]) for p in c],
                            "ws": _bytes(need)})
    return st


def _run_block(st):
    for c in st["calls"]:
        if len(c["layers"]) > 1:
            pa.lowrank_prefill_multi(c["layers"], c["pats"], c["x"], st["off"], st["pid"], c["ys"], c["ws"])
        else:
            pa.lowrank_forward(pa.PARSE_PREFILL, c["layers"][0], c["pats"][0], c["x"], st["off"], st["pid"], c["ys"][0], c["ws"])
    return [y for c in st["calls"] for y in c["ys"]]


# ---------------------------------------------------------------------------------------------------- clustered prompts, MLP layers
def _prepare_grouped(case, gen):
    G, k, calls = _projections(case)
    h, P, nc = case["hidden"], case["prompts"], case["clusters"]
    rows, slots, L = sum(_lengths(case)), 32, 3
    shapes = [p for c in calls for p in c]
    centre = torch.randn((nc, h), device=DEV, generator=gen)
    which = torch.randint(0, nc, (P,), device=DEV, generator=gen)
    emb = centre[which] + 0.1 * torch.randn((P, h), device=DEV, generator=gen)
    i32 = lambda c: torch.empty(c, dtype=torch.int32, device=DEV)  # noqa: E731
    st = {"pass": _run_grouped, "k": k, "L": L, "P": P, "rows": rows, "slots": slots, "off": _offsets(case), "emb": emb,
          "Wr": _router(gen, L, G, h), "cache": pa.Cache(slots, h, L, k, P), "entry": i32(P), "hit": torch.empty(P, dtype=torch.uint8, device=DEV),
          "sim": torch.empty(P, dtype=torch.float32, device=DEV), "sub": i32((P, L, k)),
          "bucket": (i32(P), i32(P), i32(P + 1), i32(1), i32(P)), "plan": _bytes(pa.prefill_plan_bytes(rows, P, slots)),
          "xs": {w: _tokens(gen, rows, w) for w in sorted({p[0] for p in shapes})}, "layers": [], "pats": [], "ys": []}
    for n, m, gs, gp in shapes:
        st["layers"].append(_layer(gen, n, m, G, gs, gp))
        st["pats"].append(pa.Patterns(k, slots, torch.empty((slots, k * gp, n), dtype=torch.bfloat16, device=DEV),
                                      torch.empty((slots, k * gp, m), dtype=torch.bfloat16, device=DEV)))
        st["ys"].append(_empty(rows, m))
    st["ws"] = _bytes(max(pa.lowrank_prefill_planned_workspace_bytes(l, rows, P, k, slots) for l in st["layers"]))
    return st


def _run_grouped(st):
    k, L, P = st["k"], st["L"], st["P"]
    st["cache"].clear()                # a service that has just started: the first prompt of every cluster misses
    st["cache"].lookup_or_route(st["emb"], TAU, st["Wr"], st["entry"], st["hit"], st["sim"], st["sub"])
    sub = st["sub"].view(P, L * k)
    pa.bucket_patterns(sub, L * k, L * k, st["bucket"])
    for l in range(L):
        pa.pack_new_entries(st["layers"][l], sub[:, l * k:], L * k, k, st["entry"], st["hit"], st["pats"][l].Vt_S, st["pats"][l].Ut_S)
    pa.prefill_plan(st["off"], st["entry"], st["rows"], st["slots"], st["plan"])
    for l, layer in enumerate(st["layers"]):
        pa.lowrank_prefill_planned(layer, st["pats"][l], st["xs"][layer.n], st["off"], st["entry"], st["plan"], st["ys"][l], st["ws"])
    return st["ys"] + [st["entry"], st["hit"], st["sub"], st["sim"], st["bucket"][0], st["bucket"][1]]


# ---------------------------------------------------------------------------------------------------- fp32, routed without a cache
def _prepare_routed(case, gen):
    n, m, G, k, P = case["n"], case["m"], case["G"], case["k"], case["prompts"]
    gs = case["R"] // G
    rows = sum(_lengths(case))
    Vt, Ut = _factors(gen, n, m, G, gs, gs, torch.float32)
    layer = pa.Layer(Vt, Ut, n, m, case["R"], G, pa.PARSE_ROWMAJOR)
    st = {"pass": _run_routed, "k": k, "P": P, "off": _offsets(case), "layer": layer, "Wr": _router(gen, 1, G, n)[0],
          "X": _tokens(gen, rows, n, torch.float32), "Vs": torch.empty((P, k * gs, n), device=DEV),
          "Us": torch.empty((P, k * gs, m), device=DEV), "sub": torch.empty((P, k), dtype=torch.int32, device=DEV),
          "scores": _empty(P, G, torch.float32), "ws_route": _bytes(pa.route_workspace_bytes(rows, P, n)),
          "Y": _empty(rows, m, torch.float32),
          "ws": _bytes(pa.lowrank_workspace_bytes(pa.PARSE_PREFILL, layer, rows, k, P, P))}
    i32 = lambda c: torch.empty(c, dtype=torch.int32, device=DEV)  # noqa: E731
    st["bucket"] = (i32(P), i32(P), i32(P + 1), i32(1), i32(P))
    st["pats"] = pa.Patterns(k, P, st["Vs"], st["Us"])
    return st


def _run_routed(st):
    k, P = st["k"], st["P"]
    pa.route(st["X"], st["off"], st["Wr"], k, st["sub"], k, st["scores"], None, st["ws_route"])
    pid, perm, boff, npat, rep = pa.bucket_patterns(st["sub"], k, k, st["bucket"])
    pa.pack_patterns(st["layer"], st["sub"], k, k, rep, npat, P, st["Vs"], st["Us"])
    pa.lowrank_forward(pa.PARSE_PREFILL, st["layer"], st["pats"], st["X"], st["off"], pid, st["Y"], st["ws"])
    return [st["Y"], st["sub"], st["scores"], pid, perm]


# ---------------------------------------------------------------------------------------------------- rank-granular form
def _prepare_ranks(case, gen):
    n, m, R, K, P = case["n"], case["m"], case["R"], case["K"], case["prompts"]
    rows = sum(_lengths(case))
    Vt, Ut = _factors(gen, n, m, R, 1, 1, torch.bfloat16)
    layer = pa.Layer(Vt, Ut, n, m, R, R, pa.PARSE_ROWMAJOR)
    units = pa.Layer(Vt, Ut, n, m, R, R // 32, pa.PARSE_MFMA16)      # the aggregated blocks in 32-rank units
    st = {"pass": _run_ranks, "K": K, "P": P, "off": _offsets(case), "pid": torch.arange(P, dtype=torch.int32, device=DEV),
          "layer": layer, "units": units, "Wr": _router(gen, 1, R, n)[0], "X": _tokens(gen, rows, n), "Y": _empty(rows, m),
          "sub": torch.empty((P, K), dtype=torch.int32, device=DEV), "scores": _empty(P, R, torch.float32),
          "Vs": torch.empty((P, K, n), dtype=torch.bfloat16, device=DEV), "Us": torch.empty((P, K, m), dtype=torch.bfloat16, device=DEV),
          "ws_route": _bytes(pa.lib().parse_route_ranks_workspace_bytes(rows, P, n, R)),
          "ws": _bytes(pa.lowrank_workspace_bytes(pa.PARSE_PREFILL, units, rows, K // 32, P, P))}
    st["pats"] = pa.Patterns(K // 32, P, st["Vs"], st["Us"])
    return st


def _run_ranks(st):
    pa.route_ranks(st["X"], st["off"], st["Wr"], st["K"], st["sub"], st["K"], st["scores"], None, st["ws_route"])
    pa.pack_ranks(st["layer"], st["sub"], st["K"], st["P"], st["K"], st["Vs"], st["Us"])
    pa.lowrank_forward(pa.PARSE_PREFILL, st["units"], st["pats"], st["X"], st["off"], st["pid"], st["Y"], st["ws"])
    return [st["Y"], st["scores"], st["sub"]]


# ---------------------------------------------------------------------------------------------------- router training step
def _prepare_train(case, gen):
    n, m, G, k, P = case["n"], case["m"], case["G"], case["k"], case["prompts"]
    gs = case["R"] // G
    rows = sum(_lengths(case))
    layer, rm = _layer(gen, n, m, G, gs, keep_rowmajor=True)
    X = _tokens(gen, rows, n)
    # the dense teacher's output: all ranks of the layer, and a tenth of it in directions that the layer does not have
    Yd = (X @ rm.Vt.t()) @ rm.Ut
    Yd = (Yd + 0.1 * Yd.float().std() * torch.randn(Yd.shape, device=DEV, generator=gen)).to(torch.bfloat16)
    st = {"pass": _run_train, "k": k, "P": P, "off": _offsets(case), "pid": torch.arange(P, dtype=torch.int32, device=DEV),
          "layer": layer, "left": pa.rankmajor_left_factor(rm), "Wr": _router(gen, 1, G, n)[0], "X": X, "Yd": Yd,
          "Y": _empty(rows, m), "sub": torch.empty((P, k), dtype=torch.int32, device=DEV), "scores": _empty(P, G, torch.float32),
          "emb": _empty(P, n, torch.float32), "Vs": torch.empty((P, k * gs, n), dtype=torch.bfloat16, device=DEV),
          "Us": torch.empty((P, k * gs, m), dtype=torch.bfloat16, device=DEV), "ws_route": _bytes(pa.route_workspace_bytes(rows, P, n)),
          "ws": _bytes(pa.lowrank_workspace_bytes(pa.PARSE_PREFILL, layer, rows, k, P, P))}
    cl = layer.c()
    st["ws_grad"] = _bytes(pa.lib().parse_router_grad_workspace_bytes(cl, rows, P))
    st["pats"] = pa.Patterns(k, P, st["Vs"], st["Us"])
    return st


def _run_train(st):
    k, P = st["k"], st["P"]
    pa.route(st["X"], st["off"], st["Wr"], k, st["sub"], k, st["scores"], st["emb"], st["ws_route"])
    pa.pack_patterns(st["layer"], st["sub"], k, k, None, None, P, st["Vs"], st["Us"])
    pa.lowrank_forward(pa.PARSE_PREFILL, st["layer"], st["pats"], st["X"], st["off"], st["pid"], st["Y"], st["ws"])
    loss, grad = pa.router_grad(st["layer"], st["left"], st["X"], st["off"], st["Y"], st["Yd"], st["emb"], st["scores"], k, 0.5, 1e-6,
                                st["ws_grad"])
    return [loss, grad, st["Y"], st["sub"], st["scores"]]


# ---------------------------------------------------------------------------------------------------- work and tolerance
def work(case):
    """Bytes and flops of one pass that no implementation can do without: every input read once, every output written
    once, the stored factors of the ranks in use read once (and written once where a pass aggregates them)."""
    kind = case["kind"]
    if kind in ("decode", "block", "grouped"):
        G, k, calls = _projections(case)
        rows = case["seqs"] if kind == "decode" else sum(_lengths(case))
        by = fl = 0.0
        for c in calls:
            by += rows * c[0][0] * 2
            for n, m, gs, _ in c:
                fl += 2.0 * rows * k * gs * (n + m)
                if kind == "decode":      # groups that at least one of the patterns selects (expected number)
                    blocks = G * (1.0 - (1.0 - k / G) ** case["patterns"]) * gs
                else:
                    blocks = k * gs * case["prompts" if kind == "block" else "clusters"]
                by += (3 if kind == "grouped" else 1) * blocks * (n + m) * 2 + rows * m * 2
        return {"bytes": by, "flops": fl}
    n, m, P = case["n"], case["m"], case["prompts"]
    rows = sum(_lengths(case))
    es = 4 if kind == "routed" else 2
    rS = case["K"] if kind == "ranks" else case["k"] * (case["R"] // case["G"])
    by = rows * (n + m) * es
    fl = 2.0 * rows * rS * (n + m)
    own = rS - case.get("shared", 0) * (case["R"] // case["G"] if "G" in case else 0)
    by += (P * own + rS - own) * (n + m) * es             # aggregated blocks, the shared head once
    if kind != "step" or case["cold"]:
        by += 2 * P * own * (n + m) * es                  # aggregation: read and written
        by += (case["R"] if kind == "ranks" else case["G"]) * n * 4      # the router
    if kind == "train":
        by += rows * m * 2 * 2 + 2 * case["R"] * (n + m) + P * n * 4 + case["G"] * n * 4
        fl += 2.0 * rows * case["R"] * (n + m)            # the two full-rank products of the gradient
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """Four times what the outputs are off from the same products in float64: bf16 paths 2.4e-3 (largest single value 1.9e-2
    of itself), fp32 8.3e-7 (5.7e-6).  Ids, flags and permutations stay the same."""
    if case["kind"] == "routed":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}

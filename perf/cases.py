"""The timed cases of the library: one expert-parallel rank's routing work, through the public calls.

A case is a dict of plain values.  `path` says which calls it takes:

  forward   hm_plan (with masks and load counts), hm_dispatch_pack, hm_combine with the plan's weights
  backward  hm_combine_transpose (of the output gradient), then hm_combine over the gradients that come
            back for the dispatched rows, with weight 1 on every kept slot: the gradient of x
  receiver  both hops on a receiving rank: hm_plan_mapped / hm_dispatch_pack of rows, ids and weights
            inside the node, hm_plan_mapped / hm_dispatch_pack to the local experts, hm_combine_mix back
  planner   hm_group_counts, hm_alltoall_times, hm_swap_counts_multi, hm_swap_select, hm_swap_apply
  counts    hm_expert_load and hm_group_counts: the monitoring of an iteration without a plan

Inputs are drawn on the GPU from the seed: N(0,1) router logits (with a Zipf(1.2) bias for `zipf`,
DeepSeek's group-limited choice for `grouped`), N(0,1) activations, N(0,1e-2) gradients, contiguous
expert blocks.  Plans, row buffers and workspaces are allocated once and kept, as a training loop keeps
them: row buffers have room for more rows than are expected, and hold zeros behind the rows written.
"""
import math

import torch

from paper_2508_09591_amd import binding as B

LEVELS = {"none": B.HM_DEDUP_NONE, "gpu": B.HM_DEDUP_GPU, "node": B.HM_DEDUP_NODE}

# Start-up time and inverse bandwidth of the exchanges (the paper's Fig.9 fit); entry 0 of the inter
# lists is unused.
ALPHA_INTER, BETA_INTER = [0.0, 4.97e-1, 3.01e-1, 1.49e-1], [0.0, 5.29e-7, 1.17e-7, 2.06e-8]
ALPHA_INTRA, BETA_INTRA = [7.22e-1, 5.71e-1, 1.14e-1, 2.04e-1], [5.70e-7, 1.27e-7, 2.63e-8, 1.64e-8]
GAMMA = 10.0


def _case(name, path, T, H, E, K, nodes, ranks, router, level="node", dtype="bf16", drop=0.0):
    c = {"path": path, "T": T, "H": H, "E": E, "K": K, "nodes": nodes, "ranks": ranks, "router": router,
         "level": level, "dtype": dtype, "drop": drop}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer of the benchmark set: three launches, nothing but latency
        _case("forward tiny gpu", "forward", 1024, 256, 16, 2, 2, 2, "softmax", "gpu"),
        # one decode batch of a served DeepSeek-V3-shaped layer: few tokens, long rows
        _case("forward decode node", "forward", 128, 7168, 256, 8, 4, 8, "grouped", "node"),
        # a Qwen3-30B-A3B-shaped training layer, one copy per GPU: seven short rows per token
        _case("forward qwen3 gpu", "forward", 8192, 2048, 128, 8, 4, 8, "softmax", "gpu"),
        # the headline: a DeepSeek-V3-shaped training layer, one copy per node
        _case("forward dsv3 node", "forward", 8192, 7168, 256, 8, 4, 8, "grouped", "node"),
        # the long-sequence layer: 64 Ki tokens on 8 x 8 ranks, the largest call
        _case("forward stress node", "forward", 65536, 7168, 256, 8, 8, 8, "grouped", "node"),
        # no deduplication (the plain MoE permute), a row length that is no multiple of a vector,
        # an odd token count and a router that drops slots over capacity
        _case("forward ragged none", "forward", 4097, 1030, 64, 6, 2, 4, "softmax", "none", drop=0.03),
        # the way back through the headline layer in bf16
        _case("backward dsv3 node", "backward", 8192, 7168, 256, 8, 4, 8, "grouped", "node"),
        # the way back with fp32 gradients, one copy per GPU, a skewed router
        _case("backward skew gpu f32", "backward", 16384, 2048, 128, 8, 4, 8, "zipf", "gpu", "f32"),
        # a receiving rank of the headline layer: what the 4 nodes send it, and its share of the node's rows
        _case("receiver dsv3", "receiver", 25600, 7168, 256, 8, 4, 8, "grouped"),
        # the expert-swap planner, once per iteration, on the skewed layer of the benchmark set ...
        _case("planner skew", "planner", 16384, 2048, 128, 8, 4, 8, "zipf"),
        # ... and on the headline layer
        _case("planner dsv3", "planner", 8192, 7168, 256, 8, 4, 8, "grouped"),
        # load monitoring alone, the count kernels of an iteration that keeps its plan
        _case("counts qwen3", "counts", 8192, 2048, 128, 8, 4, 8, "softmax"),
    ]


def draw(rng):
    def log_between(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    path = rng.choice(["forward"] * 8 + ["backward"] * 4 + ["receiver"] * 3 + ["planner"] * 3 + ["counts"] * 2)
    nodes, ranks = rng.choice([(2, 2), (1, 8), (2, 4), (2, 8), (4, 4), (3, 5), (4, 8), (8, 8)])
    G = nodes * ranks
    K = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 8, 10])
    E = G * max(1, log_between(16, 512) // G)   # whole blocks of experts per rank ...
    if rng.random() < 0.25:
        E = min(512, E + rng.randrange(1, G))   # ... or ranks that hold one more than others
    E = max(E, K + 1)
    if path == "receiver":
        E = min(E, 60 * G)                      # a receiving rank tells at most 64 experts of its own apart
    T = log_between(16, 65536)
    H = log_between(256, 7168)
    ragged = rng.random() < 0.2
    H = H if ragged else max(256, H // 64 * 64)
    router = rng.choice(["softmax", "zipf", "grouped"])
    if router == "grouped" and (E % 8 or K > E // 2 or E < 16):
        router = "softmax"
    c = _case(None, path, T, H, E, K, nodes, ranks, router, rng.choice(["none", "gpu", "gpu", "node", "node"]),
              rng.choice(["bf16", "bf16", "f32"]) if path == "backward" else "bf16", rng.choice([0.0, 0.0, 0.03]))
    # no dearer than the largest listed case; rows that are no multiple of a 16-byte vector, a sixteenth
    most = _forward_bytes(65536, 7168, 8, 4.0) / (16 if ragged else 1)
    while work(c)["bytes"] > most:
        c["T"] = max(16, c["T"] * 5 // 8)
    return c


# ---- inputs -------------------------------------------------------------------------------------
def _generator(seed, device):
    return torch.Generator(device=device).manual_seed(int(seed) * 7919 + 17)


def _route(c, tokens, g, device, bias=None):
    """ids [tokens,K] int32 and weights [tokens,K] fp32, slots in descending score."""
    E, K = c["E"], c["K"]
    logits = torch.randn((tokens, E), generator=g, device=device)
    if bias is not None:
        logits += bias
    if c["router"] == "grouped":   # sigmoid scores, the best 4 of 8 groups by their two best, top-K inside
        score = torch.sigmoid(logits)
        groups = score.view(tokens, 8, E // 8)
        best = groups.topk(min(2, E // 8), dim=2).values.sum(2).topk(4, dim=1).indices
        allowed = torch.zeros((tokens, 8), dtype=torch.bool, device=device).scatter_(1, best, True)
        ids = torch.where(allowed[:, :, None], groups, -1.0).view(tokens, E).topk(K, dim=1).indices
        w = score.gather(1, ids)
        w = w / w.sum(1, keepdim=True)
    else:
        top = logits.topk(K, dim=1)
        ids, w = top.indices, torch.softmax(top.values, dim=1)
    ids = ids.to(torch.int32)
    if c["drop"]:
        ids[torch.rand(ids.shape, generator=g, device=device) < c["drop"]] = -1
    return ids.contiguous(), w.contiguous()


def _bias(c, g, device):
    if c["router"] != "zipf":
        return None
    pmf = torch.arange(1, c["E"] + 1, dtype=torch.float64, device=device) ** -1.2
    return torch.log(pmf / pmf.sum()).to(torch.float32)[torch.randperm(c["E"], generator=g, device=device)]


def _placement(c, device):
    return (torch.arange(c["E"], device=device) * (c["nodes"] * c["ranks"]) // c["E"]).to(torch.int32)


def _route_to(c, rows, wanted, g, device, bias):
    """Routing of `rows` tokens that select at least one of the `wanted` experts: what arrives at a hop."""
    ids, w, have = [], [], 0
    while have < rows:
        i, v = _route(c, 2 * rows + 256, g, device, bias)
        hit = (wanted[i.clamp(min=0).long()] & (i >= 0)).any(1)
        ids.append(i[hit])
        w.append(v[hit])
        have += ids[-1].shape[0]
    return torch.cat(ids)[:rows].contiguous(), torch.cat(w)[:rows].contiguous()


def _rows(n, H, g, dtype=torch.bfloat16, sigma=1.0):
    """[n,H] normal values; in slices, so that the fp32 draw of a large buffer is not held whole."""
    out = torch.empty((n, H), dtype=dtype, device="cuda")
    for a in range(0, n, 65536):
        out[a:a + 65536] = torch.randn(out[a:a + 65536].shape, generator=g, device="cuda") * sigma
    return out


def _inputs(c, seed):
    """Everything prepare() hands to the library and exact() starts from, from the seed alone."""
    g = _generator(seed, "cuda")
    bias = _bias(c, g, "cuda")
    s = {"e2r": _placement(c, "cuda")}
    if c["path"] != "receiver":
        s["ids"], s["w"] = _route(c, c["T"], g, "cuda", bias)
    else:
        me = (1 % c["nodes"]) * c["ranks"]
        s["me"] = me
        on_node = torch.div(s["e2r"], c["ranks"], rounding_mode="floor") == me // c["ranks"]
        on_rank = s["e2r"] == me
        minus = torch.full_like(s["e2r"], -1)
        s["map_a"] = torch.where(on_node, s["e2r"] % c["ranks"], minus)
        s["map_b"] = torch.where(on_rank, torch.cumsum(on_rank, 0, dtype=torch.int32) - 1, minus)
        s["local"] = int(on_rank.sum())
        s["ids_a"], s["w_a"] = _route_to(c, c["T"], on_node, g, "cuda", bias)
        # the node's ranks each send this rank its share of what they forward: as many rows as it sends
        s["per_a"], s["per_b"] = _per_hop(c)
        s["ids_b"], s["w_b"] = _route_to(c, int(s["per_a"] * c["T"]), on_rank, g, "cuda", bias)
    s["g"] = g
    return s


# ---- one pass -----------------------------------------------------------------------------------
def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    T, H, E, K, nodes, ranks, level = c["T"], c["H"], c["E"], c["K"], c["nodes"], c["ranks"], LEVELS[c["level"]]
    g, G = s["g"], nodes * ranks
    new = lambda *shape, dtype=torch.bfloat16: torch.empty(shape, dtype=dtype, device="cuda")
    if c["path"] in ("forward", "backward"):
        cap = _capacity(c, T, _per_level(c), G if c["level"] != "node" else nodes)
        s["plan"] = p = _zeroed(B.alloc_plan(T, K, E, nodes, ranks, level, row_capacity=cap, loads=True))
        B.hm_plan(s["ids"], s["w"], s["e2r"], nodes, ranks, level, plan=p)
        total = B.hm_plan_status(p)[1]
        s["level"] = level
    if c["path"] == "forward":
        s["x"], s["y"] = _rows(T, H, g), _rows(total, H, g)
        s["packed"], s["out"] = new(cap, H).zero_(), new(T, H)
        s["outputs"] = {"packed": s["packed"], "out": s["out"], "row_weight": p.row_weight, "row_token": p.row_token,
                        "slot_row": p.slot_row, "slot_keep": p.slot_keep, "dest_count": p.dest_count, "dest_offset": p.dest_offset,
                        "rank_mask": p.rank_mask, "node_mask": p.node_mask, "status": p.status, "load_expert": p.load_expert,
                        "load_rank": p.load_rank, "load_node": p.load_node}
    elif c["path"] == "backward":
        dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
        s["gout"], s["gpacked"] = _rows(T, H, g, dt, 1e-2), _rows(total, H, g, dt, 1e-2)
        s["gy"], s["gx"], s["keep"] = new(cap, H, dtype=dt).zero_(), new(T, H, dtype=dt), p.slot_keep.to(torch.float32)
        s["outputs"] = {"gy": s["gy"], "gx": s["gx"]}
    elif c["path"] == "receiver":
        num = new(1, dtype=torch.int32)
        for st, stage in (("a", B.HM_RECV_INTRA_NODE), ("b", B.HM_RECV_LOCAL_EXPERTS)):
            n, dests = s["ids_" + st].shape[0], ranks if st == "a" else s["local"]
            s["table_" + st] = new(E, dtype=torch.int32)
            B.hm_recv_dest_map(s["e2r"], nodes, ranks, s["me"], stage, s["table_" + st], num)
            cap = _capacity(c, n, s["per_" + st], dests)
            p = _zeroed(B.alloc_plan(n, K, E, 1, 1, B.HM_DEDUP_GPU if st == "a" else B.HM_DEDUP_NONE, row_capacity=cap, num_dest=dests))
            B.hm_plan_mapped(s["ids_" + st], s["w_" + st], s["table_" + st], dests, st == "a", plan=p)
            total = B.hm_plan_status(p)[1]
            s.update({"plan_" + st: p, "x_" + st: _rows(n, H, g), "y_" + st: _rows(total, H, g),
                      "packed_" + st: new(cap, H).zero_(), "back_" + st: new(n, H)})
            s["outputs"] = dict(s.get("outputs", {}), **{
                "packed_" + st: s["packed_" + st], "back_" + st: s["back_" + st], "row_weight_" + st: p.row_weight,
                "row_token_" + st: p.row_token, "slot_row_" + st: p.slot_row, "offset_" + st: p.dest_offset})
            if st == "a":   # ids and weights travel as rows of 2K two-byte units
                s["meta_in"] = [s[k].view(torch.bfloat16).view(-1, 2 * K) for k in ("ids_a", "w_a")]
                s["meta"] = [new(cap, 2 * K).zero_(), new(cap, 2 * K).zero_()]
                s["outputs"]["meta"] = [m.view(torch.int32) for m in s["meta"]]
    else:
        U = _hierarchy(c)
        s["U"], s["own"] = U, torch.zeros((len(U), 64), dtype=torch.int32, device="cuda")
        s["groups"], s["status"] = [G] + U[1:], new(1, dtype=torch.int32)
        if c["path"] == "counts":
            s["load"] = [new(n, dtype=torch.int32) for n in (E, G, nodes)]
            s["outputs"] = {"own": s["own"], "load": s["load"], "status": s["status"]}
        else:
            cuts = _cuts(c)
            s["placed"], s["cuts"] = s["e2r"].clone(), cuts
            s["Z"] = [new(E, E, u, dtype=torch.int32) for u in cuts]
            nga = (B.ctypes.c_int32 * len(cuts))(*cuts)
            s["ws"] = new(int(B.lib().hm_swap_multi_workspace_bytes(T, K, E, G, len(cuts), nga)) // 4 + 4, dtype=torch.int32)
            s["ws_select"] = new(int(B.lib().hm_swap_select_workspace_bytes(E)) // 8 + 2, dtype=torch.float64)
            s["fan_in"] = torch.tensor(U, dtype=torch.int32, device="cuda")[:, None]
            s["intra"] = new(len(U), 64, dtype=torch.int32)
            s["times"], s["dim"] = torch.zeros(4, dtype=torch.float64, device="cuda"), new(1, dtype=torch.int32)
            s["Q"], s["pair"], s["time"] = new(E, E, dtype=torch.float64), new(2, dtype=torch.int32), new(1, dtype=torch.float64)
            s["outputs"] = {"own": s["own"], "times": s["times"], "dim": s["dim"], "Z": s["Z"], "Q": s["Q"], "pair": s["pair"],
                            "time": s["time"], "placed": s["placed"]}
    del s["g"]
    s["case"] = dict(c)
    return s


def run(s):
    c = s["case"]
    nodes, ranks = c["nodes"], c["ranks"]
    if c["path"] == "forward":
        B.hm_plan(s["ids"], s["w"], s["e2r"], nodes, ranks, s["level"], plan=s["plan"])
        B.hm_dispatch_pack(s["x"], s["plan"], s["packed"])
        B.hm_combine(s["y"], None, s["plan"], s["out"])
    elif c["path"] == "backward":
        if c["dtype"] == "f32":
            B.hm_combine_transpose(s["gout"], s["plan"], s["gy"])
            B.hm_combine_f32(s["gpacked"], s["keep"], s["plan"], s["gx"])
        else:
            B.hm_combine_transpose_bf16(s["gout"], s["plan"], s["gy"])
            B.hm_combine(s["gpacked"], s["keep"], s["plan"], s["gx"])
    elif c["path"] == "receiver":
        B.hm_plan_mapped(s["ids_a"], s["w_a"], s["table_a"], ranks, True, plan=s["plan_a"])
        B.hm_dispatch_pack(s["x_a"], s["plan_a"], s["packed_a"])
        B.hm_dispatch_pack(s["meta_in"][0], s["plan_a"], s["meta"][0])
        B.hm_dispatch_pack(s["meta_in"][1], s["plan_a"], s["meta"][1])
        B.hm_plan_mapped(s["ids_b"], s["w_b"], s["table_b"], s["local"], False, plan=s["plan_b"])
        B.hm_dispatch_pack(s["x_b"], s["plan_b"], s["packed_b"])
        B.hm_combine_mix(s["y_b"], None, s["plan_b"], s["back_b"])
        B.hm_combine_mix(s["y_a"], None, s["plan_a"], s["back_a"])
    elif c["path"] == "counts":
        B.hm_expert_load(s["ids"], s["e2r"], nodes, ranks, *s["load"], status=s["status"])
        B.hm_group_counts(s["ids"], s["e2r"], nodes * ranks, s["groups"], s["own"])
    else:
        U, G, M = s["U"], nodes * ranks, float(c["H"])
        D = len(U)
        B.hm_group_counts(s["ids"], s["placed"], G, s["groups"], s["own"])
        torch.mul(s["own"][0:1], s["fan_in"], out=s["intra"])   # rows held before Intra-level-l: own rows times the fan-in
        B.hm_alltoall_times(U, G, M, 2.0, s["own"], s["intra"], ALPHA_INTER[:D], BETA_INTER[:D], ALPHA_INTRA[:D],
                            BETA_INTRA[:D], s["times"], s["dim"])
        B.hm_swap_counts_multi(s["ids"], s["placed"], G, s["cuts"], s["Z"], workspace=s["ws"])
        z = dict(zip(s["cuts"], s["Z"]))
        B.hm_swap_select(U, G, M, 2.0, [None] + [z[u] for u in U[1:]], z[G], _scales(U), float(U[-1]), ALPHA_INTER[:D],
                         BETA_INTER[:D], ALPHA_INTRA[D - 1], BETA_INTRA[D - 1], GAMMA, s["Q"], s["pair"], s["time"],
                         workspace=s["ws_select"])
        B.hm_swap_apply(s["placed"], s["pair"])
    return s["outputs"]


def _zeroed(plan):
    plan.row_token.zero_()
    plan.row_weight.zero_()
    return plan


def _hierarchy(c):
    G, U = c["nodes"] * c["ranks"], [1]
    for u in (c["nodes"], 2 * c["nodes"], 4 * c["nodes"]):
        if u > U[-1] and u <= G and G % u == 0:
            U.append(u)
    return U


def _cuts(c):
    return sorted(set(_hierarchy(c)[1:] + [c["nodes"] * c["ranks"]]))


def _scales(U):
    return [0.0] + [float(u) for u in U[:-1]]


# ---- what a pass cannot do without -----------------------------------------------------------------
def _forward_bytes(T, H, K, per_token):
    """x read, packed written, y read, out written; the routing read, the maps and masks written."""
    return 2 * (1 + per_token) * T * H * 2 + T * K * (8 + 5) + T * 12 + per_token * T * 8


def _per_token(c, table, dedup, wanted=None):
    """Rows per token, estimated from 2,048 tokens of a fixed seed."""
    g = _generator(1, "cpu")
    bias = _bias(c, g, "cpu")
    ids = _route(c, 2048, g, "cpu", bias)[0] if wanted is None else _route_to(c, 2048, wanted, g, "cpu", bias)[0]
    return float(_kept(_dest(ids, table), dedup).sum()) / ids.shape[0]


def _per_level(c):
    e2r = _placement(c, "cpu")
    return _per_token(c, torch.div(e2r, c["ranks"], rounding_mode="floor") if c["level"] == "node" else e2r, c["level"] != "none")


def _per_hop(c):
    """(rows per received row inside the node, expert rows per row that reaches the rank)."""
    e2r = _placement(c, "cpu")
    on_node, on_rank = torch.div(e2r, c["ranks"], rounding_mode="floor") == 1 % c["nodes"], e2r == (1 % c["nodes"]) * c["ranks"]
    minus = torch.full_like(e2r, -1)
    return (_per_token(c, torch.where(on_node, e2r % c["ranks"], minus), True, on_node),
            _per_token(c, torch.where(on_rank, torch.cumsum(on_rank, 0, dtype=torch.int32) - 1, minus), False, on_rank))


def _capacity(c, tokens, per_token, dests):
    """Rows to make room for: a seventh more than expected; all there can be where popularity moves with the seed."""
    most = tokens * min(c["K"], dests)
    return most if c["router"] == "zipf" else min(most, int(1.15 * per_token * tokens) + 64)


def work(case):
    c = case
    T, H, E, K = c["T"], c["H"], c["E"], c["K"]
    if c["path"] in ("forward", "backward"):
        per = _per_level(c)
        if c["path"] == "forward":
            return {"bytes": _forward_bytes(T, H, K, per), "flops": 2 * per * T * H}
        size = 4 if c["dtype"] == "f32" else 2
        return {"bytes": 2 * (1 + per) * T * H * size + T * K * 9 + per * T * 4, "flops": 3 * per * T * H}
    if c["path"] == "receiver":
        per_a, per_b = _per_hop(c)
        rows_b = int(per_a * T)
        n = _forward_bytes(T, H, K, per_a) + _forward_bytes(rows_b, H, K, per_b) + (1 + per_a) * T * K * 8
        return {"bytes": n, "flops": 2 * H * (per_a * T + per_b * rows_b)}
    if c["path"] == "counts":
        return {"bytes": T * K * 4 + E * 8 + 256 * len(_hierarchy(c)), "flops": 2 * T * K}
    entries = E * E * sum(_cuts(c))   # Z is written; a gamma-th power and a sum per entry that Q reads
    return {"bytes": T * K * 4 + 4 * entries + 8 * E * E, "flops": 8 * entries + 2 * T * K * K}


def tolerance(case):
    """Four times what the path shows against exact(); whole numbers are the same."""
    if case["path"] == "planner":
        return {"rel": 1e-14, "max": 1e-13}
    if case["path"] == "counts":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-7, "max": 3e-6}
    return {"rel": 7e-3, "max": 2e-2}


# ---- the same in 64 bits, by plain torch -----------------------------------------------------------
def _dest(ids, table):
    return torch.where(ids >= 0, table[ids.clamp(min=0).long()], torch.full_like(ids, -1))


def _kept(dest, dedup):
    """The slots that own a row: all with a destination, or the first of a token for each destination."""
    keep = dest >= 0
    if dedup:
        for k in range(1, dest.shape[1]):
            keep[:, k] &= ~(dest[:, :k] == dest[:, k:k + 1]).any(1)
    return keep


def _lists(dest, w, dedup):
    """(token of each row, fp64 weight of each row): rows by destination, then by slot."""
    T, K = dest.shape
    keep = _kept(dest, dedup)
    flat = torch.nonzero(keep.reshape(-1)).reshape(-1)
    flat = flat[torch.sort(dest.reshape(-1)[flat], stable=True).indices]
    token = torch.div(flat, K, rounding_mode="floor")
    w = w.double()
    if not dedup:
        return token, w.reshape(-1)[flat]
    same = dest[token] == dest.reshape(-1)[flat][:, None]
    return token, (w[token] * same).sum(1)


def _merge(T, H, token, weight, y, by=None):
    """sum over a token's rows of weight * y, in fp64, a slice of the columns at a time; divided by `by`."""
    out = torch.zeros((T, H), dtype=torch.float64, device=y.device)
    step = max(1, (1 << 28) // max(1, y.shape[0]))
    for a in range(0, H, step):
        out[:, a:a + step].index_add_(0, token, y[:, a:a + step].double() * weight[:, None])
    return out if by is None else out / by[:, None]


def _padded(rows, cap):
    out = torch.zeros((cap,) + rows.shape[1:], dtype=rows.dtype, device=rows.device)
    out[:rows.shape[0]] = rows
    return out


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    T, H, g, nodes, G = c["T"], c["H"], s["g"], c["nodes"], c["nodes"] * c["ranks"]
    if c["path"] == "counts":
        return None
    if c["path"] == "planner":
        return _exact_planner(c, s)
    if c["path"] == "receiver":
        want = {}
        for st, dedup in (("a", True), ("b", False)):
            n = s["ids_" + st].shape[0]
            token, weight = _lists(_dest(s["ids_" + st], s["map_" + st]), s["w_" + st], dedup)
            x, y = _rows(n, H, g), _rows(token.numel(), H, g)
            total = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, token, weight)
            cap = _capacity(c, n, s["per_" + st], c["ranks"] if st == "a" else s["local"])
            want.update({"packed_" + st: _padded(x[token], cap), "row_weight_" + st: _padded(weight, cap), "back_" + st: _merge(n, H, token, weight, y, total)})
        return want
    table = torch.div(s["e2r"], c["ranks"], rounding_mode="floor") if c["level"] == "node" else s["e2r"]
    token, weight = _lists(_dest(s["ids"], table), s["w"], c["level"] != "none")
    cap = _capacity(c, T, _per_level(c), G if c["level"] != "node" else nodes)
    if c["path"] == "forward":
        x, y = _rows(T, H, g), _rows(token.numel(), H, g)
        return {"packed": _padded(x[token], cap), "out": _merge(T, H, token, weight, y), "row_weight": _padded(weight, cap)}
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    gout, gpacked = _rows(T, H, g, dt, 1e-2), _rows(token.numel(), H, g, dt, 1e-2)
    return {"gy": _padded(gout.double()[token] * weight[:, None], cap), "gx": _merge(T, H, token, torch.ones_like(weight), gpacked)}


def _exact_planner(c, s):
    T, E, G, M, v = c["T"], c["E"], c["nodes"] * c["ranks"], float(c["H"]), 2.0
    U, ids = _hierarchy(c), s["ids"].long()
    rank = s["e2r"].long()
    S = torch.zeros((T, E + 1), dtype=torch.float64, device="cuda")
    S.scatter_(1, torch.where(ids < 0, E, ids), 1.0)
    S = S[:, :E].contiguous()

    def groups(ng):   # selected experts per group, the group of each expert
        of = torch.div(rank, G // ng, rounding_mode="floor")
        return torch.zeros((T, ng), dtype=torch.float64, device="cuda").index_add_(1, of, S), of

    def smooth_max(x):   # over the last axis, as max * (sum (x/max)^gamma)^(1/gamma)
        m = x.max(-1, keepdim=True).values
        return (m * ((x / m.clamp(min=1e-300)) ** GAMMA).sum(-1, keepdim=True) ** (1.0 / GAMMA)).squeeze(-1)

    def swapped(ng):
        n, of = groups(ng)
        base = (n > 0).double().sum(0)
        none_of = S.T @ (n == 0).double()                               # tokens that select r and nothing in group j
        lone = (S * (n[:, of] == 1).double()).T @ (1.0 - S)             # lone[a][b]: a alone in its group, b not selected
        Z = base.repeat(E, E, 1)
        r, q = torch.arange(E, device="cuda")[:, None], torch.arange(E, device="cuda")[None, :]
        gr, gq = of[r].expand(E, E), of[q].expand(E, E)
        move = gr != gq
        R, C = torch.nonzero(move, as_tuple=True)
        Z[R, C, gq[move]] += none_of[R, gq[move]] - lone[C, R]
        Z[R, C, gr[move]] += none_of[C, gr[move]] - lone[R, C]
        return Z

    own = {u: (groups(u)[0] > 0).double().sum(0) for u in set(U + [G])}
    times = torch.zeros(4, dtype=torch.float64)
    for d in range(1, len(U) + 1):
        t = sum(ALPHA_INTER[i] + U[i] / U[i - 1] * float(own[U[i]].max()) * M * v * BETA_INTER[i] for i in range(1, d))
        times[d - 1] = t + ALPHA_INTRA[d - 1] + G / U[d - 1] * float(own[G].max()) * U[d - 1] * M * v * BETA_INTRA[d - 1]
    D, scale = len(U), _scales(U)
    Q = torch.zeros((E, E), dtype=torch.float64, device="cuda")
    for i in range(1, D):
        Q += U[i] / U[i - 1] * scale[i] * smooth_max(swapped(U[i])) * M * v * BETA_INTER[i] + ALPHA_INTER[i]
    Q += G / U[-1] * U[-1] * smooth_max(swapped(G)) * M * v * BETA_INTRA[D - 1] + ALPHA_INTRA[D - 1]
    return {"times": times, "Q": Q, "time": Q.min().reshape(1)}

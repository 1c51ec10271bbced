"""The work a user of the library has it do, as cases that can be timed and compared.

Every case is one pass through the public entry points over one batch of tokens of
one rank: a decode or prefill step of `GraceMoELayer` (eager, or replayed from a HIP
graph), the same step through the functional calls on a GPU that hosts every expert,
or the routing side alone (route, send lists, dispatch order).  Expert loads are
Zipf-skewed and the placement table comes from the planner, fed with a profile of the
same gate, so that hot experts have replicas and segments are ragged as in use.

Shapes are those of the repository's workloads (OLMoE-, Mixtral-, Qwen-, Qwen3-MoE- and
DeepSeek-V2-Lite-shaped layers, the small fp32 layer) plus tensor-parallel slices of the
expert width and a generic fp32 layer; batches run from a single token to 32768.
"""
import math

import numpy as np
import torch

import paper_2509_25041_amd as grace
from paper_2509_25041_amd import planner

# d_model, expert width, experts, top-k, shared experts, zipf exponent, nodes, GPUs per node
SHAPES = {
    "olmoe": dict(d=2048, f=1024, E=64, k=8, n_shared=0, zipf=1.2, nodes=2, gpus=2),
    "mixtral": dict(d=4096, f=14336, E=8, k=2, n_shared=0, zipf=0.8, nodes=2, gpus=4),
    "qwen": dict(d=2048, f=1408, E=60, k=4, n_shared=4, zipf=1.5, nodes=4, gpus=2),
    "qwen3moe": dict(d=2048, f=768, E=128, k=8, n_shared=0, zipf=1.2, nodes=2, gpus=4),
    "dsv2lite": dict(d=2048, f=1408, E=64, k=6, n_shared=2, zipf=1.2, nodes=4, gpus=8),
    "tiny": dict(d=128, f=256, E=8, k=2, n_shared=0, zipf=1.2, nodes=2, gpus=2),
    "f32mid": dict(d=1024, f=2816, E=16, k=2, n_shared=0, zipf=1.0, nodes=1, gpus=2),
}


def _case(name, shape, T, mode="layer", dtype="bf16", rank=0, renorm=1, policy=0, table_seed=1, **over):
    c = dict(SHAPES[shape])
    c.update(over)
    c.update(T=T, mode=mode, dtype=dtype, rank=rank, renorm=renorm, policy=policy, table_seed=table_seed)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # (tables and ranks are ones whose share of the rows is near the mean of all ranks)
        # one sequence being decoded: the smallest call, latency only
        _case("decode_1", "olmoe", 1, table_seed=15),
        # a small decode batch inside a serving loop that replays a captured step
        _case("decode_16_graph", "qwen3moe", 16, mode="graph", rank=6, table_seed=19),
        # decode batches of the sizes the paper spreads over its ranks
        _case("decode_64", "olmoe", 64, rank=3, table_seed=10),
        _case("decode_512", "olmoe", 512, rank=1, table_seed=11),
        # one GPU that hosts all experts, an odd batch, through the functional calls
        _case("single_gpu_1000", "olmoe", 1000, mode="functional", nodes=1, gpus=1, renorm=0, table_seed=5),
        # fp32 layers: the small reference layer and one of ordinary width with an odd batch
        _case("f32_tiny_256", "tiny", 256, dtype="f32", table_seed=20),
        _case("f32_1000", "f32mid", 1000, dtype="f32", rank=1, table_seed=15),
        # expert width cut four ways by tensor parallelism (1408 / 4): K of the down projections is no multiple of 64
        _case("split_width_3001", "dsv2lite", 3001, f=352, rank=6, table_seed=2),
        # prefill: few wide experts; many narrow experts with an odd batch; shared experts at the largest batch
        _case("prefill_8192_wide", "mixtral", 8192, rank=6, table_seed=11),
        _case("prefill_7001_narrow", "qwen3moe", 7001, rank=4, table_seed=14),
        _case("prefill_32768_shared", "dsv2lite", 32768, rank=27, table_seed=6),
        # planning a deployment: routing without locality, de-duplicated send lists, dispatch order without rows
        _case("send_lists_16384", "qwen", 16384, mode="lists", policy=1, rank=4, table_seed=1),
    ]


def draw(rng):
    def batch(most):
        t = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
        return max(1, min(most, t + rng.choice([0, 0, 1, -1])))

    seed = rng.randrange(1000)
    kind = rng.choice(["layer", "layer", "layer", "layer", "graph", "functional", "f32", "lists"])
    renorm, policy = rng.choice([1, 1, 0]), rng.choice([0, 0, 0, 1])
    if kind == "f32":
        shape = rng.choice(["tiny", "f32mid"])
        c = dict(SHAPES[shape])
        over = dict(d=rng.choice([c["d"], c["d"] // 2 + 36]), f=rng.choice([c["f"], c["f"] // 2 - 20]))
        return _case(None, shape, batch(1000), dtype="f32", rank=rng.randrange(c["nodes"] * c["gpus"]), renorm=renorm,
                     policy=policy, table_seed=seed, **over)
    shape = rng.choice(["olmoe", "mixtral", "qwen", "qwen3moe", "dsv2lite"])
    c = dict(SHAPES[shape])
    if kind == "lists":
        return _case(None, shape, batch(16384), mode="lists", policy=policy, rank=rng.randrange(c["nodes"] * c["gpus"]),
                     table_seed=seed)
    over = dict(f=c["f"] // rng.choice([1, 1, 1, 2, 4]))
    if kind == "functional":
        if shape == "mixtral":
            over["f"] = c["f"] // 4
        return _case(None, shape, batch(2048), mode="functional", nodes=1, gpus=1, renorm=renorm, table_seed=seed, **over)
    most = {"olmoe": 8192, "mixtral": 8192, "qwen": 8192, "qwen3moe": 8192, "dsv2lite": 32768}[shape]
    return _case(None, shape, batch(64 if kind == "graph" else most), mode=kind, rank=rng.randrange(c["nodes"] * c["gpus"]),
                 renorm=renorm, policy=policy, table_seed=seed, **over)


# ---------------------------------------------------------------- placement, from a profile of the gate --
def _gate_bias(case):
    """Zipf-shaped logit bias: expert popularity is a property of the model, not of one batch."""
    rng = np.random.default_rng([case["table_seed"], 1])
    rank = np.empty(case["E"])
    rank[rng.permutation(case["E"])] = np.arange(1, case["E"] + 1)
    return (-case["zipf"] * np.log(rank)).astype(np.float32)


def _profile(case, tokens=2048):
    """Average choices of each expert per token, from a profiling batch of the same gate."""
    rng = np.random.default_rng([case["table_seed"], 2])
    logits = rng.standard_normal((tokens, case["E"]), dtype=np.float32) + _gate_bias(case)
    top = np.argpartition(-logits, case["k"] - 1, axis=1)[:, :case["k"]]
    return np.bincount(top.reshape(-1), minlength=case["E"]) / tokens


def _plan(case):
    E, R = case["E"], case["nodes"] * case["gpus"]
    ends = [E * (r + 1) // R for r in range(R)]
    groups = [list(range(a, b)) for a, b in zip([0] + ends[:-1], ends)]
    return planner.plan_layer(_profile(case), groups, case["nodes"], case["gpus"])


def _local_rows(case):
    """Expected rows per local slot of one batch (for `work`): expert load times the share that this rank's
    instance takes (all of it when the policy prefers a local instance)."""
    pl, load = _plan(case), _profile(case)
    rows = []
    for e in range(case["E"]):
        ranks = list(pl.inst_rank[pl.inst_ptr[e]:pl.inst_ptr[e + 1]])
        if case["rank"] in ranks:
            w = [int(pl.poll_weight[r]) for r in ranks]
            share = w[ranks.index(case["rank"])] / sum(w) if case["policy"] == 1 else 1.0
            rows.append(case["T"] * load[e] * share)
    return rows


# ---------------------------------------------------------------------------------- what the user holds --
def prepare(case, seed):
    c = case
    pl = _plan(c)
    table = grace.GraceTable.from_placement(pl)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    def weight(*shape):
        # drawn one leading slice at a time: the wide shapes would need gigabytes of fp32 at once
        w = torch.empty(shape, dtype=dt, device="cuda")
        for s in range(shape[0]):
            w[s] = normal(*shape[1:]) * 0.02
        return w

    state = dict(mode=c["mode"], k=c["k"], rank=c["rank"], renorm=c["renorm"], policy=c["policy"], table=table, T=c["T"])
    state["logits"] = normal(c["T"], c["E"]) + torch.from_numpy(_gate_bias(c)).cuda()
    # round-robin counters carried over from earlier batches
    state["rr_in"] = torch.randint(0, 8, (c["E"],), generator=gen, device="cuda", dtype=torch.int32)
    state["rr_out"] = torch.zeros(c["E"], dtype=torch.int32, device="cuda")
    if c["mode"] == "lists":
        return state
    state["x"] = normal(c["T"], c["d"]).to(dt)
    S = len(table.local_experts(c["rank"]))
    state["w"] = (weight(S, c["f"], c["d"]), weight(S, c["f"], c["d"]), weight(S, c["d"], c["f"]))
    n = c["n_shared"]
    state["shared"] = (weight(n, c["f"], c["d"]), weight(n, c["f"], c["d"]), weight(n, c["d"], c["f"])) if n else None
    if c["mode"] != "functional":
        state["layer"] = grace.GraceMoELayer(table, c["rank"], c["T"], c["k"], c["d"], c["f"], dt, *state["w"],
                                             shared=state["shared"], renorm=c["renorm"], policy=c["policy"])
    if c["mode"] == "graph":
        state["graph"] = state["layer"].capture(state["logits"], state["x"], state["rr_in"], state["rr_out"])
    return state


# -------------------------------------------------------------------------------------------- one pass --
def _layer_outputs(s):
    layer = s["layer"]
    # the dispatch buffer xp is an output as well (its rows for other ranks are what the exchange sends), and so
    # is y, the rank share of the expert outputs
    return {"out": layer.out, "route": layer.route_out, "perm": layer.perm_out, "xp": layer.xp, "y": layer.y,
            "rr_out": s["rr_out"]}


def run(state):
    s = state
    if s["mode"] == "layer":
        s["layer"].forward(s["logits"], s["x"], s["rr_in"], s["rr_out"])
        return _layer_outputs(s)
    if s["mode"] == "graph":
        s["graph"].replay()
        return _layer_outputs(s)
    if s["mode"] == "functional":
        route, perm = grace.grace_route_permute(s["table"], s["rank"], s["logits"], s["k"], s["x"], renorm=s["renorm"],
                                                rr_in=s["rr_in"], rr_out=s["rr_out"], policy=s["policy"])
        pos, inst_off, xp = perm[0], perm[2], perm[5]
        y = grace.grace_expert_ffn(s["table"], s["rank"], xp, inst_off, s["T"], s["k"], *s["w"])
        ys = grace.grace_shared_ffn(s["x"], *s["shared"]) if s["shared"] else None
        return {"out": grace.grace_combine(y, pos, route[1], ys), "route": route, "perm": perm, "y": y, "rr_out": s["rr_out"]}
    route = grace.grace_route(s["table"], s["rank"], s["logits"], s["k"], renorm=s["renorm"], rr_in=s["rr_in"],
                              rr_out=s["rr_out"], policy=s["policy"])
    lists = grace.grace_send_lists(s["table"], s["rank"], route[2])
    perm = grace.grace_permute(s["table"], route[2], None)
    return {"route": route, "lists": lists, "perm": perm[:5], "rr_out": s["rr_out"]}


# ------------------------------------------------------------------------------------- what it cannot do without --
def work(case):
    c = case
    T, k, d, f, E = c["T"], c["k"], c["d"], c["f"], c["E"]
    el = 4 if c["dtype"] == "f32" else 2
    n = T * k
    nbytes = 4 * T * E + 12 * n + 8 * n             # logits; expert, weight and instance of every choice; both permutations
    if c["mode"] == "lists":
        return {"bytes": nbytes + 12 * n, "flops": 0}   # send lists per rank and node, expansion map
    rows = _local_rows(c)
    m = sum(rows)
    hit = sum(1.0 - math.exp(-r) for r in rows)     # slots that get a row and whose weights are read
    nbytes += el * (2 * T * d + n * d)              # tokens in, result out, dispatch rows out
    if c["mode"] == "functional":
        nbytes += el * n * d                        # expert outputs, returned as well
    nbytes += el * 3 * d * f * (hit + c["n_shared"])
    return {"bytes": nbytes, "flops": 6.0 * d * f * (m + c["n_shared"] * T)}


def tolerance(case):
    # Whole numbers and moved rows are the same.  For the rest, about four times what the path differs by from
    # the same layer in 64 bits: gate weights 6e-8; fp32 results 1.3e-6 (largest element 1e-5); bf16 results 3e-3
    # (two roundings, of the hidden activation and of the expert output; largest element 4e-2).
    if case["mode"] == "lists":
        return {"rel": 3e-7, "max": 1e-5, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 1e-1, "differ": 0.0}

"""What this framework is measured on: the work that its users have it do, through its public entry points
(paper_1807_05358_amd.binding and .search), over the range of sizes they use.

A user of the simulator either prices a batch of candidate strategies (`Simulator.batch`), follows a chain of changes
(`Chains.delta`), prices the proposals of a search before taking one (`Chains.try_mutations`), runs the search on the
device (`Chains.search`, `search.find_strategy`) or checks a strategy against all of its neighbours
(`Chains.neighbours`).  The graphs, machines and batch sizes of the listed cases are those of the five benchmark
configurations (paper_1807_05358_amd/workloads.py) and of bench.py; `draw` varies graph, machine, batch, chain length
and the refinements of the inputs over the same ranges.

A case is a dict of plain values:
  path     batch | delta | try | search | find | neighbours
  graph    chain | alexnet | inception | resnet | nmt; steps: unrolled steps of the nmt graph (0 otherwise)
  nodes, gpus, parts   the simulated machine and the largest number of parts of an op
  option   plain     powers of two as degrees, consecutive devices
           general   any degrees, any device strides: parts of an op may share devices
           tuple     costs keyed by the degree tuple
           links     links inside nodes and between nodes that differ per pair
           params    with the traffic that keeps the replicas of parameters in step
           train     the graph of a whole training iteration (gradient edges, tied configurations, params)
           devmaps   the device of every task given explicitly (batch only)
  B        candidates of a batch, chains of the other paths
  n        mutations of a chain, proposals per chain, steps of a search; ops whose neighbours are visited, from op
           `first` on
All results are whole nanoseconds and must be exactly the same.
"""
import math

import numpy as np
import torch

from paper_1807_05358_amd import binding, search
from paper_1807_05358_amd import workloads as W

POWERS = (1, 2, 4, 8, 16, 32, 64)
ANY_DEGREE = (1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32, 48, 64)
GRAPHS = {"chain": W.graph_tiny_chain, "alexnet": W.graph_alexnet, "inception": W.graph_inception_v3,
          "resnet": W.graph_resnet101, "nmt": W.graph_nmt}


def _case(path, graph, nodes, gpus, parts, option, B, n=0, steps=0):
    return {"path": path, "graph": graph, "steps": steps, "nodes": nodes, "gpus": gpus, "parts": parts, "option": option,
            "B": B, "n": n, "first": 0}


def listed():
    cases = {
        # the smallest call: a handful of candidates of a six-op graph, where the launch and the latency of one
        # simulation count (the tiny configuration's batch)
        "batch_chain_64": _case("batch", "chain", 1, 4, 4, "plain", 64),
        # a graph of a dozen ops on a small cluster: one wavefront per SIMD, state in LDS
        "batch_alexnet_1024": _case("batch", "alexnet", 4, 4, 16, "plain", 1024),
        # the two convolutional graphs on 64 devices, the batch a search over many chains prices at a time
        "batch_inception_4096": _case("batch", "inception", 16, 4, 64, "plain", 4096),
        "batch_resnet_4096": _case("batch", "resnet", 16, 4, 64, "plain", 4096),
        # the largest graph (2321 ops), bench.py's headline workload
        "batch_nmt_1024": _case("batch", "nmt", 16, 4, 64, "plain", 1024, steps=40),
        # a whole training iteration: forward and backward ops, gradient edges, parameter traffic
        "batch_inception_train_1024": _case("batch", "inception", 16, 4, 64, "train", 1024),
        # odd sizes throughout: degrees that do not divide the extents, device strides, three GPUs per node,
        # a batch that is no multiple of anything
        "batch_resnet_general_777": _case("batch", "resnet", 5, 3, 48, "general", 777),
        # one chain of single-op changes on the largest graph, each priced in turn (bench.py's mutation chain): out
        # and back again, so that every pass starts from the same strategy and every step is a real change
        "delta_nmt_1x16": _case("delta", "nmt", 16, 4, 64, "plain", 1, n=16, steps=40),
        # proposals against one stored timeline of the largest graph, several per resident wavefront
        "try_nmt_4096": _case("try", "nmt", 16, 4, 64, "plain", 1, n=4096, steps=40),
        # the search loop on the device, chains enough to fill it: created, run, best strategies read
        "search_inception_1024x16": _case("search", "inception", 16, 4, 64, "plain", 1024, n=16),
        # the search driver with its default chains and budget, parameter traffic simulated (what makes strategies
        # other than data parallelism pay)
        "find_alexnet_64x256": _case("find", "alexnet", 4, 4, 16, "params", 64, n=256),
        # is a strategy locally optimal: all single-op neighbours of one strategy, results on the host
        "neighbours_alexnet": _case("neighbours", "alexnet", 4, 4, 16, "plain", 1, n=12),
    }
    return [dict(c, name=name) for name, c in cases.items()]


# compute tasks and producer/consumer pairs of one strategy of each graph (measured means of the benchmark
# configurations; nmt per 40 unrolled steps), for the budget of draw() and the operations of work()
TASKS = {"chain": 18, "alexnet": 119, "inception": 4409, "resnet": 12248, "nmt": 62551}
PAIRS = {"chain": 38, "alexnet": 680, "inception": 70993, "resnet": 134588, "nmt": 534171}
OPS = {"chain": 6, "alexnet": 12, "inception": 121, "resnet": 345, "nmt": 2321}


def _per_simulation(case):
    """(compute tasks, pairs) of one simulated strategy, about"""
    f = case["steps"] / 40 if case["graph"] == "nmt" else 1.0
    f *= 2 if case["option"] == "train" else 1
    if case["graph"] not in ("chain", "alexnet"):
        f *= (case["parts"] / 64) ** 0.7
    return max(1.0, f * TASKS[case["graph"]]), max(1.0, f * PAIRS[case["graph"]])


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["batch"] * 6 + ["delta", "try", "search", "neighbours"])
    graph = rng.choice(["chain", "alexnet", "inception", "resnet", "nmt"])
    small = graph in ("chain", "alexnet")
    steps = rng.randint(3, 40) if graph == "nmt" else 0
    nodes, gpus = rng.choice([(1, 4), (2, 4), (4, 4), (3, 2), (2, 8)] if small else [(4, 4), (8, 4), (16, 4), (16, 4), (5, 3), (4, 8)])
    parts = min(nodes * gpus, 16) if small else min(64, nodes * gpus)
    options = ["plain"] * 4 + ["tuple", "links", "params", "general"]
    if path == "batch":
        options += ["train", "devmaps"] if graph != "nmt" else []
    case = _case(path, graph, nodes, gpus, parts, rng.choice(options), 1, 0, steps)
    # no more simulated pairs than a third of the largest listed case: the general forms take longer per pair
    most = 1.8e8 / _per_simulation(case)[1]
    if path == "batch":
        case["B"] = _log(rng, 1, min(16384, most))
    elif path == "delta":
        case["B"] = _log(rng, 1, max(1, min(256, most / 4)))
        case["n"] = 2 * _log(rng, 1, 6 if graph == "nmt" else 24)
    elif path == "try":
        case["B"] = _log(rng, 1, max(1, min(16, most / 8)))
        case["n"] = _log(rng, 4, max(4, min(8192, most / case["B"])))
    elif path == "search":
        case["B"] = _log(rng, 1, max(1, min(1024, most / 4)))
        case["n"] = _log(rng, 2, max(2, min(6 if graph == "nmt" else 64, most / case["B"])))
    else:
        case["n"] = rng.randint(1, 12) if small else 1
        if graph == "nmt":
            case["steps"] = rng.randint(3, 12)
        case["first"] = rng.randrange(50 * case["steps"] if graph == "nmt" else max(1, OPS[graph] - case["n"]))
    return case


def _inputs(case, seed):
    """graph, machine, costs and the space strategies are drawn from"""
    option = case["option"]
    ops, edges, flops = GRAPHS[case["graph"]](steps=case["steps"]) if case["graph"] == "nmt" else GRAPHS[case["graph"]]()
    mach = W.Machine(case["nodes"], case["gpus"])
    choices = ANY_DEGREE if option == "general" else POWERS
    params = ties = None
    if option == "general":
        mach.intra_lat_ns, mach.inter_lat_ns = 700, 5000
    if option == "links":
        mach.link_Bpns, mach.link_lat_ns = W.paired_links(case["gpus"], 40, 16, 0, 300)
        mach.node_Bpns, mach.node_lat_ns = W.ring_node_links(case["nodes"], 12, 6, 1000)
    if option == "train":
        ops, edges, flops, ties, params = W.training_graph(ops, edges, flops)
    elif option == "params":
        params = W.param_table(ops, flops)
    cost = np.ascontiguousarray(W.cost_table(1 if case["graph"] in ("chain", "alexnet") else 2, flops, seed)[:, :case["parts"]])
    if option == "tuple":
        cost = W.tuple_cost_table(ops, cost, case["parts"], choices, seed)
    return ops, edges, mach, cost, choices, params, ties


def _strategies(case, ops, choices, n, seed, rng):
    cfgs = W.strategies(ops, n, seed, case["nodes"] * case["gpus"], case["parts"], choices)
    if case["option"] == "general":
        cfgs["dev_stride"] = rng.integers(0, 8, size=cfgs.shape)
    return cfgs


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    ops, edges, mach, cost, choices, params, ties = _inputs(case, seed)
    B, n, D = case["B"], case["n"], case["nodes"] * case["gpus"]
    s = {"case": case, "seed": seed, "ops": ops, "machine": mach, "choices": choices}
    sim = s["sim"] = binding.Simulator(ops, edges, mach, cost, params=params, ties=ties)
    cfgs = _strategies(case, ops, choices, B, seed, rng)
    if case["path"] == "batch":
        s["d"] = sim.upload_strategies(cfgs)
        s["out"] = torch.empty(B, dtype=torch.int64, device="cuda")
        s["maps"] = binding.to_device(W.device_maps(cfgs, D, seed)) if case["option"] == "devmaps" else None
        sim._ensure_workspace(B)
        return s
    s["cfgs"] = cfgs
    if case["path"] in ("search", "neighbours"):
        s["space"] = W.search_space(ops, case["parts"], choices)
    if case["path"] in ("delta", "try", "neighbours"):
        s["chains"] = binding.Chains(sim, cfgs)
    if case["path"] == "delta":
        # n/2 changes, then each of them taken back in reverse order
        out = W.mutation_chains(ops, n // 2, B, seed, D, case["parts"], choices)
        back = out.copy()
        cur = cfgs.copy()
        for t in range(n // 2):
            for c in range(B):
                op = int(out[t, c]["op"])
                back[t, c]["cfg"] = cur[c, op]
                cur[c, op] = out[t, c]["cfg"]
        s["d"] = s["chains"].upload_mutations(np.concatenate([out, back[::-1]]))
        s["out"] = torch.empty((2 * (n // 2), B), dtype=torch.int64, device="cuda")
    elif case["path"] == "try":
        s["d"] = s["chains"].upload_mutations(W.mutation_chains(ops, n, B, seed, D, case["parts"], choices))
        s["out"] = torch.empty((n, B), dtype=torch.int64, device="cuda")
        s["chains"]._ensure_try_workspace(n)
    elif case["path"] == "search":
        # a proposal slower by a 50th of the starting time is taken with probability 1/e (bench.py's setting); the
        # tolerance is an input of the search and comes from a first simulation of its starting strategies
        t0 = float(np.median(sim.simulate(cfgs[:min(B, 64)])))
        s["bucket"] = max(1, int(t0) // 256)
        s["accept"] = binding.ff_sim_accept_table(50.0 / t0, s["bucket"], 256)
    return s


def run(s):
    case, sim = s["case"], s["sim"]
    path, n = case["path"], case["n"]
    if path == "batch":
        return sim.batch(s["d"], case["B"], d_out=s["out"], d_devmaps=s["maps"])
    if path == "delta":
        return s["chains"].delta(s["d"], s["out"].shape[0], d_out=s["out"])
    if path == "try":
        return s["chains"].try_mutations(s["d"], n, d_out=s["out"])
    if path == "search":
        ch = binding.Chains(sim, s["cfgs"])
        ch.search_setup(*s["space"], s["accept"], s["bucket"], s["seed"])
        trace = ch.search(n)
        best_ns, best = ch.best()
        start = ch.start_ns()
        ch.close()
        return {"start": start.view(np.int64), "trace": trace, "best_ns": best_ns.view(np.int64), "best": best.view(np.int64)}
    if path == "find":
        r = search.find_strategy(sim, s["ops"], s["machine"], case["parts"], s["choices"], n_chains=case["B"], steps=n, seed=s["seed"] % 2 ** 32)
        return {"best_ns": r.best_ns, "best": np.ascontiguousarray(r.best).view(np.int64), "chain_best": r.chain_best_ns.view(np.int64),
                "trace": r.trace_ns.view(np.int64)}
    muts, ns, best_ns, best = s["chains"].neighbours(*s["space"], case["first"], min(case["first"] + n, len(s["ops"])))
    return {"muts": np.ascontiguousarray(muts).view(np.uint32).astype(np.int64), "ns": ns.view(np.int64), "best_ns": best_ns.view(np.int64),
            "best": best.astype(np.int64)}


def work(case):
    """Bytes: strategies or mutations in, times (and best strategies) out.  Operations: per simulated task its way
    through the queue, and per producer/consumer pair the intersection of two boxes, a transfer time and two maxima; a
    simulation after one change needs about half of the timeline."""
    path, B, n = case["path"], case["B"], case["n"]
    n_ops = OPS[case["graph"]] * (case["steps"] / 40 if case["graph"] == "nmt" else 1) * (2 if case["option"] == "train" else 1)
    tasks, pairs = _per_simulation(case)
    if path == "batch":
        sims, moved = B, B * (8 * n_ops + 8) + (B * n_ops * 128 if case["option"] == "devmaps" else 0)
    elif path in ("delta", "try"):
        sims, moved = 0.5 * B * n, B * n * 20
    elif path in ("search", "find"):
        sims, moved = B * (1 + 0.5 * n), B * (16 * n_ops + 8 * n)
    else:
        m = n * case["nodes"] * case["gpus"] * 35
        sims, moved = 0.5 * m, m * 20
    return {"bytes": float(moved), "flops": float(sims * (16 * pairs + 2 * tasks * max(1.0, math.log2(tasks))))}


def tolerance(case):
    return "exact"

"""ff_sim_search with the steps to come simulated side by side (k_search_walk, k_loop_nodes): traces, best and final strategies of every chain are those
of steps made one after the other (Sections 6.1, 6.2).  Compared with calls of seven steps, which are made in turn, and with the oracle's chain."""
import numpy as np
import pytest

import oracle
from oracle import search as S
from helpers import random_graph
from paper_1807_05358_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_05358_amd import binding
    return binding


def _setup(form, seed):
    """ops, edges, machine, cost, Simulator keywords, choices of degrees"""
    rng = np.random.default_rng(seed)
    if form in ("tiny", "alexnet", "inception"):
        w = W.workload({"tiny": 0, "alexnet": 1, "inception": 2}[form])
        return w.ops, w.edges, w.machine, w.cost, {"params": W.param_table(w.ops, w.flops)} if form == "alexnet" else {}, w.choices
    if form == "train":
        w = W.workload(0)
        ops, edges, flops, ties, params = W.training_graph(w.ops, w.edges, w.flops)
        return ops, edges, w.machine, np.ascontiguousarray(W.cost_table(0, flops, seed)[:, :w.max_parts]), {"params": params, "ties": ties}, w.choices
    if form == "far":
        # transfers of seconds: links booked beyond 32 bits
        ops, edges, _ = random_graph(rng, 30)
        return ops, edges, W.Machine(2, 3, 1, 1, 2 ** 31, 2 ** 31), rng.integers(1, 2 ** 31, size=(30, 16)).astype("<u4"), {}, (1, 2, 3, 4, 5, 7)
    ops, edges, _ = random_graph(rng, 80)
    return ops, edges, W.Machine(3, 3, 11, 7, 20, 400), rng.integers(1, 9000, size=(80, 16)).astype("<u4"), {}, (1, 2, 3, 4, 5, 7)


def _search(ch, steps, per_call):
    return np.concatenate([ch.search(min(per_call, steps - a)).cpu().numpy().view("<u8") for a in range(0, steps, per_call)])


# tolerance: what is taken -- nearly nothing, some, everything; chains: one (63 nodes), few, so many that each has four nodes; steps: the fewest that
# are looked ahead at, and more than the 64 proposals drawn at a time
@pytest.mark.parametrize("form,C,n,scale,patience", [("tiny", 1, 8, 0.02, 0), ("tiny", 3, 150, 0.002, 0), ("tiny", 800, 36, 0.02, 9), ("alexnet", 64, 70, 0.02, 20),
                                                     ("inception", 5, 20, 0.02, 0), ("inception", 1, 90, 0.0, 0), ("train", 4, 40, 0.05, 0),
                                                     ("memory", 7, 33, 10.0, 0), ("memory", 2, 64, 0.01, 12), ("far", 3, 24, 0.05, 0)])
def test_steps_ahead_equal_steps_in_turn(B, form, C, n, scale, patience):
    ops, edges, mach, cost, kw, choices = _setup(form, 17 * n + C)
    parts = cost.shape[1]
    cfg0 = W.strategies(ops, C, 5, mach.n_devices, parts, choices)
    if form == "memory":
        cfg0["dev_stride"] = np.random.default_rng(1).integers(0, 4, cfg0.shape)        # general strategies, until the proposals mend them
    tp, tu = W.search_space(ops, parts, choices)
    if C > 2:
        cfg0["deg"][1, 0, 0] = 0                          # one chain starts from an invalid strategy
    sim = B.Simulator(ops, edges, mach, cost, **kw)
    one, two = B.Chains(sim, cfg0), B.Chains(sim, cfg0)
    t0 = int(one.start_ns()[0])
    bucket = max(1, t0 // 256)
    table = B.ff_sim_accept_table(1.0 / max(1.0, t0 * scale), bucket, 256)
    print(f"search: {form}, {C} chains x {n} steps, twice", flush=True)
    for ch in (one, two):
        ch.search_setup(tp, tu, table, bucket, 77, patience=patience)
    probe = one.upload_mutations(W.mutation_chains(ops, 4, C, 6, mach.n_devices, parts, choices))
    traces = []
    for call in range(2):
        got, want = _search(one, n, n), _search(two, n, 7)
        assert np.array_equal(got, want), np.argwhere(got != want)[:3]
        traces.append(got)
        (a_ns, a), (b_ns, b) = one.best(), two.best()
        assert np.array_equal(a_ns, b_ns) and a.tobytes() == b.tobytes()
        # the chains' strategies and timelines afterwards: trials against them, then forced changes
        assert np.array_equal(one.try_mutations(probe, 4).cpu().numpy(), two.try_mutations(probe, 4).cpu().numpy())
        if call == 1:
            assert np.array_equal(one.delta(probe, 4).cpu().numpy(), two.delta(probe, 4).cpu().numpy())
    assert np.array_equal(one.stats()["n_steps"], two.stats()["n_steps"])
    if not kw:
        got = np.concatenate(traces)[:, 0]
        ref = S.metropolis_chain(ops, edges, mach, cost, cfg0[0], tp, tu, table, bucket, 77, 0, 0, min(2 * n, 40), patience=patience)
        assert np.array_equal(got[:len(ref[0])], ref[0])
    one.close()
    two.close()
    sim.close()


def test_a_captured_search_after_one_that_looked_ahead(B):
    import torch
    w = W.workload(1)
    C, n = 3, 12
    cfg0 = w.strategies(C)
    tp, tu = w.search_space()
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    one, two = B.Chains(sim, cfg0), B.Chains(sim, cfg0)
    t0 = int(one.start_ns()[0])
    table, bucket = B.ff_sim_accept_table(20.0 / t0, max(1, t0 // 256), 64), max(1, t0 // 256)
    for ch in (one, two):
        ch.search_setup(tp, tu, table, bucket, seed=4)
    trace = torch.zeros((n, C), dtype=torch.int64, device="cuda")
    assert np.array_equal(one.search(n, d_trace=trace).cpu().numpy().view("<u8"), _search(two, n, 7))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        one.search(n, d_trace=trace)
    for replay in range(3):
        g.replay()
        torch.cuda.synchronize()
        two._sp["step"] = n                       # a replay draws the same steps again
        assert np.array_equal(trace.cpu().numpy().view("<u8"), _search(two, n, 7)), f"replay {replay}"
    one.close()
    two.close()
    sim.close()


@pytest.mark.parametrize("config_id,C", [(0, 256), (1, 200)])
def test_chains_that_walk_different_ways(B, config_id, C):
    """chains side by side that read long paths of their trees, next to chains that are at their next tree already: half of them have settled (long
    runs of rejections), the others start over (every other proposal taken, the best strategy copied at most steps), two are out"""
    w = W.workload(config_id)
    tp, tu = w.search_space()
    cfg0 = w.strategies(C)
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    one, two = B.Chains(sim, cfg0), B.Chains(sim, cfg0)
    t0 = int(one.start_ns()[0])
    bucket = max(1, t0 // 4096)
    table = B.ff_sim_accept_table(500.0 / t0, bucket, 256)
    over = np.zeros((w.n_ops, C), W.MUT_DT)
    fresh = W.strategies(w.ops, C, 91, w.machine.n_devices, w.max_parts, w.choices)
    for ch in (one, two):
        ch.search_setup(tp, tu, table, bucket, 13)
    print(f"search: chains that differ, config {config_id}", flush=True)
    assert np.array_equal(_search(one, 210, 210), _search(two, 210, 7))
    now = one.best()[1]
    for s in range(w.n_ops):
        over[s]["op"] = s
        over[s]["cfg"] = np.where(np.arange(C) % 2 == 0, now[:, s], fresh[:, s])
    over["op"][0, [5, 8]] = w.n_ops                  # these name no op: invalid from here on
    for ch in (one, two):
        ch.delta(ch.upload_mutations(over), w.n_ops)
    for call in range(3):
        got, want = _search(one, 70, 70), _search(two, 70, 7)
        assert np.array_equal(got, want), np.argwhere(got != want)[:3]
        (a_ns, a), (b_ns, b) = one.best(), two.best()
        assert np.array_equal(a_ns, b_ns) and a.tobytes() == b.tobytes()
    one.close()
    two.close()
    sim.close()


def _seconds(f, n=4):
    import time
    import torch
    best = 1e9
    for _ in range(n):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_only_the_nodes_of_a_tree_are_simulated(B):
    """trees of few nodes (two ops of 121 have a list): a round takes no longer where earlier trees of the same chains held strategies that take
    several times as long to simulate.  (Measured: 5.0 against 1.6 ms a call where slots beyond the nodes were simulated too.)"""
    w = W.workload(2)
    C, n_ops = 32, w.n_ops
    light = W.strategies(w.ops, C, 3, w.machine.n_devices, w.max_parts, (1,))
    tp, tu = w.search_space()
    few_p = np.concatenate([np.zeros(n_ops - 2, "<u4"), tp[n_ops - 2:] - tp[n_ops - 2]]).astype("<u4")
    to_light = np.zeros((n_ops, C), W.MUT_DT)
    to_light["op"] = np.arange(n_ops)[:, None]
    to_light["cfg"] = light.T
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    took = []
    for start in (light, w.strategies(C)):
        ch = B.Chains(sim, start)
        t0 = int(np.median(ch.start_ns()))
        bucket = max(1, t0 // 256)
        table = B.ff_sim_accept_table(50.0 / t0, bucket, 256)
        ch.search_setup(tp, tu, table, bucket, 5)
        ch.search(16)
        assert int(ch.delta(ch.upload_mutations(to_light), n_ops).cpu()[-1, 0]) > 0
        ch.search_setup(few_p, tu[tp[n_ops - 2]:], table, bucket, 5)
        took.append(_seconds(lambda: ch.search(16)))
        ch.close()
    sim.close()
    assert took[1] < 1.7 * took[0], took


@pytest.mark.parametrize("form,C", [("alexnet", 2), ("inception", 2)])
def test_snapshots_follow_the_time_a_search_has_reached(B, form, C):
    """a search that more than halves the time leaves a timeline that the next change resumes from"""
    ops, edges, mach, cost, kw, choices = _setup(form, 1)
    parts = cost.shape[1]
    cfg0 = W.strategies(ops, C, 3, mach.n_devices, parts, choices)
    sim = B.Simulator(ops, edges, mach, cost, **kw)
    ch = B.Chains(sim, cfg0)
    start = ch.start_ns().copy()
    t0 = int(np.median(start))
    bucket = max(1, t0 // 4096)
    tp, tu = W.search_space(ops, parts, choices)
    ch.search_setup(tp, tu, B.ff_sim_accept_table(2000.0 / t0, bucket, 256), bucket, 5)
    last = ch.search(1500).cpu().numpy().view("<u8")[-1]
    assert (2 * last < start).all()
    before = ch.stats()
    late = np.zeros((1, C), W.MUT_DT)
    late["op"] = len(ops) - 1
    late["cfg"] = cfg0[:, -1]
    ch.delta(ch.upload_mutations(late), 1)
    assert np.array_equal(ch.stats()["n_resumed"], before["n_resumed"] + 1)
    ch.close()
    sim.close()


@pytest.mark.parametrize("C", [1, 64])
def test_chains_that_have_stopped_are_left_alone(B, C):
    """patience has stopped every chain: their strategies and timelines stay as they are, and a call takes a fraction of one simulation.
    (Measured on the ResNet-101-shaped graph: 0.17 ms; 9.9 where their timelines were recorded again.)"""
    w = W.workload(3)
    cfg0 = w.strategies(C)
    tp, tu = w.search_space()
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    ch = B.Chains(sim, cfg0)
    t0 = int(np.median(ch.start_ns()))
    bucket = max(1, t0 // 256)
    ch.search_setup(tp, tu, B.ff_sim_accept_table(50.0 / t0, bucket, 256), bucket, 5, patience=1)
    ch.search(40)
    last = ch.search(32).cpu().numpy()
    assert np.array_equal(last, np.repeat(last[:1], 32, 0))
    d = sim.upload_strategies(cfg0[:1])
    one_simulation = _seconds(lambda: sim.batch(d, 1))
    assert _seconds(lambda: ch.search(32)) < 0.5 * one_simulation
    # and what they hold is still what they held
    probe = ch.upload_mutations(w.mutations(4, C))
    two = B.Chains(sim, cfg0)
    two.search_setup(tp, tu, B.ff_sim_accept_table(50.0 / t0, bucket, 256), bucket, 5, patience=1)
    assert np.array_equal(_search(two, 40, 7)[-1], last[-1].view("<u8"))
    assert np.array_equal(ch.try_mutations(probe, 4).cpu().numpy(), two.try_mutations(probe, 4).cpu().numpy())
    ch.close()
    two.close()
    sim.close()


def test_proposals_of_late_ops_are_made_in_turn(B):
    """only the last ten ops have a list: their proposals resume late in the timeline, and 32 steps of them take less than one full simulation.
    (Measured on the ResNet-101-shaped graph: 0.4 to 1 ms; 9 to 16 where every call looked ahead.)"""
    w = W.workload(3)
    n_ops = w.n_ops
    tp, tu = w.search_space()
    few_p = np.concatenate([np.zeros(n_ops - 10, "<u4"), tp[n_ops - 10:] - tp[n_ops - 10]]).astype("<u4")
    cfg0 = w.strategies(1)
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    one, two = B.Chains(sim, cfg0), B.Chains(sim, cfg0)
    t0 = int(one.start_ns()[0])
    bucket = max(1, t0 // 256)
    for ch in (one, two):
        ch.search_setup(few_p, tu[tp[n_ops - 10]:], B.ff_sim_accept_table(50.0 / t0, bucket, 256), bucket, 5)
    assert np.array_equal(_search(one, 320, 32), _search(two, 320, 7))
    (a_ns, a), (b_ns, b) = one.best(), two.best()
    assert np.array_equal(a_ns, b_ns) and a.tobytes() == b.tobytes()
    d = sim.upload_strategies(cfg0)
    assert _seconds(lambda: one.search(32)) < 0.5 * _seconds(lambda: sim.batch(d, 1))
    one.close()
    two.close()
    sim.close()


@pytest.mark.parametrize("config_id,C,n,most", [(2, 300, 12, 0), (4, 150, 15, 0), (4, 150, 16, 1 << 30)])
def test_memory_of_searches_that_look_ahead(B, config_id, C, n, most):
    """none for calls of too few steps to look ahead with that many chains; 1 GiB at most for the others"""
    import torch
    w = W.workload(config_id)
    sim = B.Simulator(w.ops, w.edges, w.machine, w.cost)
    ch = B.Chains(sim, w.strategies(C))
    t0 = int(np.median(ch.start_ns()))
    bucket = max(1, t0 // 256)
    tp, tu = w.search_space()
    ch.search_setup(tp, tu, B.ff_sim_accept_table(50.0 / t0, bucket, 256), bucket, 5)
    trace = torch.empty((n, C), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ch.search(n, d_trace=trace)
    torch.cuda.synchronize()
    got = before - torch.cuda.mem_get_info()[0]
    assert got <= most and (most == 0 or got > most // 2), got
    ch.close()
    sim.close()

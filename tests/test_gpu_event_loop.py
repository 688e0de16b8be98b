"""The event loop on kept set-up at the sizes where it changes form: rows of 16 and 64 lanes, queues of up to 16, up
to 64 and more ops, more ops with events than the queue has slots, events and link bookings too far ahead for 32-bit
times, and the constants of the link-time division.  Everything against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1807_05358_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_05358_amd import binding
    return binding


def draw(rng, ops, n, D, parts, choices, strides=False):
    cfgs = np.zeros((n, len(ops)), W.CFG_DT)
    for i in range(len(ops)):
        t = W.valid_degree_tuples(ops[i], parts, choices)
        cfgs["deg"][:, i] = t[rng.integers(len(t), size=n)]
    cfgs["dev_offset"] = rng.integers(0, D, size=cfgs.shape)
    cfgs["dev_stride"] = 1
    if strides:
        cfgs["dev_stride"][n // 2:] = rng.integers(0, 5, size=cfgs[n // 2:].shape)
    return cfgs


def check(B, ops, edges, mach, cost, cfgs, kernel=None, chain_steps=0, **refined):
    """refined: params and ties, as the simulator and the oracle take them"""
    want = oracle.simulate_batch(ops, edges, mach, cost, cfgs, n_threads=8, **refined)
    sim = B.Simulator(ops, edges, mach, cost, **refined)
    if kernel is not None:
        assert B.ff_sim_batch_kernel_name(sim.handle, len(cfgs)).startswith(kernel), B.ff_sim_batch_kernel_name(sim.handle, len(cfgs))
    got = sim.simulate(cfgs)
    assert np.array_equal(got, want), (np.nonzero(got != want)[0][:5], got[got != want][:3], want[got != want][:3])
    again, st = sim.simulate(cfgs, stats=True)
    assert np.array_equal(again, want) and not st["exit_code"].any()
    if chain_steps:
        # a chain of changes from the first strategy to parts of the second, op by op
        muts = np.zeros((chain_steps, 1), W.MUT_DT)
        muts["op"][:, 0] = np.arange(chain_steps) * 7 % len(ops)
        muts["cfg"][:, 0] = cfgs[1, muts["op"][:, 0]]
        ch = B.Chains(sim, cfgs[:1])
        d = ch.delta(ch.upload_mutations(muts), chain_steps).cpu().numpy().view("<u8")
        ref = oracle.simulate_delta_chain(ops, edges, mach, cost, cfgs[0], muts[:, 0], **refined)
        assert np.array_equal(d[:, 0], ref)
        t = ch.try_mutations(ch.upload_mutations(muts[::-1].copy()), chain_steps).cpu().numpy().view("<u8")
        cur = cfgs[0].copy()
        for s in range(chain_steps):
            cur[int(muts[s, 0]["op"])] = muts[s, 0]["cfg"]
        cand = np.repeat(cur[None], chain_steps, 0)
        for s in range(chain_steps):
            cand[s, int(muts[chain_steps - 1 - s, 0]["op"])] = muts[chain_steps - 1 - s, 0]["cfg"]
        assert np.array_equal(t[:, 0], oracle.simulate_batch(ops, edges, mach, cost, cand, n_threads=8, **refined))
        ch.close()
    sim.close()
    return want


@pytest.mark.parametrize("n_ops", [1, 15, 16, 17, 64, 65, 66])
@pytest.mark.parametrize("parts", [1, 15, 16, 17, 64])
def test_queue_and_row_shapes(B, n_ops, parts):
    """every combination of queue shape and lanes per row, at the edges of both, tensors of one to four dims"""
    rng = np.random.default_rng(100 * n_ops + parts)
    g = W.GraphBuilder()
    shapes = [(48,), (24, 16), (16, 5, 9), (12, 8, 7, 6)]
    for i in range(n_ops):
        nd = int(rng.integers(1, 5))
        o = g.op(W.T_ELEM, shapes[nd - 1], tuple(range(nd)), 1)
        for s in sorted(set(int(x) for x in rng.integers(0, o, size=min(o, 2)))) if o else ():
            sd = g.ops[s][0]
            g.edge(s, o, [W.ident(d) if d < nd and rng.random() < 0.7 else W.ALL for d in range(sd)])
    ops, edges, _ = g.finish()
    mach = W.Machine(5, 4, 7, 3, 2, 31)
    cost = rng.integers(1, 5000, size=(n_ops, parts)).astype("<u4")
    cfgs = draw(rng, ops, 24, mach.n_devices, parts, (1, 2, 3, 4, 5, 8, 12, 16, 48), strides=True)
    check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=min(n_ops, 6))


@pytest.mark.parametrize("parts", [4, 32])
@pytest.mark.parametrize("equal", [False, True])
def test_more_ops_with_events_than_slots(B, parts, equal):
    """300 ops without inputs are READY at time 0 (and feed 30 others): the queue's 64 slots overflow.  equal: all
    tasks take the same time, so that long stretches of events tie."""
    rng = np.random.default_rng(7)
    g = W.GraphBuilder()
    src = [g.op(W.T_ELEM, (32, 16), (0, 1), 1) for _ in range(300)]
    for k in range(30):
        o = g.op(W.T_ELEM, (32, 16), (0, 1), 1)
        for s in src[k * 10:k * 10 + 10]:
            g.edge(s, o, [W.ident(0), W.ident(1)])
    ops, edges, _ = g.finish()
    mach = W.Machine(4, 4, 3, 2)
    cost = (np.full((len(ops), parts), 1000) if equal else rng.integers(1, 90000, size=(len(ops), parts))).astype("<u4")
    cfgs = draw(rng, ops, 12, 16, parts, (1, 2, 3, 4, 8, 16), strides=True)
    check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=4)


@pytest.mark.parametrize("n_ops", [12, 80])
def test_tasks_longer_than_32_bits_of_time(B, n_ops):
    """tasks of up to 2^32 - 1 ns, next to short ones: events beyond the reach of 32-bit keys, an epoch that moves often"""
    rng = np.random.default_rng(n_ops)
    g = W.GraphBuilder()
    for i in range(n_ops):
        o = g.op(W.T_ELEM, (64, 8), (0, 1), 1)
        for s in sorted(set(int(x) for x in rng.integers(max(0, o - 5), o, size=2))) if o else ():
            g.edge(s, o, [W.ident(0), W.ident(1)])
    ops, edges, _ = g.finish()
    mach = W.Machine(4, 4)
    cost = rng.choice([5, 70000, 2 ** 31 - 1, 2 ** 31, 2 ** 32 - 1, 3 * 10 ** 9], size=(n_ops, 16)).astype("<u4")
    want = check(B, ops, edges, mach, cost, draw(rng, ops, 64, 16, 16, (1, 2, 4, 8, 16), strides=True), kernel="k_loop_batch", chain_steps=5)
    assert want.max() > 2 ** 33


def test_links_booked_beyond_32_bits_of_time(B):
    """one tensor of 1 GiB read whole by 64 parts of several ops: its transfers queue for more than 2^32 ns on the same
    links, and the candidate is simulated with 64-bit link rows"""
    g = W.GraphBuilder()
    a = g.op(W.T_ELEM, (16384, 16384), (0, 1), 1)
    for _ in range(70):
        b = g.op(W.T_ELEM, (64, 64), (0, 1), 1)
        if b <= 8:
            g.edge(a, b, [W.ALL, W.ALL])
    ops, edges, _ = g.finish()
    mach = W.Machine(16, 4, 6, 5)
    cost = np.full((len(ops), 64), 1000, "<u4")
    rng = np.random.default_rng(3)
    cfgs = draw(rng, ops, 16, 64, 64, (1, 2, 4, 8, 16, 32, 64))
    cfgs["deg"][:8, 1:9] = (8, 8, 1, 1)
    cfgs["deg"][:8, 0] = (1, 1, 1, 1)
    cfgs["deg"][12:, 1:] = (1, 1, 1, 1)
    want = check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=4)
    assert want.max() > 5 * 10 ** 9


@pytest.mark.parametrize("elem_bytes", [1, 2, 3, 4, 8, 12])
def test_link_time_constants(B, elem_bytes):
    """ceil(elements * element size / bandwidth) for bandwidths that divide, share a factor with, or have none in common
    with the element size, from 1 B/ns to the largest, with transfers of one element up to 2^27"""
    rng = np.random.default_rng(elem_bytes)
    g = W.GraphBuilder()
    a = g.op(W.T_ELEM, (4096, 32768), (0, 1), 1)
    for k in range(3):
        b = g.op(W.T_ELEM, (4096, 32768), (0, 1), 1)
        g.edge(a, b, [W.ident(0), W.ident(1)])
        c = g.op(W.T_ELEM, (61, 7), (0, 1), 1)
        g.edge(b, c, [(0, 1, 3 * k, 5 * k), (1, 2, 0, k)])
    ops, edges, _ = g.finish()
    cost = rng.integers(1, 100, size=(len(ops), 64)).astype("<u4")
    for near, far in [(1, 1), (2, 3), (20, 12), (5, 7), (24, 36), (255, 256), (65537, 1000003), (2 ** 31, 2 ** 32 - 1), (1, 2 ** 32 - 1)]:
        mach = W.Machine(4, 4, near, far, 1, 2, elem_bytes)
        check(B, ops, edges, mach, cost, draw(rng, ops, 24, 16, 64, (1, 2, 3, 5, 7, 16, 61)))


@pytest.mark.parametrize("n_ops", [12, 70])
@pytest.mark.parametrize("parts", [16, 64])
def test_chain_that_starts_from_an_invalid_strategy(B, n_ops, parts):
    """two ops with degrees their tensors do not have, mended one after the other, by changes and by a trial: the kept set-up of
    every edge is complete as soon as the strategy is valid"""
    rng = np.random.default_rng(n_ops + parts)
    g = W.GraphBuilder()
    for i in range(n_ops):
        o = g.op(W.T_ELEM, (16, 6, 8) if i % 3 else (64, 8), (0, 1, 2) if i % 3 else (0, 1), 1)
        for s in sorted(set(int(x) for x in rng.integers(max(0, o - 4), o, size=2))) if o else ():
            g.edge(s, o, [W.ident(0), W.ident(1)] + ([W.ALL] if s % 3 else []))
    ops, edges, _ = g.finish()
    mach = W.Machine(4, 4)
    cost = rng.integers(1, 9000, size=(n_ops, parts)).astype("<u4")
    cfgs = draw(rng, ops, 3, 16, parts, (1, 2, 3, 4, 8), strides=True)
    good = cfgs[0].copy()
    a, b = 3, n_ops - 2
    cfgs[0]["deg"][a] = (255, 1, 1, 1)
    cfgs[0]["deg"][b] = (0, 2, 1, 1)
    # a step that leaves it invalid, one that mends the first op, the second, and an ordinary one
    muts = np.zeros((4, 1), W.MUT_DT)
    muts["op"][:, 0] = (5, a, b, 1)
    for t, cfg in enumerate((cfgs[1, 5], good[a], cfgs[1, b], cfgs[1, 1])):
        muts[t, 0]["cfg"] = cfg
    sim = B.Simulator(ops, edges, mach, cost)
    ch = B.Chains(sim, cfgs[:1])
    invalid = np.iinfo(np.uint64).max
    assert ch.start_ns()[0] == invalid
    d = ch.delta(ch.upload_mutations(muts[:2].copy()), 2).cpu().numpy().view("<u8")
    assert (d == invalid).all()
    # a trial that mends the last op, against the chain's (invalid) strategy
    cur = cfgs[0].copy()
    cur[5], cur[a] = cfgs[1, 5], good[a]
    trial = np.zeros((2, 1), W.MUT_DT)
    trial["op"][:, 0] = (b, 2)
    trial[0, 0]["cfg"], trial[1, 0]["cfg"] = good[b], cfgs[1, 2]
    t = ch.try_mutations(ch.upload_mutations(trial), 2).cpu().numpy().view("<u8")
    mended = cur.copy()
    mended[b] = good[b]
    assert t[0, 0] == oracle.simulate_batch(ops, edges, mach, cost, mended[None])[0] and t[1, 0] == invalid
    d = ch.delta(ch.upload_mutations(muts[2:].copy()), 2).cpu().numpy().view("<u8")
    steps = np.repeat(cur[None], 2, 0)
    steps[:, b] = cfgs[1, b]
    steps[1, 1] = cfgs[1, 1]
    assert np.array_equal(d[:, 0], oracle.simulate_batch(ops, edges, mach, cost, steps))
    ch.close()
    sim.close()


@pytest.mark.parametrize("shape", [(16384, 16384), (131072, 2048)])
def test_general_strategies_queue_for_longer_than_32_bits_on_one_link(B, shape):
    """64 parts on one device read a tensor of 1 GiB whole, one after the other over one link: fewer than 2^32 ns for as many
    of them as a node has GPUs, more for all; extents within and beyond 16 bits"""
    g = W.GraphBuilder()
    a = g.op(W.T_ELEM, shape, (0, 1), 1)
    for _ in range(6):
        b = g.op(W.T_ELEM, (64, 64), (0, 1), 1)
        g.edge(a, b, [W.ALL, W.ALL])
    ops, edges, _ = g.finish()
    mach = W.Machine(16, 4, 6, 5)
    cost = np.full((len(ops), 64), 1000, "<u4")
    rng = np.random.default_rng(8)
    cfgs = draw(rng, ops, 6, 64, 64, (1, 2, 4, 8), strides=True)
    cfgs["deg"][:, 0] = (1, 1, 1, 1)
    cfgs["deg"][:4, 1:] = (8, 8, 1, 1)
    cfgs["dev_stride"][:2] = 0
    want = check(B, ops, edges, mach, cost, cfgs, chain_steps=3)
    assert want.max() > 10 * 2 ** 30


def far_fan_out(n_consumers):
    """One tensor of 1 GB in two parts of unequal size, read by consumers in two parts each over the two links between four
    nodes of one GPU: the larger part is sent first and arrives up to 4 s later, the smaller one is sent 10 us later and
    arrives earlier, so that an op with an event gets an earlier one, both too far ahead for a 32-bit key.  Behind the
    last consumer a task of 3 s, beside all of it a chain of tasks that keeps simulated time moving in between."""
    g = W.GraphBuilder()
    cost, cfg = [], []

    def op(extent, deg, dev, ns):
        o = g.op(W.T_ELEM, extent, tuple(range(len(extent))), 1)
        cost.append(ns)
        cfg.append((tuple(deg) + (1,) * (4 - len(deg)), dev))
        return o
    same = [W.ident(0), W.ident(1), W.ident(2)]
    op((1,), (1,), 0, 10000)
    big = op((5, 5000, 10000), (2,), 0, 1000)
    readers = [op((5, 5000, 10000), (2,), 2, 1000) for _ in range(n_consumers)]
    for r in readers:
        g.edge(big, r, same)
    g.edge(readers[-1], op((1, 1, 10000), (1,), 0, 3 * 10 ** 9), same)
    last = None
    for _ in range(60):
        o = op((1,), (1,), 2, 90 * 10 ** 6)
        if last is not None:
            g.edge(last, o, [W.ident(0)])
        last = o
    ops, edges, _ = g.finish()
    cfgs = np.zeros((1, len(ops)), W.CFG_DT)
    cfgs["deg"][0], cfgs["dev_offset"][0] = [c[0] for c in cfg], [c[1] for c in cfg]
    cfgs["dev_stride"] = 1
    return ops, edges, W.Machine(4, 1, 12, 12), np.repeat(np.array(cost, "<u4")[:, None], 4, 1), cfgs


@pytest.mark.parametrize("strides", [1, 5])
@pytest.mark.parametrize("n_consumers", [60, 66, 72, 84])
def test_earlier_far_event_of_an_op_without_a_slot(B, n_consumers, strides):
    """as a batch, as a chain and as trials; strides 5 = 1 modulo the number of devices, the same strategy in the general form"""
    ops, edges, mach, cost, cfgs = far_fan_out(n_consumers)
    cfgs["dev_stride"] = strides
    # the second strategy has the 3 s task elsewhere: what a chain's steps and the trials change
    cfgs = np.repeat(cfgs, 3, 0)
    cfgs["dev_offset"][1, n_consumers + 2] = 1
    cfgs["dev_offset"][1, 7], cfgs["dev_offset"][2, 0] = 1, 1
    check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=8)
    # the op ahead of the smaller part goes and comes back: every simulation starts from time 0 or from a snapshot before it matters
    muts = np.zeros((4, 1), W.MUT_DT)
    muts["op"][:, 0] = (0, n_consumers + 2, 0, n_consumers + 2)
    muts["cfg"][:, 0] = cfgs[(2, 1, 0, 0), muts["op"][:, 0]]
    sim = B.Simulator(ops, edges, mach, cost)
    ch = B.Chains(sim, cfgs[:1])
    t = ch.try_mutations(ch.upload_mutations(muts), 4).cpu().numpy().view("<u8")
    cand = np.repeat(cfgs[:1], 4, 0)
    cand[np.arange(4), muts["op"][:, 0]] = muts["cfg"][:, 0]
    assert np.array_equal(t[:, 0], oracle.simulate_batch(ops, edges, mach, cost, cand))
    d = ch.delta(ch.upload_mutations(muts), 4).cpu().numpy().view("<u8")
    assert np.array_equal(d[:, 0], oracle.simulate_delta_chain(ops, edges, mach, cost, cfgs[0], muts[:, 0]))
    ch.close()
    sim.close()


@pytest.mark.parametrize("n_ops", [12, 80])
@pytest.mark.parametrize("mach", [W.Machine(2, 2, 1, 1, 700, 900), W.Machine(4, 1, 1, 1, 0, 3 * 10 ** 9), W.Machine(1, 4, 1, 1, 10 ** 9, 0),
                                  W.Machine(2, 2, 9, 9, 0, 0, 4, np.array([[1, 1], [2, 1]], "<u4"), np.array([[0, 5], [800, 0]], "<u4"),
                                            np.array([[1, 1], [1, 1]], "<u4"), np.array([[0, 7], [2 ** 30, 0]], "<u4"))])
def test_parameter_transfers_longer_than_32_bits_of_time(B, n_ops, mach):
    """parameters of up to 2^32 - 1 bytes over links of 1 byte per ns, and latencies of seconds: the time of one transfer, not
    only when it ends, takes more than 32 bits"""
    rng = np.random.default_rng(n_ops)
    g = W.GraphBuilder()
    for i in range(n_ops):
        o = g.op(W.T_ELEM, (8, 6), (0, 1), 1)
        for s in sorted(set(int(x) for x in rng.integers(max(0, o - 4), o, size=2))) if o else ():
            g.edge(s, o, [W.ident(0), W.ident(1)])
    ops, edges, _ = g.finish()
    cost = rng.integers(1, 9000, size=(n_ops, 16)).astype("<u4")
    params = (rng.choice([0, 0, 1000, 3 * 10 ** 9, 2 ** 32 - 2, 2 ** 32 - 1], size=n_ops).astype("<u4"), rng.integers(0, 4, size=n_ops).astype(np.uint8))
    params[0][1], params[1][1] = 2 ** 32 - 1, 0
    cfgs = draw(rng, ops, 16, mach.n_devices, 16, (1, 2, 4), strides=True)
    cfgs["deg"][:4, 1] = (2, 1, 1, 1)
    want = check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=6, params=params)
    assert want.max() > 2 ** 32


def test_refused_workspace_leaves_the_results_alone(B):
    """rows of 16 lanes fit LDS and need no workspace, the 64-bit kernel behind them (transfers of seconds) does: without one
    the call is refused and nothing has been launched"""
    rng = np.random.default_rng(5)
    g = W.GraphBuilder()
    for i in range(64):
        o = g.op(W.T_ELEM, (16384, 16384) if i == 0 else (64, 64), (0, 1), 1)
        if 0 < o < 31:
            g.edge(0 if o < 4 else o - 3, o, [W.ALL, W.ALL])
    ops, edges, _ = g.finish()
    mach = W.Machine(8, 9, 6, 5)
    cost = rng.integers(1, 9000, size=(len(ops), 16)).astype("<u4")
    cfgs = draw(rng, ops, 8, 72, 16, (1, 2, 4, 8, 16))
    cfgs["deg"][:, 0] = 1
    cfgs["deg"][:4, 1:4] = (4, 4, 1, 1)
    sim = B.Simulator(ops, edges, mach, cost)
    assert B.ff_sim_batch_kernel_name(sim.handle, len(cfgs)).startswith("k_loop_batch<false, true")
    need = B.ff_sim_workspace_bytes(sim.handle, len(cfgs))
    assert need > 0
    d = sim.upload_strategies(cfgs)
    out = torch.full((len(cfgs),), 12345, dtype=torch.int64, device="cuda")
    B.ff_sim_set_stats(sim.handle, None)
    with pytest.raises(B.FFSimError):
        B.ff_sim_batch(sim.handle, d.data_ptr(), len(cfgs), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert (out == 12345).all()
    want = oracle.simulate_batch(ops, edges, mach, cost, cfgs, n_threads=8)
    assert want.max() > 2 ** 32 and np.array_equal(sim.simulate(cfgs), want)
    sim.close()


@pytest.mark.parametrize("gib", [0.01, 1.99, 3.99])
@pytest.mark.parametrize("elem_bytes", [1, 2, 3, 4, 5, 6, 12, 20])
def test_link_time_constants_for_any_element_size(B, elem_bytes, gib):
    """element sizes with and without common divisors with the bandwidths, largest tensors well below 2 GiB, at 2 GiB and at 4 GiB:
    up to 2 GiB the event loop on kept set-up serves all of them (at less than 2^30 bytes per ns)"""
    rng = np.random.default_rng(elem_bytes)
    rows = int(gib * 2 ** 30 / elem_bytes / 16384)
    g = W.GraphBuilder()
    a = g.op(W.T_ELEM, (rows // 64 + 1, 64, 16384), (0, 1, 2), 1)
    for k in range(3):
        b = g.op(W.T_ELEM, (rows // 64 + 1, 64, 16384 - 1000 * k), (0, 1, 2), 1)
        g.edge(a, b, [W.ident(0), W.ident(1), W.ident(2)])
        c = g.op(W.T_ELEM, (61, 7), (0, 1), 1)
        g.edge(b, c, [(0, 1, k, 5 * k), (1, 2, 0, k), (1, 1 + 100 * k, 0, 17 * k)])
    ops, edges, _ = g.finish()
    cost = rng.integers(1, 100, size=(len(ops), 64)).astype("<u4")
    for near, far in [(20, 14), (25, 7), (101, 97), (127, 255), (12345, 65537), (2 ** 31 - 1, 2 ** 32 - 1), (1000003, 64)]:
        mach = W.Machine(4, 4, near, far, 1, 2, elem_bytes)
        check(B, ops, edges, mach, cost, draw(rng, ops, 16, 16, 64, (1, 2, 3, 5, 7, 16, 61)), kernel="k_loop_batch" if gib < 2 and far < 2 ** 30 else None)


@pytest.mark.parametrize("refinement", ["params", "links", "node_links", "ties", "devmaps"])
@pytest.mark.parametrize("n_ops", [10, 70])
def test_bookings_beyond_32_bits_with_refined_inputs(B, n_ops, refinement):
    """what is simulated again with 64-bit link rows: parameter traffic, links that differ per pair, tied configurations with
    contributing edges, explicit devices; batches, and chains and trials where they take such inputs"""
    rng = np.random.default_rng(n_ops)
    g = W.GraphBuilder()
    a = g.op(W.T_ELEM, (16384, 16384), (0, 1), 1)
    for _ in range(n_ops - 1):
        b = g.op(W.T_ELEM, (64, 64), (0, 1), 1)
        if b <= 6:
            g.edge(a, b, [W.ALL, W.ALL])
        elif rng.random() < 0.5:
            g.edge(b - 6, b, [W.ident(0), W.ident(1)])
    ops, edges, flops = g.finish()
    mach, refined = W.Machine(4, 4, 6, 5), {}
    if refinement == "links":
        mach = W.Machine(4, 4, 6, 5, 0, 0, 4, *W.paired_links(4, 9, 4, 0, 300))
    elif refinement == "node_links":
        mach = W.Machine(4, 4, 6, 5, 0, 0, 4, None, None, *W.ring_node_links(4, 7, 4, 1000))
    elif refinement == "params":
        refined["params"] = (rng.choice([0, 5000, 10 ** 9, 2 ** 32 - 1], size=len(ops)).astype("<u4"), rng.integers(0, 4, size=len(ops)).astype(np.uint8))
    elif refinement == "ties":
        ops, edges, flops, refined["ties"], _ = W.training_graph(ops, edges, flops)
        refined["params"] = (rng.choice([0, 5000, 10 ** 9], size=len(ops)).astype("<u4"), np.ones(len(ops), np.uint8))
    cost = rng.integers(1, 9000, size=(len(ops), 16)).astype("<u4")
    cfgs = draw(rng, ops, 12, 16, 16, (1, 2, 4, 8, 16), strides=True)
    cfgs["deg"][:, 0] = 1
    cfgs["deg"][:9, 1:7] = (4, 4, 1, 1)
    want = check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=6, **refined)
    if refinement == "devmaps":
        maps = W.device_maps(cfgs, 16, 3)
        want = oracle.simulate_batch(ops, edges, mach, cost, cfgs, n_threads=8, devmaps=maps)
        sim = B.Simulator(ops, edges, mach, cost)
        assert np.array_equal(sim.simulate(cfgs, devmaps=maps), want)
        sim.close()
    assert want.max() > 2 ** 32

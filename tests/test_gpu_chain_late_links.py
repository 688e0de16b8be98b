"""Chains of changes on machines whose transfers take seconds: link rows booked beyond 32 bits while the changed timeline re-joins the
accepted one.  What a chain keeps of such a simulation is what the next changes start from.  Everything against the oracle."""
import numpy as np
import pytest

import oracle
from oracle import search as osearch
from paper_1807_05358_amd import workloads as W

pytestmark = pytest.mark.gpu

MS = 10 ** 6
MACHINE = W.Machine(4, 1, 12, 12, 0, 3000 * MS)      # one GPU per node, 3 s from node to node


@pytest.fixture(scope="module")
def B():
    from paper_1807_05358_amd import binding
    return binding


def displaced_task():
    """Op `late` reads `source` behind another reader over the same link: its transfer ends at 7 s, more than 2^32 ns after it is booked.  Taken for
    ready about 5.3 s it would run on device 1 ahead of `pushed`, ready at 6 s, whose end would go from 7 to 8.8 s.  `reader` reads `pushed` and is the
    last to end.  `elsewhere` starts at 0.5 s and is read at 1.5 s: a timeline in which nothing but that op is simulated again is the old one from
    then on, behind the booking and ahead of what depends on it.  Few steps in all."""
    g = W.GraphBuilder()
    at = {}
    cost, dev = [], []
    for name, d, ms, reads in [("first", 3, 500, ()), ("elsewhere", 3, 1000, ("first",)), ("after", 3, 100, ("elsewhere",)), ("source", 0, 1000, ()), ("ahead", 1, 100, ("source",)),
                               ("late", 1, 3500, ("source",)), ("long", 2, 3000, ()), ("pushed", 1, 1000, ("long",)), ("reader", 1, 4000, ("pushed",))]:
        at[name] = g.op(W.T_ELEM, (1,), (0,), 1)
        cost.append(ms * MS)
        dev.append(d)
        for r in reads:
            g.edge(at[r], at[name], [W.ident(0)])
    ops, edges, _ = g.finish()
    cfgs = np.zeros((1, len(ops)), W.CFG_DT)
    cfgs["deg"], cfgs["dev_offset"][0], cfgs["dev_stride"] = 1, dev, 1
    return ops, edges, np.repeat(np.array(cost, "<u4")[:, None], 4, 1), cfgs, at


def test_a_change_behind_a_task_that_a_late_transfer_does_not_displace(B):
    ops, edges, cost, cfgs, at = displaced_task()
    muts = np.zeros((3, 1), W.MUT_DT)
    muts["op"][:, 0] = at["elsewhere"], at["reader"], at["reader"]
    muts["cfg"][:, 0] = cfgs[0, muts["op"][:, 0]]          # the first change changes nothing
    muts["cfg"]["dev_offset"][1, 0] = 3
    want = oracle.simulate_delta_chain(ops, edges, MACHINE, cost, cfgs[0], muts[:, 0])
    assert want.tolist() == [14500 * MS + 1, 14000 * MS + 2, 14500 * MS + 1]
    sim = B.Simulator(ops, edges, MACHINE, cost)
    assert B.ff_sim_batch_kernel_name(sim.handle, 1).startswith("k_loop_batch")
    ch = B.Chains(sim, cfgs)
    # one change a call: the steps of one call may be cut into segments that start from time 0
    got = [int(ch.delta(ch.upload_mutations(muts[s:s + 1].copy()), 1).cpu().numpy().view("<u8")[0, 0]) for s in range(3)]
    assert int(ch.stats()["n_converged"][0]) > 0, "the first change is to re-join the accepted timeline"
    assert got == want.tolist()
    ch.close()
    sim.close()


@pytest.mark.parametrize("ahead", [0, 8])
def test_search_behind_a_task_that_a_late_transfer_does_not_displace(B, ahead):
    """the same as proposals, all of them taken: `elsewhere` and `reader` on any device"""
    ops, edges, cost, cfgs, at = displaced_task()
    C, n = 16, 24
    ptr = np.zeros(len(ops) + 1, "<u4")
    for o in (at["elsewhere"], at["reader"]):
        ptr[o + 1:] += 1
    tuples = np.full(int(ptr[-1]), 0x01010101, "<u4")
    accept = np.full(4, 2 ** 32 - 1, "<u4")
    sim = B.Simulator(ops, edges, MACHINE, cost)
    ch = B.Chains(sim, np.repeat(cfgs, C, 0))
    ch.search_setup(ptr, tuples, accept, 10 ** 9, 77)
    got = ch.search(n, ahead=ahead).cpu().numpy().view("<u8")
    for c in range(C):
        want = osearch.metropolis_chain(ops, edges, MACHINE, cost, cfgs[0], ptr, tuples, accept, 10 ** 9, 77, c, 0, n)[0]
        assert np.array_equal(got[:, c], want), c
    ch.close()
    sim.close()


@pytest.mark.parametrize("lat_ms", [1500, 3000])
@pytest.mark.parametrize("n_ops", [10, 40, 80])
def test_chains_with_transfers_of_seconds(B, n_ops, lat_ms):
    """one change a call, many of them back to where the chain was, so that timelines re-join each other"""
    rng = np.random.default_rng([n_ops, lat_ms])
    g = W.GraphBuilder()
    for i in range(n_ops):
        o = g.op(W.T_ELEM, (4,), (0,), 1)
        for s in sorted(set(int(x) for x in rng.integers(max(0, o - 6), o, size=2))) if o and rng.random() < 0.8 else ():
            g.edge(s, o, [W.ident(0)])
    ops, edges, _ = g.finish()
    mach = W.Machine(6, 1, 12, 12, 0, lat_ms * MS)
    cost = rng.integers(100 * MS, 4000 * MS, size=(n_ops, 4)).astype("<u4")
    C, n = 8, 24
    cfgs = np.zeros((C, n_ops), W.CFG_DT)
    cfgs["deg"], cfgs["dev_stride"] = 1, 1
    cfgs["deg"][..., 0] = rng.choice([1, 1, 2], size=(C, n_ops))
    cfgs["dev_offset"] = rng.integers(0, 6, size=(C, n_ops))
    muts = np.zeros((n, C), W.MUT_DT)
    muts["op"] = rng.integers(0, n_ops, size=(n, C))
    muts["cfg"] = cfgs[np.arange(C), muts["op"]]
    moved = rng.random((n, C)) < 0.5
    muts["cfg"]["dev_offset"][moved] = rng.integers(0, 6, size=int(moved.sum()))
    sim = B.Simulator(ops, edges, mach, cost)
    ch = B.Chains(sim, cfgs)
    want = np.stack([oracle.simulate_delta_chain(ops, edges, mach, cost, cfgs[c], muts[:, c]) for c in range(C)], 1)
    assert want.max() > 2 ** 33
    for s in range(n):
        got = ch.delta(ch.upload_mutations(muts[s:s + 1].copy()), 1).cpu().numpy().view("<u8")[0]
        assert np.array_equal(got, want[s]), (s, np.nonzero(got != want[s])[0])
    assert int(ch.stats()["n_converged"].max()) > 0
    ch.close()
    sim.close()

"""More ops with events than the queue has slots, where ops have several out-edges or parameters: ops that leave their slots and come back with
the first task to dequeue and the first one to release, found again from their words.  Everything against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1807_05358_amd import workloads as W
from test_gpu_event_loop import B, check, draw  # noqa: F401 (B is a fixture)

pytestmark = pytest.mark.gpu


def most_at_once(ops, edges, mach, cost, cfg, **refined):
    """the largest number of ops that have a task READY or running at one time"""
    tg = oracle.build_task_graph(ops, edges, mach, cost, cfg, **refined)
    _, ready, _, end = tg.simulate()
    op_of = np.repeat(np.arange(len(ops)), cfg["deg"].astype(np.int64).prod(axis=1))
    first, last = np.full(len(ops), 2 ** 63 - 1, np.int64), np.zeros(len(ops), np.int64)
    np.minimum.at(first, op_of, ready[:len(op_of)].astype(np.int64))
    np.maximum.at(last, op_of, end[:len(op_of)].astype(np.int64))
    return max(int(((first <= t) & (t < last)).sum()) for t in np.unique(first))


# fan: out-edges of the ops that overflow the queue, up to and beyond the edges with which an op still releases at several times
@pytest.mark.parametrize("fan", [2, 9])
@pytest.mark.parametrize("parts", [4, 16, 48])
@pytest.mark.parametrize("params", [False, True])
@pytest.mark.parametrize("equal", [False, True])
def test_ops_with_several_edges_that_leave_their_slots(B, fan, parts, params, equal):  # noqa: F811
    rng = np.random.default_rng([fan, parts, params, equal])
    g = W.GraphBuilder()
    n_src, n_dst = 200, 36
    for _ in range(n_src + n_dst):
        g.op(W.T_ELEM, (48, 16), (0, 1), 1)
    for i in range(n_src):
        for j in sorted(rng.choice(n_dst, size=fan, replace=False)):
            g.edge(i, n_src + int(j), [W.ident(0), W.ALL if (i + j) % 5 == 0 else W.ident(1)])
    for j in range(1, n_dst):
        g.edge(n_src + j - 1, n_src + j, [W.ident(0), W.ident(1)])
    ops, edges, _ = g.finish()
    nodes, gpus = (16, 4) if parts == 48 else (4, 4)
    mach = W.Machine(nodes, gpus, 3, 2)
    cost = (np.full((len(ops), parts), 700) if equal else rng.integers(1, 10 ** rng.integers(1, 5, size=(len(ops), 1)) + 1, size=(len(ops), parts))).astype("<u4")
    cfgs = draw(rng, ops, 12, nodes * gpus, parts, (1, 2, 3, 4, 8, 16, 48), strides=True)
    refined = {"params": (rng.integers(0, 3, size=len(ops)).astype("<u4") * 5000, rng.integers(0, 4, size=len(ops)).astype(np.uint8))} if params else {}
    assert most_at_once(ops, edges, mach, cost, cfgs[0], **refined) > 128
    check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=4, **refined)

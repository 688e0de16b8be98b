"""The event loop's two queues: releases that go ahead of earlier dequeues, runs of events of one kind, releases of ops with several edges or
parameters at several times, parts of an op that meet on a device or a node.  Everything against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_1807_05358_amd import workloads as W
from test_gpu_event_loop import B, check, draw  # noqa: F401 (B is a fixture)

pytestmark = pytest.mark.gpu


# fan: out-edges per op (runs of releases: up to 8 edges); n_ops: both queue shapes, and more ops with events than slots (fan 1)
@pytest.mark.parametrize("fan", [1, 2, 8, 9])
@pytest.mark.parametrize("nodes,gpus,parts", [(4, 4, 16), (5, 3, 48), (16, 4, 64), (2, 8, 16), (1, 4, 8)])
@pytest.mark.parametrize("n_ops,params", [(14, False), (14, True), (90, False), (90, True)])
def test_order_of_releases_and_dequeues(B, fan, nodes, gpus, parts, n_ops, params):  # noqa: F811
    rng = np.random.default_rng([fan, nodes, gpus, n_ops, params])
    g = W.GraphBuilder()
    for i in range(n_ops):
        g.op(W.T_ELEM, (64, 48), (0, 1), 1)
    for i in range(n_ops):
        for j in sorted(set(int(x) for x in i + 1 + rng.integers(0, 2 * fan, size=fan))):
            if j < n_ops:
                g.edge(i, j, [W.ident(0), W.ALL if (i + j) % 5 == 0 else W.ident(1)])
    ops, edges, _ = g.finish()
    mach = W.Machine(nodes, gpus, 3, 2)
    # tasks shorter, as long as and longer than a transfer, so that the horizon falls before, among and behind the events of an op
    cost = rng.integers(1, 10 ** rng.integers(1, 5, size=(n_ops, 1)) + 1, size=(n_ops, parts)).astype("<u4")
    cfgs = draw(rng, ops, 24, nodes * gpus, parts, (1, 2, 3, 4, 8, 16, 48, 64), strides=True)
    refined = {"params": (rng.integers(0, 3, size=n_ops).astype("<u4") * 5000, rng.integers(0, 4, size=n_ops).astype(np.uint8))} if params else {}
    check(B, ops, edges, mach, cost, cfgs, kernel="k_loop_batch", chain_steps=4, **refined)

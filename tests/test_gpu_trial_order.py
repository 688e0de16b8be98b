"""Trials ordered by length (k_trial_class, k_trial_place, trial_first_place): from one per SIMD on, every trial of a call runs exactly once
wherever its place in the list is, whatever mix of full, resumed and refused ones the call holds.  Section 5.3: the result of a trial is the full
simulation of the mutated strategy; the oracle gives it."""
import numpy as np
import pytest

import oracle
from paper_1807_05358_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_05358_amd import binding
    return binding


# one more than the SIMDs of the card; a last round of places that is not full; more trials than wavefronts at once (both ways of drawing);
# a graph with its state in memory; extents beyond 16 bits (the other event loop)
@pytest.mark.parametrize("config_id,C,M,wide", [(0, 1, 1025, False), (0, 3, 700, False), (1, 2, 3001, False), (2, 1, 1100, False), (0, 2, 777, True)])
def test_every_trial_runs_once_in_any_order(B, config_id, C, M, wide):
    import torch
    w = W.workload(config_id)
    ops = w.ops.copy()
    if wide:
        ops["extent"][:, 0] = 70000
    cfg0 = w.strategies(C)
    muts = w.mutations(M, C).copy()
    rng = np.random.default_rng(M)
    muts["op"][rng.integers(0, M, 5), rng.integers(0, C, 5)] = w.n_ops + 3           # names no op: invalid
    muts["cfg"]["deg"][rng.integers(0, M, 5), rng.integers(0, C, 5), 0] = 0          # no configuration: invalid
    print(f"trials: config {config_id}, {C} chains x {M} proposals, wide {wide}", flush=True)
    cfgs = np.repeat(cfg0[None], M, 0)
    known = muts["op"] < w.n_ops
    m, c = np.nonzero(known)
    cfgs[m, c, muts["op"][m, c]] = muts["cfg"][m, c]
    want = oracle.simulate_batch(ops, w.edges, w.machine, w.cost, cfgs.reshape(M * C, -1), n_threads=16).reshape(M, C)
    want[~known] = np.uint64(2 ** 64 - 1)
    assert len(np.unique(want)) >= 20          # (neighbouring trials differ: one in another's place would be seen)
    sim = B.Simulator(ops, w.edges, w.machine, w.cost)
    ch = B.Chains(sim, cfg0)
    d = ch.upload_mutations(muts)
    got = ch.try_mutations(d, M).cpu().numpy().view("<u8")
    assert np.array_equal(got, want)
    # a workspace with room for the wavefronts' slots alone is still enough
    need = B.ff_sim_delta_try_workspace_bytes(ch.handle, M)
    less = need - (M * C * 8 + 255) // 256 * 256
    ws = torch.empty(less, dtype=torch.uint8, device="cuda")
    out = torch.zeros((M, C), dtype=torch.int64, device="cuda")
    B.ff_sim_set_workspace(sim.handle, ws.data_ptr(), less)
    B.ff_sim_delta_try(ch.handle, d.data_ptr(), M, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert np.array_equal(out.cpu().numpy().view("<u8"), want)
    assert B.lib().ff_sim_set_workspace(sim.handle, ws.data_ptr(), less - 256) == B.FF_OK
    assert B.lib().ff_sim_delta_try(ch.handle, d.data_ptr(), M, out.data_ptr(), None) == B.FF_EWORKSPACE
    torch.cuda.synchronize()
    ch.close()
    sim.close()

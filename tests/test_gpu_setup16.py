"""The set-up of four edges at a time (kept_edges16: rows of 16 lanes, state in LDS) and the release of edges asked for early (run_loop): numbers of ops and
edges that do not divide by four, several edges into one consumer, tensors of one to four dims, degrees that do not divide the extents, general
strategies and explicit devices, extents up to 16 bits.  Every result is the oracle's (Section 5.1)."""
import numpy as np
import pytest

import oracle
from helpers import random_graph
from paper_1807_05358_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_05358_amd import binding
    return binding


@pytest.mark.parametrize("n_ops", [1, 2, 3, 5, 8, 16, 17, 30])
@pytest.mark.parametrize("form", ["regular", "general", "devmaps", "long"])
def test_small_graphs_with_up_to_16_parts(B, n_ops, form):
    rng = np.random.default_rng(1000 * n_ops + len(form))
    ops, edges, _ = random_graph(rng, n_ops)
    if form == "long":
        # extents up to the largest that the kept rows hold: quotients just below and at whole numbers
        wide = rng.random(ops["extent"].shape) < 0.5
        ops["extent"] = np.where(wide & (ops["extent"] > 1), rng.choice([65535, 65534, 65521, 32768, 4097], ops["extent"].shape), ops["extent"])
        ops["extent"][np.prod(ops["extent"].astype(float), axis=1) >= 2 ** 29] = 16
        ops["extent"][np.arange(4)[None, :] >= ops["ndim"][:, None]] = 1
    mach = W.Machine(4, 4, 11, 7, 3, 40) if form != "general" else W.Machine(3, 5, 11, 7, 3, 40)
    cost = rng.integers(1, 9000, size=(n_ops, 16)).astype("<u4")
    cfgs = W.strategies(ops, 40, n_ops, mach.n_devices, 16, (1, 2, 3, 4, 5, 7, 8, 11, 13, 16))
    if form == "general":
        cfgs["dev_stride"] = rng.integers(0, 9, cfgs.shape)
    maps = W.device_maps(cfgs, mach.n_devices, 3) if form == "devmaps" else None
    print(f"set-up: {n_ops} ops, {len(edges)} edges, {form}", flush=True)
    want = oracle.simulate_batch(ops, edges, mach, cost, cfgs, n_threads=8, devmaps=maps)
    sim = B.Simulator(ops, edges, mach, cost)
    assert np.array_equal(sim.simulate(cfgs, devmaps=maps), want)
    if maps is None:
        # a chain set up the same way, then changed op by op
        ch = B.Chains(sim, cfgs[:3])
        assert np.array_equal(ch.start_ns(), want[:3])
        muts = W.mutation_chains(ops, 6, 3, 9, mach.n_devices, 16, (1, 2, 3, 4, 5, 7, 8, 11, 13, 16))
        got = ch.delta(ch.upload_mutations(muts), 6).cpu().numpy().view("<u8")
        for c in range(3):
            assert np.array_equal(got[:, c], oracle.simulate_delta_chain(ops, edges, mach, cost, cfgs[c], muts[:, c]))
        ch.close()
    sim.close()

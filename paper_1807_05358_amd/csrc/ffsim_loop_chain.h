// Chains on kept set-up: the steps of ffsim_chain.h and trial proposals with the event loop of ffsim_loop.h.
//
// Against run_events the loop itself gains what it gains in a batch (see run_loop), and a change of one op recomputes the
// kept rows of that op's edges only, also where the simulation starts from time 0.  Graphs of up to 64 ops keep the
// state of a chain or of a trial in LDS.  A pass, against the same bookkeeping on run_events: one chain of 16 changes on the NMT-shaped
// graph 1000 -> 619 ms, 4096 trials there 189 -> 95 ms, 1024 chains x 16 search steps (Inception-v3-shaped,
// chains created and closed) 112 -> 73 ms, 64 chains x 256 steps (AlexNet-shaped, parameter traffic) 77.0 -> 50.0 ms,
// its neighbour sweep 0.876 -> 0.639 ms.
#pragma once
#include "ffsim_chain.h"
#include "ffsim_loop_kernels.h"

namespace ffsim {

// LDS of one wavefront: (chains: the strategy,) the state if it is kept there, device and link rows (64 bits each: the form
// with 64-bit link rows uses the same memory), tags
__host__ __device__ inline size_t loop_chain_lds_bytes(const SimDev& S, uint32_t rowl, bool lds, bool strategy) {
    return (strategy ? (size_t)S.n_ops_pad * 8 : 0) + (lds ? slot_layout(S.n_ops, S.n_ops_pad, S.n_edges, S.n_kept, rowl, true).bytes : 0) +
           (size_t)S.n_rows * 8 + ((S.n_rows + 15) & ~15u);
}

__device__ __forceinline__ void carve_rows64(LoopMem& mem, unsigned char* lds, const SimDev& S) {
    mem.crow = (u64*)lds;
    mem.lrow64 = mem.crow + S.n_dev;
    mem.lrow = (uint32_t*)mem.lrow64;
    mem.tag = (uint8_t*)(lds + (size_t)S.n_rows * 8);
}

// Recomputes the kept rows of every edge of op mo.  Edges with an end whose configuration is not valid for it are left as they
// are: no simulation reads them before that end changes.
template <int ROWL, class SimX>
__device__ __forceinline__ void refresh_rows_for_op(const SimX& m, const LoopMem& mem, uint32_t mo) {
    const OpCfg c = m.cfg(mo);
    if (!cfg_ok(m.T.ops[mo], c, m.S)) return;
    const uint32_t ib = m.T.ops[mo].in_begin, n_in = m.T.ops[mo].in_end - ib;
    const uint32_t ob = m.T.ops[mo].out_begin, n_out = m.T.ops[mo].out_end - ob;
    for (uint32_t t = 0; t < n_in + n_out; t++) {
        const bool in = t < n_in;
        const DEdge e = in ? m.T.in_edges[ib + t] : m.T.edges[ob + (t - n_in)];
        const uint32_t other = in ? e.src : e.dst;
        const OpCfg co = m.cfg(other);
        if (!cfg_ok(m.T.ops[other], co, m.S)) continue;
        uint32_t* row = mem.rows + (size_t)mem.edge_lite[e.eid].row * ROWL;
        if (SimX::kOvr && mem.priv) row = mem.priv + (size_t)t * (KEPT_ROWS * ROWL);     // (in-edges, then out-edges: see run_loop)
        kept_edge<ROWL>(m, row, e, in ? co : c, in ? c : co);
    }
    __threadfence_block();
    wave_sync();
}

// One simulation, from time 0 (k = 0; fill: no edge has kept rows yet) or from snapshot k with op mo changed from
// configuration ocfg.  Result as for run_loop, never RESULT_RETRY: a run that books a link more than 2^32 ns ahead is
// started again with 64-bit link rows, under a tag of its own: the first run may have gone on for some steps with times that did not fit,
// and what it recorded must not be taken for the second one's, which may re-join the accepted timeline without writing the same entries.
template <bool RECORD, int Q, int ROWL, class SimX>
__device__ __forceinline__ u64 simulate_loop(SimX& m, const LoopMem& mem, StrategyClass cls, Counters& cnt, Recorder& rec, bool fill, uint32_t k,
                                             uint32_t mo, uint2 ocfg, uint32_t pend_new, u64& mk) {
    LoopState st;
    const Recorder rec0 = rec;
    const Counters cnt0 = cnt;
    auto patch = [&]() {
        patch_states_for_op<ROWL>(m, 1, [&](uint32_t) { return mem.words; }, mo, ocfg, pend_new);
        wave_sync();
    };
    u64 rc = RESULT_RETRY;
    bool fits = true;
    if (k == 0) {
        init_loop<Q, ROWL>(m, mem, st, cnt, fill);
    } else {
        fits = load_loop_snapshot<Q, ROWL, false>(m, mem, st, rec, k);
        patch();
    }
    if (fits) {
        rc = cls == STRATEGY_REGULAR ? run_loop<RECORD, true, false, Q, ROWL>(m, mem, st, cnt, rec)
                                     : run_loop<RECORD, false, false, Q, ROWL>(m, mem, st, cnt, rec);
        if (!rc) mk = loop_makespan(m, mem, st);
    }
    if (rc == RESULT_RETRY) {
        rec = rec0;
        rec.tag |= 1ull << 63;
        cnt = cnt0;
        if (k == 0) {
            init_loop<Q, ROWL, true>(m, mem, st, cnt, false);
        } else {
            load_loop_snapshot<Q, ROWL, true>(m, mem, st, rec, k);
            patch();
        }
        rc = run_loop<RECORD, false, false, Q, ROWL, true>(m, mem, st, cnt, rec);
        if (!rc) mk = loop_makespan<true>(m, mem, st);
    }
    return rc;
}

template <bool LDSW, int Q, int ROWL, class SimX>
struct LoopEngine {
    SimX& m;
    const ChainMem& cm;
    const LoopMem& mem;
    bool tied;                 // tied configurations: a change concerns several ops, every simulation sets up all edges
    bool filled;               // every edge between ops with valid configurations has its kept rows
    u64 mk;
    static constexpr int kRowl = ROWL;
    __device__ __forceinline__ StrategyClass validate() {
        const StrategyClass cls = validate_loop<Q>(m, mem);
        if (cls == STRATEGY_INVALID && !filled) {
            // a chain that starts from an invalid strategy: later changes may mend it op by op
            for (uint32_t j = 0; j < m.S.n_ops; j++) op_changed(j);
            filled = true;
        }
        return cls;
    }
    __device__ __forceinline__ void op_changed(uint32_t mo) const { if (!tied) refresh_rows_for_op<ROWL>(m, mem, mo); }
    __device__ __forceinline__ void op_reverted(uint32_t mo) const { op_changed(mo); }
    __device__ __forceinline__ u64 simulate(StrategyClass cls, Counters& cnt, Recorder& rec, uint32_t k, uint32_t mo, uint2 ocfg, uint32_t pend_new) {
        const bool fill = tied || !filled;
        filled = true;
        return simulate_loop<true, Q, ROWL>(m, mem, cls, cnt, rec, fill, k, mo, ocfg, pend_new, mk);
    }
    __device__ __forceinline__ u64 makespan() const { return mk; }
    __device__ __forceinline__ void finish() const { if (LDSW) copy_u32(cm.rows, mem.rows, m.S.n_kept * ROWL); }
};

// LDSW, Q, ROWL as for k_loop_batch; EXT, GPN as for k_sim_chain_steps
template <bool LDSW, int Q, int ROWL, int EXT, int GPN>
__global__ __launch_bounds__(WAVE) void k_loop_chain_steps(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ edges,
                                                           const DEdge* __restrict__ in_edges, const OpLite* __restrict__ op_lite,
                                                           const EdgeLite* __restrict__ edge_lite, const uint32_t* __restrict__ cost,
                                                           const uint32_t* __restrict__ magic, unsigned char* chain_mem, size_t chain_stride,
                                                           uint32_t n_snaps, uint32_t C, const uint32_t* __restrict__ muts, uint32_t n_steps,
                                                           u64* __restrict__ out_ns, uint32_t* chain_flags, SearchDev search, uint32_t n_segs,
                                                           SpareBlocks spare) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const Tables T{ops, edges, in_edges, cost};
    if (blockIdx.x >= C * n_segs) return;
    const ChainSeg seg = chain_segment(blockIdx.x, C, chain_segments(blockIdx.x, C, n_segs, spare), n_steps, chain_mem, chain_stride, chain_flags, spare);
    if (seg.p >= seg.n) return;
    uint2* cfg_lds = (uint2*)lds_raw;
    unsigned char* lds = lds_raw + (size_t)S.n_ops_pad * 8;
    const ChainMem cm = carve_chain(seg.block, S, n_snaps, ROWL);
    LoopMem mem;
    mem.priv = nullptr;
    mem.op_lite = op_lite;
    mem.edge_lite = edge_lite;
    mem.links = (const uint4*)(magic + loop_links_at(S.gpus_per_node, S.n_nodes, S.n_ops));
    // the kept rows do not belong to the strategy yet: a chain's first launch, and segments of its steps
    const bool fresh = (!muts && !search.enabled) || seg.n > 1;
    if (LDSW) {
        const SlotLayout sl = slot_layout(S.n_ops, S.n_ops_pad, S.n_edges, S.n_kept, ROWL, true);
        carve_lds_state(mem, lds, sl, S, op_lite, edge_lite);
        carve_rows64(mem, lds + sl.bytes, S);
        if (!fresh) copy_u32(mem.rows, cm.rows, S.n_kept * ROWL);
    } else {
        mem.words = cm.words;
        mem.hdr = cm.hdr;
        mem.rows = cm.rows;
        mem.spill_key = cm.spill_key;
        mem.spill_op = cm.spill_op;
        carve_rows64(mem, lds, S);
    }
    const WaveLds L{mem.crow, nullptr, nullptr, mem.tag};
    const uint32_t magic_v = load_magic(magic);
    for (uint32_t i = lane_id(); i < S.n_ops; i += WAVE) cfg_lds[i] = cm.cfgs[i];
    wave_sync();
    typedef SimT<false, EXT, GPN> SimX;
    SimX m{S, T, cfg_lds, mem.words, nullptr, L, magic_v, 0, false, NO_OVERRIDE, make_uint2(0, 0), nullptr, true};
    if (EXT) { m.links = (const uint4*)(magic + LINK_TABLE_AT); m.node_links = m.links + (size_t)S.gpus_per_node * S.gpus_per_node; }
    if (EXT >= 2 && S.ties) m.tie = magic + tie_table_at(S.gpus_per_node, S.n_nodes);
    m.want_sort = true;          // a later step may make the strategy a general one: the kept rows are always complete
    LoopEngine<LDSW, Q, ROWL, SimX> en{m, cm, mem, EXT >= 2 && S.ties, !fresh, 0};
    chain_steps(en, m, S, cm, cfg_lds, n_snaps, seg, C, muts, n_steps, out_ns, search);
}

// Trial mutations (see k_sim_chain_try).  The rows of the changed op's edges are the trial's own: in LDS with a copy of all
// others, else in its slot of the workspace beside the chain's rows, which are only read.
template <bool LDSW, int Q, int ROWL, int EXT, int GPN>
__global__ __launch_bounds__(WAVE) void k_loop_chain_try(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ edges,
                                                         const DEdge* __restrict__ in_edges, const OpLite* __restrict__ op_lite,
                                                         const EdgeLite* __restrict__ edge_lite, const uint32_t* __restrict__ cost,
                                                         const uint32_t* __restrict__ magic, const unsigned char* __restrict__ chain_mem,
                                                         size_t chain_stride, uint32_t n_snaps, uint32_t C, const uint32_t* __restrict__ muts,
                                                         uint32_t M, u64* __restrict__ out_ns, const uint32_t* __restrict__ chain_flags,
                                                         uint32_t* __restrict__ next_item, unsigned char* __restrict__ ws, size_t slot_stride,
                                                         const uint32_t* __restrict__ order, uint32_t n_simds) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const Tables T{ops, edges, in_edges, cost};
    const SlotLayout sl = slot_layout(S.n_ops, S.n_ops_pad, S.n_edges, S.n_kept, ROWL, LDSW);
    unsigned char* slot = LDSW ? lds_raw : ws + (size_t)blockIdx.x * slot_stride;
    const bool tied = EXT >= 2 && S.ties;
    LoopMem mem;
    mem.op_lite = op_lite;
    mem.edge_lite = edge_lite;
    mem.links = (const uint4*)(magic + loop_links_at(S.gpus_per_node, S.n_nodes, S.n_ops));
    if (LDSW) {
        carve_lds_state(mem, lds_raw, sl, S, op_lite, edge_lite);
    } else {
        mem.words = (u64*)(slot + sl.words);
        mem.hdr = (uint4*)(slot + sl.hdr);
        mem.rows = (uint32_t*)(slot + sl.rows);
        mem.spill_key = (u64*)(slot + sl.spill_key);
        mem.spill_op = (uint32_t*)(slot + sl.spill_op);
    }
    mem.priv = (LDSW || tied) ? nullptr : mem.rows;
    carve_rows64(mem, LDSW ? lds_raw + sl.bytes : lds_raw, S);
    const WaveLds L{mem.crow, nullptr, nullptr, mem.tag};
    const uint32_t magic_v = load_magic(magic);
    const uint32_t total = M * C;
    for (bool first = order != nullptr;;) {
        const uint32_t at = first ? trial_first_place(blockIdx.x, gridDim.x, n_simds) : trial_next_place(next_item, order ? gridDim.x : 0u);
        first = false;
        if (at >= total) break;
        const uint32_t id = order ? first_u32(order[at]) : at;
        const uint32_t c = id % C;
        // the chain is only read here
        const ChainMem cm = carve_chain(const_cast<unsigned char*>(chain_mem) + (size_t)c * chain_stride, S, n_snaps, ROWL);
        ChainMeta meta = *cm.meta;
        meta.step = first_u64(meta.step);
        meta.n_valid = first_u32(meta.n_valid);
        meta.stale = first_u32(meta.stale);
        const uint32_t* mu = muts + (size_t)id * 3;     // [M][C] records {op, cfg.x, cfg.y}
        const uint32_t op = first_u32(mu[0]);
        u64 mk = RESULT_INVALID;
        if (op < S.n_ops && first_u32(chain_flags[c]) == 0) {
            const uint2 ocfg = cm.cfgs[op];
            SimT<true, EXT, GPN> m{S, T, cm.cfgs, mem.words, nullptr, L, magic_v, 0, false, op, make_uint2(first_u32(mu[1]), first_u32(mu[2])),
                                   nullptr, false};
            if (EXT) { m.links = (const uint4*)(magic + LINK_TABLE_AT); m.node_links = m.links + (size_t)S.gpus_per_node * S.gpus_per_node; }
            if (EXT >= 2 && S.ties) m.tie = magic + tie_table_at(S.gpus_per_node, S.n_nodes);
            m.want_sort = true;
            m.ov_in = ops[op].in_end - ops[op].in_begin;
            const StrategyClass cls = validate_loop<Q>(m, mem);
            if (cls != STRATEGY_INVALID) {
                Counters cnt = {};
                Recorder rec{nullptr, cm.snap_words, nullptr, cm.snap_free, meta.step, 0, first_u32(meta.loc), n_snaps, 1, 0, 0};
                uint32_t k = 0, pend_new = 0;
                if (!tied) {
                    if (LDSW) {
                        copy_u32(mem.rows, cm.rows, S.n_kept * ROWL);
                        wave_sync();
                    } else {
                        mem.rows = cm.rows;
                    }
                    refresh_rows_for_op<ROWL>(m, mem, op);
                    if (!meta.stale && meta.n_valid > 1 && meta.step != 0) k = resume_point<ROWL>(m, cm.end_of, meta, op, ocfg, pend_new);
                }
                const u64 rc = simulate_loop<false, Q, ROWL>(m, mem, cls, cnt, rec, tied, k, op, ocfg, pend_new, mk);
                if (rc) mk = rc;
            }
        }
        if (lane_id() == 0) out_ns[id] = mk;
        wave_sync();
    }
}

// Where the nodes of large graphs keep their state: where the chains have their snapshots (per_chain slots in every block; the search leaves the
// timelines to be recorded again), then in memory of their own.
struct NodeSlots {
    unsigned char* blocks;     // the first chain's snapshots
    size_t stride, bytes;      // from chain to chain; of a slot
    uint32_t per_chain, in_blocks;
    unsigned char* more;
    __device__ __forceinline__ unsigned char* of(uint32_t b) const {
        return b < in_blocks ? blocks + (size_t)(b / per_chain) * stride + (size_t)(b % per_chain) * bytes : more + (size_t)(b - in_blocks) * bytes;
    }
};

// One full simulation per strategy and wavefront: the first *n of the strategies of a search that looks ahead (ffsim_ahead.h).  As k_loop_batch, but
// strategies that book a link more than 2^32 ns ahead are simulated again here.
template <bool LDSW, int Q, int ROWL, int EXT, int GPN>
__global__ __launch_bounds__(WAVE) void k_loop_nodes(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ edges, const DEdge* __restrict__ in_edges,
                                                     const OpLite* __restrict__ op_lite, const EdgeLite* __restrict__ edge_lite,
                                                     const uint32_t* __restrict__ cost, const uint32_t* __restrict__ magic,
                                                     const uint2* __restrict__ strategies, const uint32_t* __restrict__ n, uint32_t capacity,
                                                     u64* __restrict__ out_ns, NodeSlots slots) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const uint32_t b = blockIdx.x;
    if (b >= *n || b >= capacity) return;
    const Tables T{ops, edges, in_edges, cost};
    const SlotLayout sl = slot_layout(S.n_ops, S.n_ops_pad, S.n_edges, S.n_kept, ROWL, LDSW);
    LoopMem mem;
    mem.priv = nullptr;
    mem.op_lite = op_lite;
    mem.edge_lite = edge_lite;
    mem.links = (const uint4*)(magic + loop_links_at(S.gpus_per_node, S.n_nodes, S.n_ops));
    if (LDSW) {
        carve_lds_state(mem, lds_raw, sl, S, op_lite, edge_lite);
        carve_rows64(mem, lds_raw + sl.bytes, S);
    } else {
        unsigned char* slot = slots.of(b);
        mem.words = (u64*)(slot + sl.words);
        mem.hdr = (uint4*)(slot + sl.hdr);
        mem.rows = (uint32_t*)(slot + sl.rows);
        mem.spill_key = (u64*)(slot + sl.spill_key);
        mem.spill_op = (uint32_t*)(slot + sl.spill_op);
        carve_rows64(mem, lds_raw, S);
    }
    const WaveLds L{mem.crow, nullptr, nullptr, mem.tag};
    const uint32_t magic_v = load_magic(magic);
    SimT<false, EXT, GPN> m{S, T, strategies + (size_t)b * S.n_ops, mem.words, nullptr, L, magic_v, 0, false, NO_OVERRIDE, make_uint2(0, 0), nullptr, true};
    if (EXT) { m.links = (const uint4*)(magic + LINK_TABLE_AT); m.node_links = m.links + (size_t)S.gpus_per_node * S.gpus_per_node; }
    if (EXT >= 2 && S.ties) m.tie = magic + tie_table_at(S.gpus_per_node, S.n_nodes);
    u64 mk = RESULT_INVALID;
    const StrategyClass cls = validate_loop<Q>(m, mem);
    if (cls != STRATEGY_INVALID) {
        Counters cnt = {};
        Recorder none = {};
        LoopState st;
        m.want_sort = cls != STRATEGY_REGULAR;
        init_loop<Q, ROWL>(m, mem, st, cnt, true);
        const Pace pace{0, S.n_ops};
        u64 rc = cls == STRATEGY_REGULAR ? run_loop<false, true, false, Q, ROWL>(m, mem, st, cnt, none, pace)
                                         : run_loop<false, false, false, Q, ROWL>(m, mem, st, cnt, none, pace);
        if (!rc) mk = loop_makespan(m, mem, st);
        if (rc == RESULT_RETRY) {
            m.want_sort = true;          // (the general form's rows)
            init_loop<Q, ROWL, true>(m, mem, st, cnt, true);
            rc = run_loop<false, false, false, Q, ROWL, true>(m, mem, st, cnt, none);
            if (!rc) mk = loop_makespan<true>(m, mem, st);
        }
        if (rc) mk = rc;
    }
    if (lane_id() == 0) out_ns[b] = mk;
}

}  // namespace ffsim

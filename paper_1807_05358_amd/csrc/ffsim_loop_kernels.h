// Batch kernel on kept set-up (ffsim_loop.h): one candidate strategy per wavefront.
#pragma once
#include "ffsim_kernels.h"
#include "ffsim_loop.h"

namespace ffsim {

// ---- memory of one candidate -----------------------------------------------------------------
//
// In LDS (small graphs): words, op records (kept and static), edge records, kept rows, then device and link rows and the tags.
// In HBM (a slot of the caller's workspace per resident wavefront): words, op records, spill list, kept rows; only
// device and link rows and the tags are in LDS.
struct SlotLayout { size_t words, hdr, op_lite, edge_lite, spill_key, spill_op, rows, bytes; };
__host__ __device__ inline SlotLayout slot_layout(uint32_t n_ops, uint32_t n_ops_pad, uint32_t n_edges, uint32_t n_kept, uint32_t rowl, bool lds) {
    SlotLayout s;
    size_t b = 0;
    s.words = b; b += (size_t)n_ops * rowl * 8;
    s.hdr = b; b += (size_t)(lds ? n_ops : n_ops_pad) * 16;
    s.op_lite = b; b += lds ? (size_t)n_ops * sizeof(OpLite) : 0;
    s.edge_lite = b; b += lds ? (size_t)n_edges * sizeof(EdgeLite) : 0;
    s.spill_key = b; b += lds ? 0 : (size_t)n_ops_pad * 8;
    s.spill_op = b; b += lds ? 0 : (size_t)n_ops_pad * 4;
    s.rows = b; b += (size_t)n_kept * rowl * 4;
    s.bytes = lds ? (b + 15) & ~(size_t)15 : (b + 255) & ~(size_t)255;
    return s;
}
// device rows (64 bits), link rows (32 bits), tags
__host__ __device__ inline size_t loop_rows_bytes(uint32_t n_rows, uint32_t n_dev) { return (size_t)n_dev * 8 + (size_t)(n_rows - n_dev) * 4; }
__host__ __device__ inline size_t loop_lds_bytes(uint32_t n_rows, uint32_t n_dev) { return loop_rows_bytes(n_rows, n_dev) + ((n_rows + 15) & ~15u); }

__device__ __forceinline__ void carve_rows(LoopMem& mem, unsigned char* lds, const SimDev& S) {
    mem.crow = (u64*)lds;
    mem.lrow = (uint32_t*)(mem.crow + S.n_dev);
    mem.lrow64 = nullptr;
    mem.tag = (uint8_t*)(lds + loop_rows_bytes(S.n_rows, S.n_dev));
}

// n words of 32 bits between LDS and HBM
__device__ __forceinline__ void copy_u32(uint32_t* __restrict__ dst, const uint32_t* __restrict__ src, uint32_t n) {
    constexpr uint32_t FEW = 8;
    for (uint32_t b = 0; b < n; b += FEW * WAVE) {
        uint32_t v[FEW];
#pragma unroll
        for (uint32_t u = 0; u < FEW; u++) { const uint32_t t = b + u * WAVE + lane_id(); v[u] = src[t < n ? t : n - 1]; }
#pragma unroll
        for (uint32_t u = 0; u < FEW; u++) { const uint32_t t = b + u * WAVE + lane_id(); if (t < n) dst[t] = v[u]; }
    }
}

// the parts of a candidate's state that live in LDS with it, and copies of the static records
__device__ __forceinline__ void carve_lds_state(LoopMem& mem, unsigned char* lds, const SlotLayout& sl, const SimDev& S, const OpLite* op_lite,
                                                const EdgeLite* edge_lite) {
    mem.words = (u64*)(lds + sl.words);
    mem.hdr = (uint4*)(lds + sl.hdr);
    mem.rows = (uint32_t*)(lds + sl.rows);
    mem.spill_key = nullptr;
    mem.spill_op = nullptr;
    copy_u32((uint32_t*)(lds + sl.op_lite), (const uint32_t*)op_lite, S.n_ops * (uint32_t)(sizeof(OpLite) / 4));
    copy_u32((uint32_t*)(lds + sl.edge_lite), (const uint32_t*)edge_lite, S.n_edges * (uint32_t)(sizeof(EdgeLite) / 4));
    mem.op_lite = (const OpLite*)(lds + sl.op_lite);
    mem.edge_lite = (const EdgeLite*)(lds + sl.edge_lite);
    wave_sync();
}

// LDSW: the candidate's whole state is in LDS.  Q: LoopQueue.  ROWL: lanes per row (16 where no op has more parts).
template <bool STATS, bool LDSW, int Q, int ROWL, int EXT, int GPN>
__global__ __launch_bounds__(WAVE) void k_loop_batch(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ in_edges,
                                                     const OpLite* __restrict__ op_lite, const EdgeLite* __restrict__ edge_lite,
                                                     const uint32_t* __restrict__ cost, const uint32_t* __restrict__ magic,
                                                     const uint2* __restrict__ strategies, uint32_t B, u64* __restrict__ out_ns,
                                                     Counters* __restrict__ stats, unsigned char* __restrict__ ws, size_t slot_stride,
                                                     const DEdge* __restrict__ edges, const uint16_t* __restrict__ devmaps) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const Tables T{ops, edges, in_edges, cost};
    const SlotLayout sl = slot_layout(S.n_ops, S.n_ops_pad, S.n_edges, S.n_kept, ROWL, LDSW);
    LoopMem mem;
    mem.priv = nullptr;
    mem.op_lite = op_lite;
    mem.edge_lite = edge_lite;
    mem.links = (const uint4*)(magic + loop_links_at(S.gpus_per_node, S.n_nodes, S.n_ops));
    if (LDSW) {
        carve_lds_state(mem, lds_raw, sl, S, op_lite, edge_lite);
        carve_rows(mem, lds_raw + sl.bytes, S);
    } else {
        unsigned char* slot = ws + (size_t)blockIdx.x * slot_stride;
        mem.words = (u64*)(slot + sl.words);
        mem.hdr = (uint4*)(slot + sl.hdr);
        mem.rows = (uint32_t*)(slot + sl.rows);
        mem.spill_key = (u64*)(slot + sl.spill_key);
        mem.spill_op = (uint32_t*)(slot + sl.spill_op);
        carve_rows(mem, lds_raw, S);
    }
    const WaveLds L{mem.crow, nullptr, nullptr, mem.tag};
    const uint32_t magic_v = load_magic(magic);
    for (uint32_t b = blockIdx.x; b < B; b += gridDim.x) {
        Counters cnt = {};
        Recorder none = {};
        SimT<false, EXT, GPN> m{S, T, strategies + (size_t)b * S.n_ops, mem.words, nullptr, L, magic_v, 0, false, NO_OVERRIDE, make_uint2(0, 0), nullptr, true};
        if (EXT) {
            m.links = (const uint4*)(magic + LINK_TABLE_AT);
            m.node_links = m.links + (size_t)S.gpus_per_node * S.gpus_per_node;
            if (EXT >= 2 && S.ties) m.tie = magic + tie_table_at(S.gpus_per_node, S.n_nodes);
            if (devmaps) m.devmap = devmaps + (size_t)b * S.n_ops * WAVE;
        }
#ifdef FFSIM_PROFILE
        const u64 prof_t0 = __builtin_readcyclecounter();
#endif
        u64 mk = RESULT_INVALID;
        const StrategyClass cls = validate_loop<Q>(m, mem);
        if (cls != STRATEGY_INVALID) {
            LoopState st;
            m.want_sort = cls != STRATEGY_REGULAR;
            init_loop<Q, ROWL>(m, mem, st, cnt, true);
#ifdef FFSIM_PROFILE
            cnt.exit_code = __builtin_readcyclecounter() - prof_t0;   // reported as section 0
#endif
            const Pace pace{b / gridDim.x * S.n_ops, ((B - 1 - blockIdx.x) / gridDim.x + 1) * S.n_ops};
            u64 rc = cls == STRATEGY_REGULAR ? run_loop<false, true, STATS, Q, ROWL>(m, mem, st, cnt, none, pace)
                                             : run_loop<false, false, STATS, Q, ROWL>(m, mem, st, cnt, none, pace);
            mk = rc == RESULT_RETRY ? RESULT_MARK_RETRY : rc ? rc : loop_makespan(m, mem, st);
            if (STATS)   // diagnostics: tasks that never ran (0 in a correct run)
                for (uint32_t j = 0; j < S.n_ops; j++) cnt.n_stuck += __popcll(ballot(load_word<ROWL>(mem.words, j) != W_NONE));
        }
        if (lane_id() == 0) out_ns[b] = mk;
        if (STATS) store_counters(cnt, stats + b);
        wave_sync();
    }
}

}  // namespace ffsim

// What the event loop needs to know about every tensor edge and every op of one strategy, computed once per
// candidate (or once per change of a chain) and kept: the geometry of Section 5.1 step 2 does not depend on when a
// task finishes.  Used by the event loop of ffsim_loop.h; needs extents that fit 16 bits.
#pragma once
#include "ffsim_strategy.h"

namespace ffsim {

// Kept rows of an edge: KEPT_ROWS rows of 32-bit words, one word per part (ROWL words per row).  Ranges are pairs of
// 16-bit values (dims 0 and 1, dims 2 and 3), so that the intersection of a producer part with a consumer part is
// three packed instructions per pair of dims.  C: range of the producer's tensor that the consumer part of this
// lane reads (an empty range on lanes that are no part: they never meet a producer); P: box of the producer
// part of this lane.  (On a contributing edge both are taken in the consumer's tensor.)  Rows *2 exist only for
// tensors of more than two dims: a release of an edge of a two-dim tensor loads 5 rows of 256 bytes.
enum KeptRow : uint32_t {
    KR_F = 0,      // consumer part: device, node, place in its run (see kept_fields)
    KR_CLO, KR_CHI, KR_PLO, KR_PHI,          // dims 0, 1
    KR_SORT,       // EdgeLane::sortw, and in bits 24..30 the number of producer parts this consumer part reads
    KEPT_ROWS_2,   // rows of an edge of a tensor of one or two dims
    KR_CLO2 = KEPT_ROWS_2, KR_CHI2, KR_PLO2, KR_PHI2,      // dims 2, 3
    KEPT_ROWS      // rows of any other edge
};

// Kept record of an op (16 bytes, the same for all lanes): exeTime of its tasks, device offset | stride << 16, exeTime of the
// tasks of its first out-edge's consumer (the bound of a run of releases), number of parts | HDR_* flags.
constexpr uint32_t HDR_SPLIT01 = 1u << 16;   // dim 0 or 1 is split
constexpr uint32_t HDR_SPLIT23 = 1u << 17;   // dim 2 or 3 is split

// Static records, small enough to stay close (the full records are 176 bytes per op and 128 per edge).
struct EdgeLite { uint32_t word, in_pos, row, unused; };    // consumer | EL_* flags, position among the consumer's in-edges, first kept row
struct OpLite { uint32_t out_begin, out_end, param_bytes, unused; EdgeLite first; };   // first: copy of the first out-edge
constexpr uint32_t EL_DST = 0xffffu;
constexpr uint32_t EL_FOUR = 1u << 16;       // the tensor has more than two dims
constexpr uint32_t EL_CONTRIB = 1u << 17;    // contributing edge

// A word of KR_F: device 10 bits, node 10, then one bit per distance s = 1..7 "the part s lanes below is in the same
// run of consumer parts on one node" (the runs of the regular form: see EdgeLane), last run, wrapped, first_len - 1 (3).
__device__ __forceinline__ uint32_t kept_fields(const EdgeLane& el) {
    const uint32_t below = (1u << el.pos) - 1u;          // pos lanes of the run lie below this one
    const uint32_t fl = el.first_len ? el.first_len - 1 : 0u;
    return el.dev_c | (el.node_c << 10) | ((below & 0x7fu) << 20) | ((el.last_run_mask & 1u) << 27) | ((uint32_t)el.wrapped << 28) | (fl << 29);
}

// stores the consumer's side of an edge; n_inputs: producer parts read
template <int ROWL>
__device__ __forceinline__ void kept_store_consumer(uint32_t* row, const DEdge& e, const EdgeLane& el, uint32_t n_inputs, bool sort) {
    const uint32_t lane = lane_id();
    if (ROWL < WAVE && lane >= (uint32_t)ROWL) return;
    uint32_t* p = row + lane;
    p[KR_F * ROWL] = kept_fields(el);
    const uint32_t live = el.mine ? 0xffffffffu : 0u;
    p[KR_CLO * ROWL] = ((uint32_t)el.nlo[0] | ((uint32_t)el.nlo[1] << 16)) & live;
    p[KR_CHI * ROWL] = ((uint32_t)el.nhi[0] | ((uint32_t)el.nhi[1] << 16)) & live;
    if (e.src_ndim > 2) {
        p[KR_CLO2 * ROWL] = ((uint32_t)el.nlo[2] | ((uint32_t)el.nlo[3] << 16)) & live;
        p[KR_CHI2 * ROWL] = ((uint32_t)el.nhi[2] | ((uint32_t)el.nhi[3] << 16)) & live;
    }
    if (sort) p[KR_SORT * ROWL] = el.sortw | ((n_inputs & 0x7fu) << 24);
}

// stores the producer's side of an edge: the box of every part of the producer (configuration cp)
template <int ROWL, class SimX>
__device__ __forceinline__ void kept_store_producer(const SimX& m, uint32_t* row, const DEdge& e, const OpCfg& cp) {
    const uint32_t lane = lane_id();
    uint32_t lo[4], hi[4];
    if (SimX::kTrain && e.kind) {
        // the range of the consumer's tensor that the part contributes to
        const uint32_t digits = part_digits(cp, lane, m.magic_v);
#pragma unroll
        for (int d = 0; d < 4; d++) {
            int32_t l = 0, h = 1;
            if ((uint32_t)d < e.src_ndim) needed_range(e.map[d], e.src_extent[d], cp.x, digits, m.magic_v, l, h);
            lo[d] = (uint32_t)l; hi[d] = (uint32_t)h;
        }
    } else {
        const Box b = part_box(e.src_extent, cp, lane, m.magic_v);
#pragma unroll
        for (int d = 0; d < 4; d++) { lo[d] = b.lo[d]; hi[d] = b.hi[d]; }
    }
    if (ROWL < WAVE && lane >= (uint32_t)ROWL) return;
    // lanes beyond the parts hold boxes outside the tensor, possibly past 16 bits: they are never looked at
    uint32_t* p = row + lane;
    p[KR_PLO * ROWL] = (lo[0] & 0xffffu) | (lo[1] << 16);
    p[KR_PHI * ROWL] = (hi[0] & 0xffffu) | (hi[1] << 16);
    if (e.src_ndim > 2) {
        p[KR_PLO2 * ROWL] = (lo[2] & 0xffffu) | (lo[3] << 16);
        p[KR_PHI2 * ROWL] = (hi[2] & 0xffffu) | (hi[3] << 16);
    }
}

// how many producer parts (configuration cp) each consumer part reads through edge e, from its range
template <bool TRAIN>
__device__ __forceinline__ uint32_t kept_count_inputs(const DEdge& e, const OpCfg& cp, const EdgeLane& el, uint32_t magic_v) {
    if (TRAIN && e.kind) return count_contributors(e, cp, el.nlo, el.nhi, magic_v);
    uint32_t n = 1;
#pragma unroll
    for (int d = 0; d < 4; d++) {
        if ((uint32_t)d < e.src_ndim) {
            uint32_t c;
            if (cp.deg[d] == 1) {
                c = el.nhi[d] > el.nlo[d] ? 1u : 0u;           // the producer does not split this dim (uniform)
            } else if (e.map[d].src_dim < 0) {
                c = cp.deg[d];                                   // the whole extent is read: every part (uniform)
            } else {
                c = 0;
                if (el.nhi[d] > el.nlo[d])
                    c = owner_part((uint32_t)el.nhi[d] - 1, e.src_extent[d], cp.deg[d]) - owner_part((uint32_t)el.nlo[d], e.src_extent[d], cp.deg[d]) + 1;
            }
            n *= c;
        }
    }
    return n;
}

// the whole set-up of one edge: both sides; returns the number of producer parts each consumer part reads
template <int ROWL, class SimX>
__device__ __forceinline__ uint32_t kept_edge(const SimX& m, uint32_t* row, const DEdge& e, const OpCfg& cp, const OpCfg& cj) {
    const EdgeLane el = edge_lane(m, e, cj);
    const uint32_t n = kept_count_inputs<SimX::kTrain>(e, cp, el, m.magic_v);
    kept_store_consumer<ROWL>(row, e, el, n, m.want_sort);
    kept_store_producer<ROWL>(m, row, e, cp);
    return n;
}

// the kept record of op i, from its configuration and exeTime
__device__ __forceinline__ uint4 kept_header(const OpCfg& c, uint32_t exe) {
    return make_uint4(exe, c.off | (c.stride << 16), 0u,
                      c.parts | ((c.deg[0] > 1 || c.deg[1] > 1) ? HDR_SPLIT01 : 0u) | ((c.deg[2] > 1 || c.deg[3] > 1) ? HDR_SPLIT23 : 0u));
}

}  // namespace ffsim

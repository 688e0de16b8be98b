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

// Kept record of an op (16 bytes, the same for all lanes): exeTime of its tasks, device offset | stride << 16, the least exeTime
// among the consumers of its out-edges (the bound of a run of releases; all ones: no out-edge, 0: too many to look at), number of
// parts | HDR_* flags.
constexpr uint32_t HDR_SPLIT01 = 1u << 16;   // dim 0 or 1 is split
constexpr uint32_t HDR_SPLIT23 = 1u << 17;   // dim 2 or 3 is split
constexpr uint32_t HDR_RELEASES = 1u << 18;  // the op's tasks have something to release when they have finished

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

// ---- four edges at a time ----------------------------------------------------------------
//
// The set-up of all edges where rows have 16 lanes: lanes 16 g .. 16 g + 15 take the parts of the g-th of four edges, so everything about an edge
// is a value of a lane.  Against kept_edge one edge at a time: a quarter of the iterations, and the edge records of each come in one trip
// through the vector unit instead of several through the scalar unit that nothing hides (a graph of a dozen ops is set up once per candidate, from
// tables no wavefront of the compute unit has read before).
// Set-up of the tiny chain (5 edges) 19.0 -> 11.4 thousand clock ticks, of the AlexNet-shaped graph (11 edges) 39.7 -> 15.5; 64 x tiny chain 22.2 -> 19.1 us,
// 1024 x AlexNet-shaped 196 -> 190 us, with parameter traffic 296 -> 266.

// floor(n / d) with the lane's constant of load_magic for d (0 for d = 1); as div_by
__device__ __forceinline__ uint32_t div_lane(uint32_t n, uint32_t d, uint32_t m) { return d == 1 ? n : __umulhi(n, m); }

// index of part k along each dim, a byte each (part_digits with degrees that differ per lane); mg: the constants of the four degrees
__device__ __forceinline__ uint32_t part_digits_lane(const OpCfg& c, const uint32_t mg[4], uint32_t k) {
    uint32_t rem = k, packed = 0;
#pragma unroll
    for (int d = 3; d >= 0; d--) {
        const uint32_t q = div_lane(rem, c.deg[d], mg[d]);
        packed |= ((rem - q * c.deg[d]) & 0xffu) << (8 * d);
        rem = q;
    }
    return packed;
}

// index of the producer part that owns coordinate x (owner_part): a quotient below 64 from the reciprocal, put right by what remains
__device__ __forceinline__ uint32_t owner_part_lane(uint32_t x, uint32_t E, float rcp_E, uint32_t deg) {
    const uint32_t n = (x + 1) * deg - 1;
    uint32_t q = (uint32_t)((float)n * rcp_E);
    const int32_t r = (int32_t)(n - q * E);
    q += r >= (int32_t)E ? 1u : 0u;
    q -= r < 0 ? 1u : 0u;
    return q;
}

// pend: [n_ops][16] words of 64 bits, zero on entry; the low half of each receives the number of producer parts that consumer part reads
template <class SimX, class Rows>
__device__ __forceinline__ void kept_edges16(const SimX& m, Rows rows_of, u64* pend) {
    static_assert(!SimX::kTrain, "reading edges only");
    const SimDev& S = m.S;
    uint32_t lane = lane_id();
    asm volatile("" : "+v"(lane));        // (a number of its own: what follows from it is not to be kept for the event loop)
    const uint32_t k = lane & 15u, g = lane >> 4;
    const uint32_t G = m.gpn();
    for (uint32_t base = 0; base < S.n_edges; base += 4) {
        const bool live = base + g < S.n_edges;
        const DEdge* at = m.T.in_edges + (live ? base + g : S.n_edges - 1);
        static_assert(sizeof(DEdge) % 16 == 0, "in pieces of 16 bytes");
        uint4 piece[sizeof(DEdge) / 16];
#pragma unroll
        for (int t = 0; t < (int)(sizeof(DEdge) / 16); t++) piece[t] = ((const uint4*)at)[t];
        DEdge e;
        __builtin_memcpy(&e, piece, sizeof(DEdge));
        const OpCfg cp = unpack_cfg_lane(m.cfg_raw(e.src)), cj = unpack_cfg_lane(m.cfg_raw(e.dst));
        uint32_t mp[4], mj[4];
#pragma unroll
        for (int d = 0; d < 4; d++) {
            mp[d] = gather_u32(m.magic_v, (cp.deg[d] - 1) & 63u);
            mj[d] = gather_u32(m.magic_v, (cj.deg[d] - 1) & 63u);
        }
        const bool mine = k < cj.parts;
        const uint32_t dj = part_digits_lane(cj, mj, k);
        // Section 4: the range of every producer dim that the consumer part reads (needed_range), and how many producer parts that is
        uint32_t nlo[4], nhi[4], n_inputs = 1;
#pragma unroll
        for (int d = 0; d < 4; d++) {
            const DMap mp_d = e.map[d];
            const bool in = (uint32_t)d < e.src_ndim;
            const int32_t E = in ? (int32_t)e.src_extent[d] : 1;
            const uint32_t sd = (uint32_t)mp_d.src_dim & 3u, sh = 8u * sd;
            const uint32_t deg = (cj.x >> sh) & 0xffu, idx = (dj >> sh) & 0xffu;
            const uint32_t mg = sd == 0 ? mj[0] : (sd == 1 ? mj[1] : (sd == 2 ? mj[2] : mj[3]));
            const int32_t clo = (int32_t)div_lane(idx * mp_d.cext, deg, mg), chi = (int32_t)div_lane((idx + 1) * mp_d.cext, deg, mg);
            int32_t l = clo * (int32_t)mp_d.stride + mp_d.a, h = (chi - 1) * (int32_t)mp_d.stride + mp_d.b + 1;
            l = l < 0 ? 0 : (l > E ? E : l);
            h = h < 0 ? 0 : (h > E ? E : h);
            h = h < l ? l : h;
            const bool all = !in || mp_d.src_dim < 0;
            l = all ? 0 : l;
            h = all ? E : h;
            nlo[d] = (uint32_t)l;
            nhi[d] = (uint32_t)h;
            const float rcp_E = __builtin_amdgcn_rcpf((float)E);
            uint32_t c = owner_part_lane((uint32_t)h - 1, (uint32_t)E, rcp_E, cp.deg[d]) - owner_part_lane((uint32_t)l, (uint32_t)E, rcp_E, cp.deg[d]) + 1;
            c = h > l ? c : 0u;
            c = mp_d.src_dim < 0 ? cp.deg[d] : c;
            n_inputs *= in ? c : 1u;
        }
        // the part's device and its place among the consumer's parts (edge_lane)
        EdgeLane el;
        const bool consecutive = cj.stride == 1 && cj.parts <= S.n_dev && G <= MAX_RUN && !(SimX::kExt && m.devmap);
        const uint32_t n = cj.off + k * cj.stride;
        el.dev_c = n - div_magic(n, S.magic_dev, S.pass_dev) * S.n_dev;
        if (SimX::kExt && m.devmap) el.dev_c = mine ? m.devmap[(size_t)e.dst * WAVE + k] : 0u;
        el.node_c = m.node_of(el.dev_c);
        el.pos = 0; el.first_len = 0; el.last_run_mask = 0; el.wrapped = false; el.sortw = 0;
        if (m.want_sort) {
            uint32_t rank = 0;
            bool dup = false;
            for (uint32_t t = 0; t < 16; t++) {
                const uint32_t n2 = gather_u32(el.node_c, (lane & 48u) | t), d2 = gather_u32(el.dev_c, (lane & 48u) | t);
                const bool part = t < cj.parts;
                rank += (part && (n2 < el.node_c || (n2 == el.node_c && t < k))) ? 1u : 0u;
                dup = dup || (part && d2 == el.dev_c && t < k);
            }
            const uint32_t spos = mine ? rank : k;
            const uint32_t part_here = scatter_u32(k, (lane & 48u) | spos), node_here = scatter_u32(el.node_c, (lane & 48u) | spos);
            const uint32_t node_before = wave_shr1_u32(node_here);
            const bool head = k == 0 || k >= cj.parts || node_here != node_before;
            el.sortw = part_here | (spos << 6) | (node_here << 12) | ((uint32_t)head << 22) | ((uint32_t)(dup && mine) << 23);
        }
        if (consecutive) {
            const uint32_t node0 = m.node_of(cj.off), room = G - (cj.off - node0 * G), local_c = m.local_of(el.dev_c, el.node_c);
            el.first_len = cj.parts < room ? cj.parts : room;
            el.pos = k < el.first_len ? k : local_c;
            const uint32_t last = cj.off + cj.parts - 1;
            el.wrapped = last >= S.n_dev && m.node_of(last - S.n_dev) == node0;
            el.last_run_mask = (el.wrapped && k >= el.first_len && el.node_c == node0) ? 0xffffffffu : 0u;
        }
        // the box of the producer part (part_box)
        uint32_t blo[4], bhi[4];
        const uint32_t dp = part_digits_lane(cp, mp, k);
#pragma unroll
        for (int d = 0; d < 4; d++) {
            const uint32_t idx = (dp >> (8 * d)) & 0xffu;
            blo[d] = div_lane(idx * e.src_extent[d], cp.deg[d], mp[d]);
            bhi[d] = div_lane((idx + 1) * e.src_extent[d], cp.deg[d], mp[d]);
        }
        if (live) {
            uint32_t* p = rows_of(e.eid) + k;
            const uint32_t keep = mine ? 0xffffffffu : 0u;
            p[KR_F * 16] = kept_fields(el);
            p[KR_CLO * 16] = (nlo[0] | (nlo[1] << 16)) & keep;
            p[KR_CHI * 16] = (nhi[0] | (nhi[1] << 16)) & keep;
            p[KR_PLO * 16] = (blo[0] & 0xffffu) | (blo[1] << 16);
            p[KR_PHI * 16] = (bhi[0] & 0xffffu) | (bhi[1] << 16);
            if (m.want_sort) p[KR_SORT * 16] = el.sortw | ((n_inputs & 0x7fu) << 24);
            if (e.src_ndim > 2) {
                p[KR_CLO2 * 16] = (nlo[2] | (nlo[3] << 16)) & keep;
                p[KR_CHI2 * 16] = (nhi[2] | (nhi[3] << 16)) & keep;
                p[KR_PLO2 * 16] = (blo[2] & 0xffffu) | (blo[3] << 16);
                p[KR_PHI2 * 16] = (bhi[2] & 0xffffu) | (bhi[3] << 16);
            }
            // (several of the four edges may have one consumer)
            atomicAdd((unsigned int*)&pend[(size_t)e.dst * 16 + k], n_inputs);
        }
    }
}

}  // namespace ffsim

// Small kernels around the trial-mutation kernel: the list of a strategy's neighbours, the
// reduction over their times, and a counter reset.  Included by the host file only (the
// kernels here are not templates: one definition in the library).
#pragma once
#include "ffsim_chain.h"

namespace ffsim {

// ---- neighbour sweep (Section 8: is a strategy locally optimal?) --------------------------
//
// The neighbours of a strategy differ from it in the configuration of one op.  Neighbour k of
// the enumeration: ops op_begin..op_end-1 in order; per op every degree tuple of its list, in
// list order; per tuple every device offset 0..n_dev-1; stride 1.  first[o - op_begin] is the
// index of the first neighbour of op o.  Writes the same mutation for every chain ([M][C]).
// status: null, or one word that is nonzero if `first` could not be built (see k_neighbour_first): every
// mutation then names an op outside the graph, which the trial kernel answers with "invalid".
__global__ __launch_bounds__(WAVE) void k_neighbour_list(const uint32_t* __restrict__ tuple_ptr, const uint32_t* __restrict__ tuples,
                                                         const uint32_t* __restrict__ first, uint32_t op_begin, uint32_t op_end,
                                                         uint32_t n_dev, uint32_t M, uint32_t C, uint32_t* __restrict__ muts,
                                                         const uint32_t* __restrict__ status) {
    const uint32_t k = blockIdx.x * WAVE + threadIdx.x;
    if (k >= M) return;
    if (status && *status) {
        for (uint32_t c = 0; c < C; c++) {
            uint32_t* mu = muts + ((size_t)k * C + c) * 3;
            mu[0] = 0xffffffffu; mu[1] = 0; mu[2] = 0;
        }
        return;
    }
    // binary search for the op whose range holds k
    uint32_t lo = 0, hi = op_end - op_begin;       // first[lo] <= k < first[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (first[mid] <= k) lo = mid; else hi = mid;
    }
    const uint32_t op = op_begin + lo;
    const uint32_t r = k - first[lo];
    const uint32_t deg = tuples[tuple_ptr[op] + r / n_dev];
    const uint32_t off = r % n_dev;
    for (uint32_t c = 0; c < C; c++) {
        uint32_t* mu = muts + ((size_t)k * C + c) * 3;
        mu[0] = op; mu[1] = deg; mu[2] = off | (1u << 16);
    }
}

// The index of every op's first neighbour, built on the device (one wavefront): first[o - op_begin]
// for o = op_begin..op_end (the last entry is the total).  *status = 0 if every range of tuple_ptr is
// well formed (ascending, inside the list of n_tuples entries), the total fits 32 bits and equals the
// M the caller sized its buffers for; 1 otherwise.  Writes op_end - op_begin + 1 entries of first.
__global__ __launch_bounds__(WAVE) void k_neighbour_first(const uint32_t* __restrict__ tuple_ptr, uint32_t n_tuples, uint32_t op_begin,
                                                          uint32_t op_end, uint32_t n_dev, uint32_t M, uint32_t* __restrict__ first,
                                                          uint32_t* __restrict__ status) {
    const int lane = lane_id();
    u64 carry = 0;
    bool bad = false;
    for (uint32_t base = op_begin; base < op_end; base += WAVE) {
        const uint32_t o = base + lane;
        u64 n = 0;
        if (o < op_end) {
            const uint32_t a = tuple_ptr[o], b = tuple_ptr[o + 1];
            if (a > b || b > n_tuples) bad = true; else n = (u64)(b - a) * n_dev;
        }
        // inclusive prefix sum over the lanes
        u64 incl = n;
#pragma unroll
        for (int sft = 1; sft < WAVE; sft <<= 1) {
            const uint32_t lo = __shfl_up((uint32_t)incl, sft), hi = __shfl_up((uint32_t)(incl >> 32), sft);
            if (lane >= sft) incl += ((u64)hi << 32) | lo;
        }
        const u64 excl = carry + incl - n;
        if (o < op_end) {
            if (excl > 0xffffffffull) bad = true;
            first[o - op_begin] = (uint32_t)excl;
        }
        carry += readlane_u64(incl, WAVE - 1);
    }
    if (carry > 0xffffffffull || carry != M) bad = true;
    const bool any_bad = ballot(bad) != 0;
    if (lane == 0) {
        first[op_end - op_begin] = (uint32_t)carry;
        *status = any_bad ? 1u : 0u;
    }
}

// per chain: the smallest time among its M results ([M][C]) and the lowest index that has it;
// one wavefront per chain
__global__ __launch_bounds__(WAVE) void k_best_of(const u64* __restrict__ ns, uint32_t M, uint32_t C, u64* __restrict__ best_ns,
                                                  uint32_t* __restrict__ best_idx) {
    const uint32_t c = blockIdx.x;
    if (c >= C) return;
    u64 b = ~0ull;
    uint32_t bi = 0xffffffffu;
    for (uint32_t k = lane_id(); k < M; k += WAVE) {
        const u64 v = ns[(size_t)k * C + c];
        if (v < b) { b = v; bi = k; }        // ascending k: the first index wins inside a lane
    }
    const u64 m = wave_min_u64(b);
    const uint32_t mi = wave_min_u32(b == m ? bi : 0xffffffffu);
    if (lane_id() == 0) { best_ns[c] = m; best_idx[c] = mi; }
}

// the proposals of the steps done[c] .. done[c] + n_ahead - 1 of every chain, as mutation records
// [n_ahead][C] {op, cfg.x, cfg.y}; op = all ones where there is none (no list, or beyond the call's steps)
__global__ void k_search_ahead_proposals(SearchDev search, uint32_t n_ops, uint32_t n_dev, uint32_t C, uint32_t n_steps, uint32_t* muts) {
    const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= search.n_ahead * C) return;
    const uint32_t j = idx / C, c = idx % C;
    const uint32_t s = search.done[c] + j;
    uint32_t op = 0xffffffffu;
    uint2 cfg = make_uint2(0, 0);
    if (s < n_steps) {
        uint32_t o;
        if (search_proposal(search, n_ops, n_dev, c, search.first_step + s, o, cfg)) op = o;
    }
    muts[(size_t)idx * 3 + 0] = op;
    muts[(size_t)idx * 3 + 1] = cfg.x;
    muts[(size_t)idx * 3 + 2] = cfg.y;
}

// (a kernel and not a memset, so that a captured stream sees a kernel node)
__global__ void k_zero_words(uint32_t* p, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---- forced mutations in segments (chain_segment) ------------------------------------------
//
// The blocks of a new chain set: bookkeeping and tags of endTimes empty (clear_bytes from clear_at on, both multiples of 16), the strategies at the
// heads of the first C blocks (0: spare blocks, without one).  Workgroups: blocks x pieces of what is to be cleared, which is 1 MB of a block of the NMT-shaped
// graph, but with its extents beyond 16 bits all of it: 80 MB, 0.7 ms for a single workgroup.
constexpr uint32_t CLEAR_PIECES = 64;
inline uint32_t clear_pieces(size_t clear_bytes) { return (uint32_t)(clear_bytes >> 16 < CLEAR_PIECES ? (clear_bytes >> 16) + 1 : CLEAR_PIECES); }
__global__ __launch_bounds__(256) void k_chain_blocks(unsigned char* __restrict__ chain_mem, size_t chain_stride, size_t clear_at, size_t clear_bytes,
                                                      const uint2* __restrict__ strategies, uint32_t n_ops, uint32_t C, uint32_t* __restrict__ chain_flags) {
    unsigned char* block = chain_mem + (size_t)blockIdx.x * chain_stride;
    uint4* p = (uint4*)(block + clear_at);
    for (size_t i = blockIdx.y * 256 + threadIdx.x; i < clear_bytes / 16; i += (size_t)gridDim.y * 256) p[i] = make_uint4(0, 0, 0, 0);
    if (blockIdx.y) return;
    if (blockIdx.x < C)
        for (uint32_t i = threadIdx.x; i < n_ops; i += 256) ((uint2*)block)[i] = strategies[(size_t)blockIdx.x * n_ops + i];
    if (threadIdx.x == 0) chain_flags[blockIdx.x] = 0;
}

// How many segments the steps of a chain are cut into: the number with which the longest one is estimated to take least, 1 (steps in turn) where cutting gives
// nothing.  A step takes what is left of the stored timeline from where the change can matter first (first_input_at; half of it without a timeline), the
// first one of a segment all of it, and every step per_step besides.  With more than SPLIT_STEPS steps that many of them stand for all.  left: what each
// of the m steps takes; called by one wavefront, a lane per number.  (Where per_step alone decides, the host says so and nothing is estimated.)
constexpr uint32_t SPLIT_STEPS = 128;
__device__ __forceinline__ uint32_t choose_segments(const uint32_t* left, uint32_t m, uint32_t n_steps, uint32_t most, uint32_t first, uint32_t per_step) {
    const uint32_t P = (uint32_t)lane_id() + 1;
    const float w = (float)n_steps / (float)m;
    float longest = 0.0f, sum = 0.0f;
    const uint32_t q = m / P, r = m - q * P;
    uint32_t err = 0, end = 0;                           // the next segment begins at floor(m * p / P)
    for (uint32_t i = 0; i < m; i++) {
        const float f = (float)left[i] + (float)per_step;
        if (i == end) {
            sum = P > 1 || i ? (float)WHOLE + (float)per_step + (w - 1.0f) * f : (float)first + (float)per_step + (w - 1.0f) * f;
            end += q;
            err += r;
            if (err >= P) { err -= P; end++; }
        } else {
            sum += w * f;
        }
        longest = sum > longest ? sum : longest;
    }
    // (below 2^25: compared as whole numbers, the smallest number of segments among equals)
    const float capped = longest < 33000000.0f ? longest : 33000000.0f;
    const uint32_t key = P <= most && P <= m ? ((uint32_t)capped << 6) | (P - 1) : 0xffffffffu;
    const uint32_t in_turn = readlane_u32(key, 0) >> 6, best = wave_min_u32(key);
    return (best >> 6) + WHOLE / 16 < in_turn ? (best & 63u) + 1 : 1u;
}

// Decides how many segments there are and writes into the block of each the strategy that its steps start from: the chain's with all mutations before them
// applied.  The stored timelines of the blocks belong to other strategies from then on.  One workgroup per chain; the mutations are applied in order by one lane.
// Cut by what the steps take rather than always, one chain, three changes: of the last 3 % of the ops of the NMT-shaped graph 69 -> 7.7 to 34 ms,
// of the ResNet-101-shaped one 8.9 -> 0.7 to 1.2; 800 chains x 3 on the Inception-v3-shaped one 7.1 -> 3.0, of any ops there 11 as before (in turn 12.7).
constexpr uint32_t SPLIT_THREADS = 256;       // (more only wait for one another at the barriers)
__global__ __launch_bounds__(SPLIT_THREADS) void k_chain_split(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ in_edges,
                                                     unsigned char* __restrict__ chain_mem, size_t chain_stride, uint32_t n_snaps,
                                                     uint32_t rowl, uint32_t C, uint32_t n_segs, const uint32_t* __restrict__ muts,
                                                     uint32_t n_steps, uint32_t* __restrict__ chain_flags, SpareBlocks spare, uint32_t per_step, bool cut) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint2* cfgs = (uint2*)lds_raw;                       // [n_ops]
    constexpr uint32_t FEW = 256;
    __shared__ uint32_t mu[FEW * 3];
    __shared__ uint32_t left[SPLIT_STEPS];
    __shared__ uint32_t poisoned, chosen;
    const uint32_t c = blockIdx.x, t = threadIdx.x, wave = first_u32(t / WAVE);
    const ChainMem own = carve_chain(chain_mem + (size_t)c * chain_stride, S, n_snaps, rowl);
    const ChainMeta meta = *own.meta;
    for (uint32_t i = t; i < S.n_ops; i += SPLIT_THREADS) cfgs[i] = own.cfgs[i];
    if (t == 0) poisoned = chain_flags[c];
    const uint32_t m = cut ? 0 : (n_steps < SPLIT_STEPS ? n_steps : SPLIT_STEPS);
    for (uint32_t i = wave; i < m; i += SPLIT_THREADS / WAVE) {
        const uint32_t op = first_u32(muts[((u64)n_steps * i / m * C + c) * 3]);
        uint32_t share = WHOLE;
        if (op >= S.n_ops) share = 0;                    // (neither it nor anything behind it is simulated)
        else if (!S.ties) share = meta.stale ? WHOLE / 2 : share_from(meta, first_input_at(ops, in_edges, own, rowl ? rowl : (uint32_t)WAVE, op));
        if (lane_id() == 0) left[i] = share;
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t n = poisoned ? 1u : cut ? n_segs : choose_segments(left, m, n_steps, n_segs, meta.stale || meta.n_valid < 2 ? WHOLE : left[0], per_step);
        if (t == 0) { chosen = n; spare.segs[c] = n; }
    }
    __syncthreads();
    const uint32_t n_mine = chosen;
    if (n_mine < 2) return;
    for (uint32_t p = 0; p < n_mine; p++) {
        const ChainSeg seg = chain_segment(p * C + c, C, n_mine, n_steps, chain_mem, chain_stride, chain_flags, spare);
        const ChainMem cm = carve_chain(seg.block, S, n_snaps, rowl);
        for (uint32_t i = t; i < S.n_ops; i += SPLIT_THREADS) cm.cfgs[i] = cfgs[i];
        if (t == 0) {
            cm.meta->step = meta.step;
            cm.meta->n_valid = 0;
            cm.meta->stale = 1;
            cm.meta->cur_ns = RESULT_INVALID;
            *seg.flag = poisoned;
        }
        for (uint32_t s = seg.s_begin; s < seg.s_end; s += FEW) {
            const uint32_t n = seg.s_end - s < FEW ? seg.s_end - s : FEW;
            __syncthreads();
            if (t < n)
                for (uint32_t k = 0; k < 3; k++) mu[t * 3 + k] = muts[((size_t)(s + t) * C + c) * 3 + k];
            __syncthreads();
            if (t == 0) {
                for (uint32_t k = 0; k < n && !poisoned; k++) {
                    if (mu[k * 3] >= S.n_ops) poisoned = 1;
                    else cfgs[mu[k * 3]] = make_uint2(mu[k * 3 + 1], mu[k * 3 + 2]);
                }
            }
        }
        __syncthreads();
    }
}

// ---- trials, longest first ------------------------------------------------------------------
//
// How long a trial takes follows from where it may resume: from nothing (the last snapshot) to a full simulation.  A launch lasts as long as its
// fullest SIMD, so where a SIMD gets several trials they are dealt out by length (trial_first_place).  Two small kernels: a wavefront per trial
// finds the class (the snapshot before the first endTime of the changed op's producers; parts without inputs are not looked for, the class is
// only an estimate) and its place in it, then every trial goes to its place in the list.
// Against trials drawn as they come, both kernels included: 4096 on the NMT-shaped graph 93.8 -> 66.1 ms (the longest one alone takes about 60),
// 8192 141 -> 97.5, 16384 234 -> 170; 1200 / 4096 / 20000 on the Inception-v3-shaped one 4.07 -> 3.70, 5.71 -> 3.82, 16.7 -> 13.0; 1200 / 4096 /
// 20000 on the AlexNet-shaped one 0.135 -> 0.123, 0.202 -> 0.130, 0.509 -> 0.478.
constexpr uint32_t TRIAL_CLASSES = 32;           // one per snapshot
constexpr uint32_t MAX_PLANNED_TRIALS = 1u << 26;
constexpr uint32_t TRIALS_PER_BLOCK = 16;        // (places are counted per workgroup first: one global atomic per class and workgroup)
__global__ __launch_bounds__(TRIALS_PER_BLOCK * WAVE) void k_trial_class(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ in_edges,
                                                     const unsigned char* __restrict__ chain_mem, size_t chain_stride, uint32_t n_snaps,
                                                     uint32_t rowl, uint32_t C, const uint32_t* __restrict__ muts, uint32_t total,
                                                     const uint32_t* __restrict__ chain_flags, uint32_t* __restrict__ counts,
                                                     uint32_t* __restrict__ key) {
    __shared__ uint32_t here[TRIAL_CLASSES], begin[TRIAL_CLASSES];
    if (threadIdx.x < TRIAL_CLASSES) here[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t id_raw = blockIdx.x * TRIALS_PER_BLOCK + first_u32(threadIdx.x / WAVE);
    const bool live = id_raw < total;
    const uint32_t id = live ? id_raw : total - 1;
    const uint32_t c = id % C;
    const ChainMem cm = carve_chain(const_cast<unsigned char*>(chain_mem) + (size_t)c * chain_stride, S, n_snaps, rowl);
    const uint32_t row = rowl ? rowl : (uint32_t)WAVE;
    const uint32_t op = muts[(size_t)id * 3];
    uint32_t k = TRIAL_CLASSES - 1;              // trials that are not simulated come last
    if (op < S.n_ops && chain_flags[c] == 0) {
        const ChainMeta meta = *cm.meta;
        k = 0;
        if (!meta.stale && meta.n_valid > 1 && meta.step != 0 && !S.ties) {
            const u64 at = (2 * first_input_at(ops, in_edges, cm, row, op)) / meta.step;
            const uint32_t last = meta.n_valid - 1 < TRIAL_CLASSES - 1 ? meta.n_valid - 1 : TRIAL_CLASSES - 1;
            k = at < last ? (uint32_t)at : last;
        }
    }
    uint32_t place = 0;
    if (live && lane_id() == 0) place = atomicAdd(&here[k], 1u);
    __syncthreads();
    if (threadIdx.x < TRIAL_CLASSES && here[threadIdx.x]) begin[threadIdx.x] = atomicAdd(&counts[threadIdx.x], here[threadIdx.x]);
    __syncthreads();
    if (live && lane_id() == 0) key[id] = k | ((begin[k] + place) << 5);
}
__global__ __launch_bounds__(256) void k_trial_place(const uint32_t* __restrict__ counts, const uint32_t* __restrict__ key, uint32_t total,
                                                     uint32_t* __restrict__ order) {
    const uint32_t id = blockIdx.x * 256 + threadIdx.x;
    if (id >= total) return;
    const uint32_t k = key[id] & (TRIAL_CLASSES - 1);
    uint32_t at = key[id] >> 5;
    for (uint32_t j = 0; j < k; j++) at += counts[j];
    order[at] = id;
}

}  // namespace ffsim

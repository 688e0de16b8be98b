// The search loop (Section 6) with the simulations of coming steps made side by side: what ff_sim_search launches where the device has room for
// several simulations per chain.
//
// The proposal of a step follows from the random draws alone, so the strategies that a chain may have to price in the next steps are known up to
// which of the proposals before them are taken.  They form a binary tree: a node is the proposal of one step, made to the chain's strategy with
// some of the proposals above it taken; its children are the proposals of the next step after it was taken or not.  A round prices a part of that
// tree (k_loop_nodes: one full simulation per node and wavefront) and then every chain walks down from the root, with the decisions of Section 6.1
// and the draws of its own steps, until it leaves the part (k_search_walk), which is where its next tree begins.  Traces, best strategies
// and final strategies are those of steps made one after the other.
//
// Which nodes: the likeliest ones, with the share of proposals a chain has taken lately as the chance of every decision.  With W nodes a chain
// advances by log2(W + 1) steps where that share is a half and by more the further it is from it.  Chains that have finished leave their nodes
// to the others.
//
// Passes with the chains created and closed, in turn -> ahead: 64 chains x 256 steps on the AlexNet-shaped graph with parameter traffic (the search
// driver's default) 47.0 -> 19.3 ms, 30 x 60 11.9 -> 4.5; Inception-v3-shaped 1 x 16 35.8 -> 18.7, 100 x 30 88.9 -> 47.7, 1024 x 64 201 -> 171;
// ResNet-101-shaped 10 x 20 111 -> 48.8, 300 x 16 116 -> 83.6; NMT-shaped (20 steps) 3 x 12 286 -> 157; tiny chain 1 x 16 0.76 -> 0.49.  What bounds
// it is the slowest simulation of a round: every round waits for it.
#pragma once
#include "ffsim_chain.h"

namespace ffsim {

// parent: the node above in the chain's tree (NO_NODE: root), via: 1 if this node supposes that it was taken; child: numbers within the
// chain's tree of the nodes after this one was taken (low half) and not (high half), 0xffff where there is none
struct AheadNode { uint32_t parent, via, step, op, x, y, child; };
constexpr uint32_t NO_NODE = 0xffffffffu;
constexpr uint32_t MAX_TREE = 63;            // nodes of a chain in one round: a lane per node and one more for what may come next
constexpr uint32_t AHEAD_RING = 4;           // rounds whose counters are kept

struct AheadDev {
    AheadNode* nodes;        // [C][MAX_TREE]: a chain's tree is its own, since the chains walk side by side and some lay out their next tree while others still read theirs
    u64* ns;                 // [capacity] simulated time of every node
    uint2* strategies;       // [capacity][n_ops]
    uint32_t* counters;      // [AHEAD_RING][2]: chains with a tree, slots given out; then what k_search_plan finds: chains that go on, the
                             // most that a chain's steps take in turn (1024ths of a simulation), the most proposals
    uint32_t* tree;          // [C][2]: first slot, nodes
    uint32_t* done;          // [C] steps of the call a chain has finished
    uint32_t capacity;
    float per_round;         // steps that a round takes a chain further where the share of accepted proposals is middling
    float per_step;          // what a step in turn takes besides its simulation, in 1024ths of one
};

constexpr uint32_t AHEAD_PLAN = AHEAD_RING * 2, AHEAD_WORDS = AHEAD_PLAN + 4;

// a chain whose strategy is valid and whose patience has not run out
__device__ __forceinline__ bool search_goes_on(const SearchDev& search, const ChainMeta& meta, uint32_t flag) {
    return flag == 0 && meta.stale == 0 && !(search.patience && meta.idle_steps >= search.patience);
}

// Is it worth looking ahead?  Counts the chains that still propose, and estimates what the call's steps take in turn (share_from, for the proposals of the
// first steps) and as a tree (rounds of full simulations and one that is recorded), both for the chain with the most to do.  Without a
// chain that proposes there will be no tree, so that no timeline has to be recorded again for its sake: 32 steps of 64 such chains on the
// ResNet-101-shaped graph 9.9 -> 0.17 ms.  Proposals of late ops (the others have no list) resume late in the timeline, and their steps are made in turn where that
// is less: 16 steps of one chain on the NMT-shaped graph (20 steps unrolled) with lists for the last 3 % of the ops 33 to 60 -> 0.5 to 2.5 ms.  (Graphs simulated in
// LDS take about a sixth of a simulation per step besides: 64 steps of one chain on the AlexNet-shaped graph, lists for its last three ops, 1.1 ms in turn,
// 0.6 as a tree.)
constexpr uint32_t PLAN_STEPS = 64, PLAN_WAVES = 16;
__device__ __forceinline__ bool worth_looking_ahead(const AheadDev& ah, uint32_t n_steps) {
    const uint32_t* plan = ah.counters + AHEAD_PLAN;
    const float scale = n_steps > PLAN_STEPS ? (float)n_steps / PLAN_STEPS : 1.0f;
    const float rounds = scale * (float)first_u32(plan[2]) / ah.per_round;
    return scale * (float)first_u32(plan[1]) + ah.per_step * (float)n_steps > (float)WHOLE * ((rounds > 1.0f ? rounds : 1.0f) + 1.0f);
}
__global__ __launch_bounds__(PLAN_WAVES * WAVE) void k_search_plan(SimDev S, const DOp* __restrict__ ops, const DEdge* __restrict__ in_edges,
                                                                   unsigned char* __restrict__ chain_mem, size_t chain_stride, uint32_t n_snaps, uint32_t rowl,
                                                                   uint32_t n_steps, const uint32_t* __restrict__ chain_flags, SearchDev search,
                                                                   uint32_t* __restrict__ plan) {
    __shared__ uint32_t share, proposals;
    const uint32_t c = blockIdx.x;
    const ChainMem cm = carve_chain(chain_mem + (size_t)c * chain_stride, S, n_snaps, rowl);
    const ChainMeta meta = *cm.meta;
    if (!search_goes_on(search, meta, chain_flags[c])) return;
    if (threadIdx.x == 0) { share = 0; proposals = 0; }
    __syncthreads();
    for (uint32_t s = first_u32(threadIdx.x / WAVE); s < (n_steps < PLAN_STEPS ? n_steps : PLAN_STEPS); s += PLAN_WAVES) {
        uint32_t op;
        uint2 cfg;
        if (!search_proposal(search, S.n_ops, S.n_dev, c, search.first_step + s, op, cfg)) continue;   // (no list)
        op = first_u32(op);
        const uint32_t left = S.ties ? WHOLE : share_from(meta, first_input_at(ops, in_edges, cm, rowl, op));
        if (lane_id() == 0) { atomicAdd(&share, left); atomicAdd(&proposals, 1u); }
    }
    __syncthreads();
    if (threadIdx.x == 0) { atomicAdd(&plan[0], 1u); atomicMax(&plan[1], share); atomicMax(&plan[2], proposals); }
}

// One wavefront per chain: the decisions that the round before allows, then the chain's next tree.
__global__ __launch_bounds__(WAVE) void k_search_walk(SimDev S, unsigned char* __restrict__ chain_mem, size_t chain_stride, uint32_t n_snaps, uint32_t rowl,
                                                      uint32_t C, uint32_t n_steps, u64* __restrict__ out_ns, const uint32_t* __restrict__ chain_flags,
                                                      SearchDev search, AheadDev ah, uint32_t slots_in_blocks, uint32_t round) {
    __shared__ AheadNode tree[WAVE];
    const uint32_t c = blockIdx.x, lane = lane_id();
    if (c == 0 && lane < 2) ah.counters[((round + 2) % AHEAD_RING) * 2 + lane] = 0;
    const bool any = first_u32(ah.counters[AHEAD_PLAN]) != 0;
    if (any && !worth_looking_ahead(ah, n_steps)) {
        // (all steps are left to the launch behind the rounds)
        if (lane == 0 && round == 0) ah.done[c] = 0;
        return;
    }
    uint32_t pos = round ? first_u32(ah.done[c]) : 0u;
    if (pos >= n_steps) return;
    // (with slots in the chains' blocks every stored timeline is lost, whether its chain moves or not -- if there is to be any tree at all)
    const ChainMem cm = carve_chain(chain_mem + (size_t)c * chain_stride, S, n_snaps, rowl);
    ChainMeta meta = *cm.meta;
    const bool poisoned = first_u32(chain_flags[c]) != 0;
    u64 best = first_u64(search.best_ns[c]), cur = first_u64(meta.cur_ns), idle = first_u64(meta.idle_steps);
    AheadNode* mine = ah.nodes + (size_t)c * MAX_TREE;
    auto keep_best = [&]() {
        best = cur;
        __threadfence_block();
        wave_sync();
        for (uint32_t i = lane; i < S.n_ops; i += WAVE) search.best_cfgs[(size_t)c * S.n_ops + i] = cm.cfgs[i];
    };
    auto step_done = [&](u64 ns) { if (lane == 0) out_ns[(size_t)pos * C + c] = ns; pos++; idle++; };
    const bool live = !poisoned && first_u32(meta.stale) == 0;
    if (round == 0 && live) {
        if (cur < best) keep_best();       // the strategy the search starts from counts as seen
        if (slots_in_blocks && any) meta.moved = 1;
    }
    if (round) {
        const uint32_t base = first_u32(ah.tree[2 * c]), count = first_u32(ah.tree[2 * c + 1]);
        for (uint32_t k = 0; k < count;) {
            const AheadNode node = mine[k];
            const uint32_t at = first_u32(node.step);
            while (pos < at) step_done(cur);                  // steps without a proposal
            if (search.patience && idle >= search.patience) break;
            const u64 mk = first_u64(ah.ns[base + k]);
            const bool taken = search_accepts(search, c, search.first_step + pos, mk, cur);
            meta.n_steps++;
            meta.n_tried++;
            if (taken) {
                meta.n_taken++;
                meta.moved = 1;
                if (lane == 0) cm.cfgs[node.op] = make_uint2(node.x, node.y);
                cur = mk;
            }
            step_done(cur);
            if (cur < best) { keep_best(); idle = 0; }
            k = first_u32(taken ? node.child & 0xffffu : node.child >> 16);
        }
        __threadfence_block();
        wave_sync();
    }
    // the proposals of the next 64 steps, a lane each
    const bool proposes = live && !(search.patience && idle >= search.patience);
    uint32_t op = 0;
    uint2 cfg = make_uint2(0, 0);
    const bool has = proposes && pos + lane < n_steps && search_proposal(search, S.n_ops, S.n_dev, c, search.first_step + pos + lane, op, cfg);
    const u64 has_m = ballot(has);
    uint32_t n = 0;
    if (!has_m) {
        // none to come (or none among the next 64, which are passed here; the rest is left to the next round)
        const uint32_t end = proposes && n_steps - pos > WAVE ? pos + WAVE : n_steps;
        while (pos < end) step_done(poisoned ? RESULT_INVALID : cur);
    } else {
        const uint32_t chains = round ? first_u32(ah.counters[((round - 1) % AHEAD_RING) * 2]) : C;
        uint32_t quota = ah.capacity / (chains ? chains : 1u);
        quota = quota > MAX_TREE ? MAX_TREE : quota;
        if (meta.n_tried > 64) { meta.n_tried /= 2; meta.n_taken /= 2; }
        const float p = ((float)meta.n_taken + 1.0f) / ((float)meta.n_tried + 2.0f);
        // What may come next, a lane per candidate: its chance (as bits: numbers that are not negative compare alike), the node above it and
        // whether that was taken, its step.
        uint32_t chance = lane == 0 ? __float_as_uint(1.0f) : 0u, up = NO_NODE, via = 0, t = (uint32_t)__builtin_ctzll(has_m);
        for (; n < quota; n++) {
            const uint32_t top = ~wave_min_u32(~chance);
            if (!top) break;
            const int l = __builtin_ctzll(ballot(chance == top));
            const uint32_t n_up = readlane_u32(up, l), n_via = readlane_u32(via, l), n_t = readlane_u32(t, l);
            const AheadNode node{n_up, n_via, pos + n_t, readlane_u32(op, n_t), readlane_u32(cfg.x, n_t), readlane_u32(cfg.y, n_t), NO_NODE};
            if (lane == 0) {
                tree[n] = node;
                if (n_up != NO_NODE) tree[n_up].child = n_via ? (tree[n_up].child & 0xffff0000u) | n : (tree[n_up].child & 0xffffu) | (n << 16);
            }
            // the proposal after it: not taken (in its own lane) and taken (in the next free one)
            const u64 later = n_t < WAVE - 1 ? has_m & ~((2ull << n_t) - 1) : 0ull;
            const uint32_t next = later ? (uint32_t)__builtin_ctzll(later) : 0u;
            const float here = __uint_as_float(top);
            if ((int)lane == l) { chance = later ? __float_as_uint(here * (1.0f - p)) : 0u; up = n; via = 0; t = next; }
            if (lane == n + 1) { chance = later ? __float_as_uint(here * p) : 0u; up = n; via = 1; t = next; }
        }
        wave_sync();
        uint32_t base = 0;
        // (a slot per node and no more: whatever a slot holds is simulated, and the round lasts as long.  What the quotas add up to does not exceed
        // the capacity: no more chains have a tree than in the round before)
        if (lane == 0) base = atomicAdd(&ah.counters[(round % AHEAD_RING) * 2 + 1], n);
        base = first_u32(base);
        if (lane < n) mine[lane] = tree[lane];
        if (lane == 0) ah.tree[2 * c] = base;
        // the strategies of the nodes: the chain's, then the proposals on the way down from the root
        for (uint32_t i = lane; i < S.n_ops; i += WAVE) {
            const uint2 v = cm.cfgs[i];
            for (uint32_t k = 0; k < n; k++) ah.strategies[(size_t)(base + k) * S.n_ops + i] = v;
        }
        __threadfence_block();
        wave_sync();
        if (lane < n) {
            uint2* strategy = ah.strategies + (size_t)(base + lane) * S.n_ops;
            u64 made = 1ull << lane;
            for (uint32_t k = lane; tree[k].parent != NO_NODE; k = tree[k].parent)
                if (tree[k].via) made |= 1ull << tree[k].parent;
            // (a node comes after the one above it: in ascending order, so that the last proposal for an op holds)
            for (; made; made &= made - 1) {
                const AheadNode& node = tree[__builtin_ctzll(made)];
                strategy[node.op] = make_uint2(node.x, node.y);
            }
        }
    }
    // (the timeline of a chain that has moved is recorded anew behind the last round: with snapshots as far apart as chain_steps wants them for the
    // time the chain has now, or the run would drop them again)
    if (meta.moved) {
        const u64 ideal = (2 * cur) / n_snaps + 1;
        if (ideal * 2 < meta.step || ideal > meta.step * 2) meta.step = ideal;
    }
    if (lane == 0) {
        ah.tree[2 * c + 1] = n;
        ah.done[c] = pos;
        if (pos < n_steps) atomicAdd(&ah.counters[(round % AHEAD_RING) * 2], 1u);
        meta.cur_ns = cur;
        meta.idle_steps = idle;
        *cm.meta = meta;
        search.best_ns[c] = best;
    }
}

}  // namespace ffsim

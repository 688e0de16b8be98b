// The event loop (Algorithm 1) on kept set-up (ffsim_kept.h).
#pragma once
#include "ffsim_events.h"
#include "ffsim_kept.h"
#include <type_traits>

namespace ffsim {

// ---- queue of pending events -------------------------------------------------------------
//
// Only ops with a pending event matter to the queue, and there are few of them at any time: 2 to 10 on the
// convolutional graphs, about 100 in the first moments of the unrolled recurrent graph and 7 after that.  So the queue is one
// register, a lane per op with an event:
//   Q_OP16 / Q_OP   graphs of at most 16 / 64 ops: lane = op;
//   Q_SLOT          any graph: lane = slot, a second register holds the slot's op; when all 64 slots are taken, the op
//                   with the latest first event moves to a spill list in memory and comes back when its turn does.
// There are two keys per op, of its first task to dequeue and of its first one to release (see run_loop for why they are kept apart).
// A key is the event's word (2 * time + kind) relative to 2 * E, in 32 bits.  E, the epoch, follows the simulated time
// in steps of about a second (advance_epoch); KEY_FAR stands for an event at a distance that does not fit (its word in
// memory has it in full), KEY_NONE for no event.
enum LoopQueue : int { Q_OP16 = 0, Q_OP = 1, Q_SLOT = 2 };
constexpr uint32_t KEY_NONE = 0xffffffffu, KEY_FAR = 0xfffffffeu;
constexpr uint32_t KEY_REFRESH = 0x80000000u;    // a smallest key from here on: no event left, or time to move the epoch
constexpr uint32_t NO_OP = 0xffffffffu;
constexpr u64 RESULT_RETRY = 2;                  // a link row is booked beyond 32 bits: simulate again with 64-bit rows
constexpr uint32_t RUN_SPAN = 0x40000000u;       // events of one step lie at most this far apart
constexpr uint32_t FAR_AWAY = 0xfffffffeu;       // a distance between events of one kind that 32 bits do not hold
constexpr int32_t LOST = INT32_MIN;              // steps left (see run_loop) once the queue is found to have lost an event
// Ops with more out-edges release at one time only: the set-up looks at the exeTimes behind all of them, and few have more.  Against 8, one edge takes
// 1.17 times as long on 1024 training iterations (Inception-v3-shaped; its batch of 4096 1.08), two 1.04 (1.06), four 1.01 (1.00), 16 and 64 the same within 2 %.
constexpr uint32_t RUN_EDGES = 8;

struct Queue {
    uint32_t kd, kr, op;        // per lane: keys of the first task to be dequeued and of the first to release, the op they are of
    uint32_t ex;                // per lane: 2 * exeTime of that op (at most RUN_SPAN): none of the tasks still to be dequeued releases before kd + ex
    uint32_t n_spill;           // uniform
    u64 spill_min;              // smallest word on the spill list (absolute; W_NONE if it is empty)
};

// per-candidate state of the loop that outlives a call of run_loop
struct LoopState {
    Queue q;
    u64 E;                      // epoch (ns)
};

// memory of one candidate (see slot_layout)
struct LoopMem {
    u64* words;                 // [n_ops][ROWL]
    uint4* hdr;                 // [n_ops_pad]
    uint32_t* rows;             // [n_edges][KEPT_ROWS][ROWL]
    uint32_t* priv;             // trial mutations: the rows of the mutated op's in-edges, then of its out-edges
    u64* spill_key;             // [n_ops_pad]
    uint32_t* spill_op;         // [n_ops_pad]
    u64* crow;                  // LDS [n_dev]: endTime of the last task of every compute device
    uint32_t* lrow;             // LDS [n_links]: endTime of the last transfer of every link row, relative to E
    u64* lrow64;                // the same memory as absolute times (the form with 64-bit link rows; null where there is none)
    uint8_t* tag;               // LDS [n_rows]: see fifo_commit
    const uint4* links;         // {m, k, lat1, 0} per ordered pair of local GPUs, then per ordered pair of nodes; or null
    const OpLite* op_lite;      // static records (ffsim_kept.h)
    const EdgeLite* edge_lite;
};

// minimum over the parts of a row of ROWL lanes (lanes beyond them hold the identity)
template <int ROWL>
__device__ __forceinline__ uint32_t part_min_u32(uint32_t v) { return ROWL == 16 ? row0_min_u32(v) : wave_min_u32(v); }

// the minimum of v over the lanes of a mask that is often a single lane
template <int ROWL>
__device__ __forceinline__ uint32_t part_min_of(uint32_t v, u64 mask) {
    if ((mask & (mask - 1)) == 0) return readlane_u32(v, __builtin_ctzll(mask));
    return part_min_u32<ROWL>(lanes_of(mask) ? v : KEY_NONE);
}

// smallest pending event of an op, from its words in memory (W_NONE: none); of one kind (1: dequeue, 0: release) if that is asked for
template <int ROWL>
__device__ __forceinline__ u64 op_min_word(const u64* words, uint32_t op, int kind = -1) {
    u64 w = load_word<ROWL>(words, op);
    if (kind >= 0 && (int)(w & 1) != kind) w = W_NONE;
    const u64 m = wave_min_u64(w);
    return m >> 63 ? W_NONE : m;
}
// the bound that an op's exeTime sets, as a difference of keys
__device__ __forceinline__ uint32_t exe_span(uint32_t exe) { return exe >= RUN_SPAN / 2 ? RUN_SPAN : 2 * exe; }
__device__ __forceinline__ uint32_t rel_key(u64 word, u64 E) {
    const u64 d = word - 2 * E;
    return d >= KEY_FAR ? KEY_FAR : (uint32_t)d;
}
__device__ __forceinline__ uint32_t rel_key_or_none(u64 word, u64 E) { return word >> 63 ? KEY_NONE : rel_key(word, E); }

template <int Q>
__device__ __forceinline__ void queue_clear(const LoopMem& mem, Queue& q, uint32_t n_ops) {
    q.kd = KEY_NONE; q.kr = KEY_NONE; q.op = NO_OP; q.n_spill = 0; q.spill_min = W_NONE;
    q.ex = Q != Q_SLOT && (uint32_t)lane_id() < n_ops ? exe_span(mem.hdr[lane_id()].x) : 0u;
}
// the key of an op's event at distance d behind the popped one (FAR_AWAY, or KEY_NONE: none)
__device__ __forceinline__ uint32_t next_key(uint32_t kmin, uint32_t d) {
    uint32_t k = __builtin_elementwise_add_sat(kmin, d);
    k = k < KEY_FAR ? k : KEY_FAR;
    return k > d ? k : d;
}
// first event of a slot, of either kind
__device__ __forceinline__ uint32_t slot_key(const Queue& q) { return q.kd < q.kr ? q.kd : q.kr; }

__device__ __forceinline__ void spill_push(const LoopMem& mem, Queue& q, uint32_t op, u64 word) {
    if (lane_id() == 0) { mem.spill_key[q.n_spill] = word; mem.spill_op[q.n_spill] = op; }
    q.n_spill++;
    q.spill_min = word < q.spill_min ? word : q.spill_min;
    wave_sync();
}
// recomputes the minimum of the spill list
__device__ __forceinline__ void spill_scan(const LoopMem& mem, Queue& q) {
    u64 v = W_NONE;
    for (uint32_t t = lane_id(); t < q.n_spill; t += WAVE) { const u64 w = mem.spill_key[t]; v = w < v ? w : v; }
    q.spill_min = wave_min_u64(v);
}
// takes entry t off the spill list
__device__ __forceinline__ void spill_remove(const LoopMem& mem, Queue& q, uint32_t t) {
    q.n_spill--;
    if (lane_id() == 0) { mem.spill_key[t] = mem.spill_key[q.n_spill]; mem.spill_op[t] = mem.spill_op[q.n_spill]; }
    wave_sync();
    spill_scan(mem, q);
}

// All slots are taken and op j, which has none, gets an event: the op with the latest of the 65 first events goes to the spill list.
template <int ROWL>
__device__ __forceinline__ void queue_spill(const LoopMem& mem, LoopState& st, uint32_t j, uint32_t kd, uint32_t kr, uint32_t ex) {
    Queue& q = st.q;
    const uint32_t key = kd < kr ? kd : kr, sk = slot_key(q);
    const uint32_t kmax = ~wave_min_u32(~sk);
    // (a far event has its true word in memory; so has any other: the word is read back rather than rebuilt)
    if (key >= kmax) {
        spill_push(mem, q, j, key >= KEY_FAR ? op_min_word<ROWL>(mem.words, j) : 2 * st.E + key);
        return;
    }
    const uint32_t slot = __builtin_ctzll(ballot(sk == kmax));
    const uint32_t old = readlane_u32(q.op, slot);
    spill_push(mem, q, old, kmax >= KEY_FAR ? op_min_word<ROWL>(mem.words, old) : 2 * st.E + kmax);
    if ((uint32_t)lane_id() == slot) { q.kd = kd; q.kr = kr; q.op = j; q.ex = ex; }
}

// gives op j the events kd (a task to dequeue) and kr (one to release), KEY_NONE for none, where they are earlier than what it has (it may end
// up on the spill list: only with n_spill > 0).
template <int Q, int ROWL>
__device__ __forceinline__ void queue_insert(const LoopMem& mem, LoopState& st, uint32_t j, uint32_t kd, uint32_t kr, uint32_t ex) {
    Queue& q = st.q;
    if (Q != Q_SLOT) {
        const bool me = (uint32_t)lane_id() == j;
        const uint32_t d = me ? kd : KEY_NONE, r = me ? kr : KEY_NONE;
        q.kd = d < q.kd ? d : q.kd;
        q.kr = r < q.kr ? r : q.kr;
        return;
    }
    // on the spill list already?
    auto spilled = [&]() __attribute__((always_inline)) {
        const uint32_t key = kd < kr ? kd : kr;
        for (uint32_t b = 0; b < q.n_spill; b += WAVE) {
            const uint32_t t = b + lane_id();
            const u64 hit = ballot(t < q.n_spill && mem.spill_op[t < q.n_spill ? t : 0] == j);
            if (hit) {
                const uint32_t at_t = b + __builtin_ctzll(hit);
                const u64 word = key >= KEY_FAR ? op_min_word<ROWL>(mem.words, j) : 2 * st.E + key;
                if (lane_id() == 0 && word < mem.spill_key[at_t]) mem.spill_key[at_t] = word;
                wave_sync();
                spill_scan(mem, q);
                return true;
            }
        }
        return false;
    };
    // its slot, else the first free one
    u64 at = ballot(q.op == j);
    const u64 open = ballot(q.op == NO_OP);
    if (__builtin_expect(at == 0 && (q.n_spill != 0 || open == 0), 0)) {
        if (spilled()) return;
        if (!open) { queue_spill<ROWL>(mem, st, j, kd, kr, ex); return; }
    }
    at = at ? at : open & (0 - open);
    const bool me = lanes_of(at);
    const uint32_t d = me ? kd : KEY_NONE, r = me ? kr : KEY_NONE;
    q.kd = d < q.kd ? d : q.kd;
    q.kr = r < q.kr ? r : q.kr;
    q.op = me ? j : q.op;
    q.ex = me ? ex : q.ex;
}

// The smallest event on the spill list is not later than the smallest one in the slots: its op changes places with the
// one with the latest first event there (or takes a free slot).
template <int ROWL>
__device__ __forceinline__ void queue_unspill(const LoopMem& mem, LoopState& st) {
    Queue& q = st.q;
    // the entry with the smallest word, the lowest op among equal ones
    u64 best = W_NONE;
    uint32_t bop = NO_OP, bt = 0;
    for (uint32_t t = lane_id(); t < q.n_spill; t += WAVE) {
        const u64 w = mem.spill_key[t];
        const uint32_t o = mem.spill_op[t];
        if (w < best || (w == best && o < bop)) { best = w; bop = o; bt = t; }
    }
    const u64 m = wave_min_u64(best);
    const uint32_t mop = wave_min_u32(best == m ? bop : NO_OP);
    const uint32_t t = readlane_u32(bt, __builtin_ctzll(ballot(best == m && bop == mop)));
    spill_remove(mem, q, t);
    const uint32_t kd = rel_key_or_none(op_min_word<ROWL>(mem.words, mop, 1), st.E), kr = rel_key_or_none(op_min_word<ROWL>(mem.words, mop, 0), st.E);
    const uint32_t ex = exe_span(mem.hdr[mop].x);
    u64 at = ballot(q.op == NO_OP);
    uint32_t slot;
    if (at) {
        slot = __builtin_ctzll(at);
    } else {
        // the latest slot makes room (never a loop: the entry just taken off is not later than any slot that would
        // bring it back; among equal keys the highest op leaves)
        const uint32_t sk = slot_key(q);
        const uint32_t kmax = ~wave_min_u32(~sk);
        const uint32_t omax = ~wave_min_u32(sk == kmax ? ~q.op : NO_OP);
        slot = __builtin_ctzll(ballot(sk == kmax && q.op == omax));
        spill_push(mem, q, omax, kmax >= KEY_FAR ? op_min_word<ROWL>(mem.words, omax) : 2 * st.E + kmax);
    }
    if ((uint32_t)lane_id() == slot) { q.kd = kd; q.kr = kr; q.op = mop; q.ex = ex; }
}

// Moves the epoch to the next pending event.  Returns false if there is none.
// (What a link row holds below the epoch no longer matters: nothing becomes ready before it.  So the epoch never moves back; an event
// before it would be one that the queue has lost, keeps the key KEY_FAR and ends the run as an internal error where it is popped.)
template <int Q, int ROWL, bool L64>
__device__ __forceinline__ bool advance_epoch(const LoopMem& mem, LoopState& st, uint32_t n_links) {
    Queue& q = st.q;
    u64 wd = q.kd >= KEY_FAR ? W_NONE : 2 * st.E + q.kd, wr = q.kr >= KEY_FAR ? W_NONE : 2 * st.E + q.kr;      // this lane's events in full
    u64 far = ballot(q.kd == KEY_FAR || q.kr == KEY_FAR);
    while (far) {
        const int l = __builtin_ctzll(far);
        far &= far - 1;
        const uint32_t op = Q == Q_SLOT ? readlane_u32(q.op, l) : (uint32_t)l;
        const u64 d = op_min_word<ROWL>(mem.words, op, 1), r = op_min_word<ROWL>(mem.words, op, 0);
        if (lane_id() == l) { wd = d; wr = r; }
    }
    u64 next = wave_min_u64(wd < wr ? wd : wr);
    if (Q == Q_SLOT) next = q.spill_min < next ? q.spill_min : next;
    if (next >> 63) return false;
    const u64 E = (next >> 1) > st.E ? next >> 1 : st.E;
    const u64 delta = E - st.E;
    st.E = E;
    q.kd = rel_key_or_none(wd, E);
    q.kr = rel_key_or_none(wr, E);
    if (!L64) {
        const uint32_t d32 = delta >> 32 ? 0xffffffffu : (uint32_t)delta;
        for (uint32_t r = lane_id(); r < n_links; r += WAVE) mem.lrow[r] = __builtin_elementwise_sub_sat(mem.lrow[r], d32);
        wave_sync();
    }
    return true;
}

// ---- state: start, snapshots, result -------------------------------------------------------

// endTime of device row or link row t (device rows first), absolute; a link row idle before the epoch reads as the epoch or less
template <bool L64>
__device__ __forceinline__ u64 row_time(const LoopMem& mem, const LoopState& st, uint32_t t, uint32_t n_dev) {
    return t < n_dev ? mem.crow[t] : (L64 ? mem.lrow64[t - n_dev] : st.E + mem.lrow[t - n_dev]);
}

// Writes the next snapshot: the task words, and endTimes of all device and link rows (absolute).  The queue is not
// stored: it follows from the words.  next_ns: time of the first pending event.  Returns true if the comparison is on and the
// state equals the accepted timeline's snapshot of the same index for everything that can still matter: all words, and
// the rows, where rows that are idle when the first event comes count as equal (with equal words it is the same event).
template <int ROWL, bool L64, class SimX>
__device__ __forceinline__ bool save_loop_snapshot(const SimX& m, const LoopMem& mem, const LoopState& st, Recorder& rec, u64 next_ns) {
    const uint32_t lane = lane_id();
    const uint32_t idx = rec.next, n_rows = m.S.n_rows, n_dev = m.S.n_dev;
    const size_t k = (size_t)((((rec.loc >> idx) & 1u) ^ 1u) * rec.n_snaps + idx);   // the place the accepted timeline does not use
    const bool check = idx < rec.check_below;
    bool differs = false;
    const size_t nw = (size_t)m.S.n_ops * ROWL;
    u64* fr = rec.snap_free + k * (size_t)n_rows;
    if (check) {
        const size_t old = (size_t)(((rec.loc >> idx) & 1u) * rec.n_snaps + idx);
        differs = copy_words_compare(rec.snap_words + k * nw, mem.words, rec.snap_words + old * nw, (uint32_t)nw);
        const u64* ofr = rec.snap_free + old * (size_t)n_rows;
        for (uint32_t t = lane; t < n_rows; t += WAVE) {
            const u64 a = row_time<L64>(mem, st, t, n_dev), b = ofr[t];
            differs = differs || (a > next_ns ? a : next_ns) != (b > next_ns ? b : next_ns);
        }
        // a task of the changed op still pending would make equal words mean different things
        differs = differs || load_word<ROWL>(mem.words, rec.check_op) != W_NONE;
    } else {
        copy_words(rec.snap_words + k * nw, mem.words, (uint32_t)nw);
    }
    for (uint32_t t = lane; t < n_rows; t += WAVE) fr[t] = row_time<L64>(mem, st, t, n_dev);
    rec.next++;
    return check && !ballot(differs);
}

// The state of snapshot k of the accepted timeline: words copied, rows and queue rebuilt.  False if a link row is booked
// beyond 32 bits after the snapshot's time (and the rows are not 64-bit ones).
template <int Q, int ROWL, bool L64, class SimX>
__device__ __forceinline__ bool load_loop_snapshot(const SimX& m, const LoopMem& mem, LoopState& st, const Recorder& rec, uint32_t k) {
    const uint32_t lane = lane_id();
    const uint32_t n_rows = m.S.n_rows, n_dev = m.S.n_dev, n_ops = m.S.n_ops;
    const size_t at = (size_t)(((rec.loc >> k) & 1u) * rec.n_snaps + k);
    const u64 E = ((u64)k * rec.step) >> 1;        // no event before it
    st.E = E;
    bool beyond = false;
    const u64* fr = rec.snap_free + at * (size_t)n_rows;
    for (uint32_t t = lane; t < n_rows; t += WAVE) {
        const u64 a = fr[t];
        if (t < n_dev) { mem.crow[t] = a; continue; }
        if (L64) { mem.lrow64[t - n_dev] = a; continue; }
        const u64 r = a > E ? a - E : 0;
        beyond = beyond || r >= 0xffffffffull;
        mem.lrow[t - n_dev] = (uint32_t)r;
    }
    queue_clear<Q>(mem, st.q, n_ops);
    const u64* src = rec.snap_words + at * (size_t)n_ops * ROWL;
    // eight rows of 64 words in flight; a row of ROWL = 16 holds the words of four ops.  Q_SLOT: ops with an event are listed
    // first (where the queue's spill list will be) and get their slots afterwards.
    constexpr uint32_t PER = WAVE / ROWL;
    const uint32_t n_words = n_ops * ROWL;
    uint32_t n_listed = 0;
    for (uint32_t b = 0; b < n_words; b += 8 * WAVE) {
        u64 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) { const uint32_t t = b + u * WAVE + lane; v[u] = t < n_words ? src[t] : W_NONE; }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const uint32_t t = b + u * WAVE + lane;
            if (t < n_words) mem.words[t] = v[u];
            if (ballot(!(v[u] >> 63))) {
                for (uint32_t g = 0; g < PER; g++) {
                    const u64 mine = lane / ROWL == g ? v[u] : W_NONE;
                    if (!ballot(!(mine >> 63))) continue;
                    const uint32_t op = (b + u * WAVE) / ROWL + g;
                    if (Q == Q_SLOT) {
                        if (lane == 0) mem.spill_op[n_listed] = op;
                        n_listed++;
                    } else {
                        queue_insert<Q, ROWL>(mem, st, op, rel_key_or_none(wave_min_u64(mine & 1 ? mine : W_NONE), E),
                                              rel_key_or_none(wave_min_u64(mine & 1 ? W_NONE : mine), E), 0u);
                    }
                }
            }
        }
    }
    wave_sync();
    if (Q == Q_SLOT) {
        n_listed = first_u32(n_listed);
        // (an insertion puts at most one entry back on the list, over one already read)
        for (uint32_t t = 0; t < n_listed; t++) {
            const uint32_t op = first_u32(mem.spill_op[t]);
            queue_insert<Q, ROWL>(mem, st, op, rel_key_or_none(op_min_word<ROWL>(mem.words, op, 1), E), rel_key_or_none(op_min_word<ROWL>(mem.words, op, 0), E),
                                  exe_span(first_u32(mem.hdr[op].x)));
        }
    }
    return !ballot(beyond);
}

// Section 5.1 step 1 and the start of Algorithm 1: the tasks, how many inputs each waits for, the initial READY set,
// idle devices.  FILL: computes and keeps the set-up of every edge; otherwise the kept rows are valid and only read.
// Configurations are loaded 64 at a time and read from registers, so that no op waits for its own loads.
template <int Q, int ROWL, bool L64 = false, class SimX>
__device__ __forceinline__ void init_loop(SimX& m, const LoopMem& mem, LoopState& st, Counters& cnt, bool fill) {
    const uint32_t lane = lane_id();
    const uint32_t n_ops = m.S.n_ops, n_edges = m.S.n_edges;
    for (uint32_t r = lane; r < m.S.n_dev; r += WAVE) mem.crow[r] = 0;
    for (uint32_t r = lane; r < m.S.n_rows - m.S.n_dev; r += WAVE) {
        if (L64) mem.lrow64[r] = 0; else mem.lrow[r] = 0;
    }
    queue_clear<Q>(mem, st.q, n_ops);
    st.E = 0;
    if constexpr (ROWL == 16 && Q != Q_SLOT && !SimX::kTrain) {
        if (fill) {
            uint32_t own = lane;
            asm volatile("" : "+v"(own));         // (see kept_edges16)
            for (uint32_t t = own; t < n_ops * 16; t += WAVE) mem.words[t] = 0;
            wave_sync();
            kept_edges16(m, [&](uint32_t eid) { return mem.rows + (size_t)mem.edge_lite[eid].row * 16; }, mem.words);
            wave_sync();
            // the tasks, four ops at a time
            const uint32_t k = own & 15u, g = own >> 4;
            for (uint32_t base = 0; base < n_ops; base += 4) {
                const bool live = base + g < n_ops;
                const uint32_t j = live ? base + g : n_ops - 1;
                const uint32_t parts = unpack_cfg_lane(m.cfg_raw(j)).parts;
                const uint32_t pending = (uint32_t)mem.words[(size_t)j * 16 + k];
                const bool task = live && k < parts;
                const u64 w = !task ? W_NONE : (pending == 0 ? 1ull : (W_WAIT | ((u64)pending << 48)));
                wave_sync();
                if (live) mem.words[(size_t)j * 16 + k] = w;
                const u64 now_m = ballot(w == 1ull);
                const uint32_t mine = own - base;              // op `lane` is the mine-th of these four
                if (mine < 4 && ((uint32_t)(now_m >> (16 * mine)) & 0xffffu)) st.q.kd = 1u;
                cnt.n_compute += __popcll(ballot(task));
            }
            wave_sync();
            return;
        }
    }
    uint2 sc = make_uint2(0, 0);                    // configurations of the producers of the next 64 in-edges
    uint32_t seid = 0, ssrc = 0;                    // their edge ids and producers
    for (uint32_t base = 0; base < n_ops; base += WAVE) {
        const uint32_t jl = base + lane < n_ops ? base + lane : n_ops - 1;
        const uint2 cv = m.cfg_raw(jl);
        const uint32_t ibv = m.T.ops[jl].in_begin, iev = m.T.ops[jl].in_end;
        const uint32_t n = n_ops - base < (uint32_t)WAVE ? n_ops - base : (uint32_t)WAVE;
        for (uint32_t jj = 0; jj < n; jj++) {
            const uint32_t j = base + jj;
            const OpCfg cj = unpack_cfg(make_uint2(readlane_u32(cv.x, jj), readlane_u32(cv.y, jj)));
            const uint32_t ib = readlane_u32(ibv, jj), ie = readlane_u32(iev, jj);
            uint32_t pending = 0;
            for (uint32_t e_at = ib; e_at < ie; e_at++) {
                const uint32_t el = e_at & (WAVE - 1);
                if (el == 0) {
                    const uint32_t t = e_at + lane < n_edges ? e_at + lane : n_edges - 1;
                    ssrc = m.T.in_edges[t].src;
                    seid = m.T.in_edges[t].eid;
                    sc = m.cfg_raw(ssrc);
                }
                const uint32_t eid = readlane_u32(seid, el);
                uint32_t* row = mem.rows + (size_t)mem.edge_lite[eid].row * ROWL;
                if (fill) {
                    const DEdge e = m.T.in_edges[e_at];
                    const OpCfg cp = unpack_cfg(make_uint2(readlane_u32(sc.x, el), readlane_u32(sc.y, el)));
                    pending += kept_edge<ROWL>(m, row, e, cp, cj);
                } else {
                    if (SimX::kOvr && mem.priv) {
                        const uint32_t src = readlane_u32(ssrc, el);
                        if (src == m.ov_op) row = mem.priv + (size_t)(m.ov_in + (eid - m.T.ops[src].out_begin)) * (KEPT_ROWS * ROWL);
                        else if (j == m.ov_op) row = mem.priv + (size_t)(e_at - ib) * (KEPT_ROWS * ROWL);
                    }
                    pending += (row[KR_SORT * ROWL + (lane & (ROWL - 1))] >> 24) & 0x7fu;
                }
            }
            // pending < PENDING_LIMIT is guaranteed by ff_sim_create (at most 511 in-edges per op)
            const u64 w = lane >= cj.parts ? W_NONE : (pending == 0 ? 1ull : (W_WAIT | ((u64)pending << 48)));
            if (ROWL == WAVE || lane < (uint32_t)ROWL) mem.words[(size_t)j * ROWL + lane] = w;
            if (ballot(w == 1ull)) queue_insert<Q, ROWL>(mem, st, j, 1u, KEY_NONE, Q == Q_SLOT ? exe_span(first_u32(mem.hdr[j].x)) : 0u);
            cnt.n_compute += cj.parts;
        }
    }
    wave_sync();
}

// Section 4: every configuration valid?  Fills the kept op records.
template <int Q, class SimX>
__device__ __forceinline__ StrategyClass validate_loop(const SimX& m, const LoopMem& mem) {
    const StrategyClass cls = validate_with(m, [&](uint32_t i, const OpCfg& c, uint32_t exe) __attribute__((always_inline)) {
        uint4 h = kept_header(c, exe);
        const OpLite& o = mem.op_lite[i];
        if (o.out_end > o.out_begin || (SimX::kExt && m.S.sync && o.param_bytes != 0)) h.w |= HDR_RELEASES;
        mem.hdr[i] = h;
    });
    if (cls != STRATEGY_INVALID) {
        wave_sync();
        for (uint32_t i = lane_id(); i < m.S.n_ops; i += WAVE) {
            const OpLite o = mem.op_lite[i];
            uint32_t least = 0xffffffffu;
            if (o.out_end > o.out_begin) {
                least = mem.hdr[o.first.word & EL_DST].x;
                if (o.out_end - o.out_begin > RUN_EDGES) least = 0;
                else for (uint32_t e = o.out_begin + 1; e < o.out_end; e++) { const uint32_t x = mem.hdr[mem.edge_lite[e].word & EL_DST].x; least = x < least ? x : least; }
            }
            mem.hdr[i].z = least;
        }
    }
    wave_sync();
    return cls;
}

// Algorithm 1, result: see makespan (ffsim_events.h)
template <bool L64 = false, class SimX>
__device__ __forceinline__ u64 loop_makespan(const SimX& m, const LoopMem& mem, const LoopState& st) {
    u64 mk = 0;
    for (uint32_t d = lane_id(); d < m.S.n_dev; d += WAVE) mk = mem.crow[d] > mk ? mem.crow[d] : mk;
    if (SimX::kExt && m.S.sync) {
        for (uint32_t r = lane_id(); r < m.S.n_rows - m.S.n_dev; r += WAVE) {
            const u64 t = L64 ? mem.lrow64[r] : (mem.lrow[r] ? st.E + mem.lrow[r] : 0);
            mk = t > mk ? t : mk;
        }
    }
    return wave_max_u64(mk);
}

// ---- link rows in general order ----------------------------------------------------------

// fifo_commit (ffsim_events.h) on link rows: the same serialisation in 32-bit times relative to the epoch; sums that do
// not fit stick at 2^32 - 1 (the caller simulates again)
__device__ __forceinline__ uint32_t fifo_links(bool act, uint32_t row, uint32_t exe, uint32_t r, bool may_share, const LoopMem& mem) {
    const int lane = lane_id();
    uint32_t f = 0;
    bool lost = false;
    if (may_share) {
        if (act) mem.tag[row] = (uint8_t)lane;
        wave_sync();
        if (act) { lost = mem.tag[row] != (uint8_t)lane; f = mem.lrow[row]; }
    } else if (act) {
        f = mem.lrow[row];
    }
    const uint32_t base = f > r ? f : r;
    uint32_t end = __builtin_elementwise_add_sat(base, exe);
    u64 todo = ballot(lost);
    while (todo) {
        const int l = __builtin_ctzll(todo);
        const uint32_t lrow = readlane_u32(row, l);
        const bool peer = act && row == lrow;
        const u64 peers = ballot(peer);
        todo &= ~peers;
        uint32_t t = 0;
        u64 pm = peers;
        while (pm) {
            const int p = __builtin_ctzll(pm);
            pm &= pm - 1;
            t = __builtin_elementwise_add_sat(t, readlane_u32(exe, p));
            if (lane == p) end = __builtin_elementwise_add_sat(base, t);
        }
    }
    if (act) __hip_atomic_fetch_max(&mem.lrow[row], end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    wave_sync();
    return end;
}

// ---- the loop ----------------------------------------------------------------------------

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
// (one instruction that reads both halves; the compiler would rather multiply the halves by other factors one by one)
__device__ __forceinline__ uint32_t pair_product(u16x2 v) {
    uint32_t r;
    asm("v_mul_u32_u24_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1" : "=v"(r) : "v"(v));
    return r;
}
// Nothing is moved across: loads asked for above are all on their way before the first of them is waited for below.
__device__ __forceinline__ void in_flight() { __builtin_amdgcn_sched_barrier(0); }
// FAR_AWAY where the high half h of a distance between events of one kind is not 0, else its low half (the high half is looked at by itself: a comparison of
// all 64 bits wants its bound in two scalar registers, and the loop has none to spare)
__device__ __forceinline__ uint32_t near_u32(u64 d) {
    uint32_t hi = (uint32_t)(d >> 32);
    asm("" : "+v"(hi));
    const uint32_t lo = (uint32_t)d < FAR_AWAY ? (uint32_t)d : FAR_AWAY;
    return hi ? FAR_AWAY : lo;
}
// Distance of an event from the popped word K: KEY_NONE for events of the other kind (at odd distances), ones that lie before it and words that
// are no events; FAR_AWAY where it does not fit 32 bits.  (A waiting task's word may come out as FAR_AWAY where K is beyond 2^48.  Such a key
// delays nothing: it is looked into when the epoch gets there.)
__device__ __forceinline__ uint32_t event_distance(u64 word, u64 K) {
    const u64 d = word - K;
    const int32_t x = (int32_t)(((uint32_t)d << 31) | (uint32_t)(d >> 32));      // 0: of the same kind, and fits; positive: of the same kind, does not fit
    const uint32_t far = (uint32_t)(x >> 31) | FAR_AWAY;
    return x == 0 ? (uint32_t)d : far;
}
// n + 1 on the lanes of a mask
__device__ __forceinline__ uint32_t count_lanes(uint32_t n, u64 mask) {
    asm("v_addc_co_u32 %0, vcc, 0, %0, %1" : "+v"(n) : "s"(mask) : "vcc");
    return n;
}
// Behind a rarely taken branch with loads: nothing is in flight where it joins the main path, which would otherwise wait there for
// whatever this branch may have left in the air -- and with it for the stores of the step before.
__device__ __forceinline__ void vector_loads_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }
// a uniform value the compiler is not to recompute (or to move into a branch of its own)
__device__ __forceinline__ uint32_t opaque(uint32_t uniform) { asm("" : "+s"(uniform)); return uniform; }
// LDS addresses as numbers
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ uint32_t lds_addr(uint32_t* p) { return (uint32_t)(uintptr_t)(lds_u32*)p; }
__device__ __forceinline__ lds_u32* lds_at(uint32_t addr) { return (lds_u32*)(uintptr_t)addr; }
// *at = max(*at, v) on the lanes of both masks, which are combined at the last moment (see reg_passes), without a branch around
// it.  Call with all 64 lanes active; at must be in range on every lane of the masks.
__device__ __forceinline__ void row_max_of(uint32_t at, uint32_t v, u64 mask_a, u64 mask_b) {
    asm volatile("s_and_b64 exec, %2, %3\n\tds_max_u32 %0, %1\n\ts_mov_b64 exec, -1" : : "v"(at), "v"(v), "s"(mask_a), "s"(mask_b) : "memory", "scc");
}
// a & ~b, not before v is there
__device__ __forceinline__ u64 mask_without(u64 a, u64 b, uint32_t v) {
    u64 r;
    asm("s_andn2_b64 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b), "v"(v) : "scc");
    return r;
}
// lrow[row] = max(lrow[row], v) on the lanes of a mask, without a branch around it.  Call with all 64 lanes active; row must
// be in range on every lane of the mask.
__device__ __forceinline__ void row_max(uint32_t* lrow, uint32_t row, uint32_t v, u64 mask) {
    const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)(lrow + row);
    asm volatile("s_mov_b64 exec, %2\n\tds_max_u32 %0, %1\n\ts_mov_b64 exec, -1" : : "v"(at), "v"(v), "s"(mask) : "memory");
}
// lengths of the intersection of two pairs of ranges [lo, hi), 0 where they do not meet
__device__ __forceinline__ u16x2 meet(uint32_t lo_a, uint32_t hi_a, uint32_t lo_b, uint32_t hi_b) {
    const u16x2 lo = __builtin_elementwise_max(as_u16x2(lo_a), as_u16x2(lo_b));
    const u16x2 hi = __builtin_elementwise_min(as_u16x2(hi_a), as_u16x2(hi_b));
    return __builtin_elementwise_sub_sat(hi, lo);
}

// what a release has of an edge in registers: the consumer's words, the kept rows of both sides
struct EdgeLoad { u64 w; uint32_t exe, f, clo, chi, plo, phi, clo2, chi2, plo2, phi2, sortw; };

// ---- pace ----------------------------------------------------------------------------------
//
// Wavefronts that share a SIMD and have nothing behind them should finish together: with four the vector unit is busy, the last one alone leaves three
// quarters of it idle, and how long a candidate takes is only known when it has been simulated.  So a wavefront gives way as it gets on: its priority
// falls by one where half, three quarters and nine tenths of its ops are behind it (of all candidates it will simulate), and the others catch up.
// They do so slowly, with no more than the difference between their share and a lone wavefront's pace (those ahead still get every slot that is
// left), so the bounds come early: with the first at 0.7 or 0.8 half of the gain is lost; a quarter, a half and three quarters give 2 % less;
// priorities that change hands by the clock give nothing (the shares are even enough, the lengths are not).  One box, before the queues were
// split: 4096 x Inception-v3-shaped 6.82 -> 6.05 ms, x ResNet-101-shaped 13.4 -> 11.3, 8192 x AlexNet-shaped 0.45 -> 0.40; after that, with and without: 5.94 -> 5.34,
// 11.5 -> 9.85, 0.42 -> 0.37, 1024 searches x 32 steps (nodes four to a SIMD) 87.0 -> 80.5.  With one wavefront per SIMD nobody is waited for, and the code placed
// around it moves times by 2 to 3 % either way (1024 x AlexNet-shaped 160 -> 155 us, x NMT-shaped 55.9 -> 57.1 ms).  Kernels of another stream run at priority 0, below
// all but the last tenth: beside 4096 x Inception-v3-shaped a vector-bound one (the sine of 64 Mi values) takes 285 -> 450 us, a copy of 256 MiB 137 -> 142, a
// product of 2048^3 55 -> 38, and the batch itself is done in 5.9 instead of 8.0 ms; beside one wavefront per SIMD they take what they took (131 and 131 us, 112 and
// 112), so such launches have no rule of their own.  How far a wavefront is is looked at every 32 steps, where the loop's own bound is: a count of events costs such lone
// wavefronts 1 to 4 %.  (Trials are dealt out by length already and gain nothing.)
constexpr uint32_t PACE_STEPS = 32;      // queue steps between two looks at how far a wavefront is
struct NoPace {
    static constexpr bool kOn = false;
    __device__ __forceinline__ void at(uint32_t) {}
};
struct Pace {
    static constexpr bool kOn = true;
    uint32_t before, all;                // ops of the candidates done, of all candidates of this wavefront
    // op i is released or dequeued (ops are numbered in an order their tensors allow, so that is how far the candidate is)
    __device__ __forceinline__ void at(uint32_t i) {
        const u64 done = (u64)(before + i) * 256;
        if (done < (u64)all * 128) __builtin_amdgcn_s_setprio(3);
        else if (done < (u64)all * 192) __builtin_amdgcn_s_setprio(2);
        else if (done < (u64)all * 232) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
    }
};

// Algorithm 1 from the current state to the end.  RECORD, REG, STATS as for run_events; Q: LoopQueue; ROWL: lanes per row.
// Returns 0, RUN_CONVERGED, RESULT_RETRY or a RESULT_* code.
//
// What bounds it: one wavefront is one chain of instructions.  With one wavefront per SIMD the chain is the time; with four
// the vector unit is busy 91 to 99 % of it.  Both ask for fewer instructions per event (boxes of parts as pairs of 16-bit values, times in
// 32 bits, the queue in a register: a pass over the consumer parts took 95 instructions in run_events, it takes 51 to 58
// here), the former also for fewer crossings from the vector to the scalar unit and fewer taken branches: on a lone wavefront any
// instruction takes 4.6 to 6.4 cycles, dependent or not, but a scalar instruction that reads a mask or a lane's value
// just found waits 20, a taken branch 25.  So what is rare is looked for once per step, in one comparison; errors and bookings beyond 32 bits are
// noticed behind the loop (or every 32 steps); loads are kept in flight together (in_flight: left to itself the compiler now and then waits for one before it asks
// for the next, a trip to memory per step), the first edge of a release is asked for as soon as it is known that there is one.
//
// Order.  A dequeue touches its device row, a release the link rows of its node and the words of consumers.  So the only orders that matter are those of the
// dequeues on a device, of the releases on a node, and that everything that may make a task READY has been released before one that is READY later is
// dequeued, and the other way round.  Hence two queues: releases go on until the horizon, before which no task that is still to be dequeued can end (the first
// READY time of every op and its exeTime: q.kd + q.ex), then dequeues until the next release.  Within a step an op's events of one kind go together up
// to the other ops' first one (run_mask), whatever lies between them of the other kind; ops with several edges, or parameters, release of every node the
// parts that come first.  Against one queue in the order of time, with runs of ops with one edge: steps of the Inception-v3-shaped graph 1980 -> 1732,
// ResNet-101 4024 -> 3195, NMT 39148 -> 33224, AlexNet 158 -> 132.
// Both together (with the parts of a step sorted only where two on a node are out of order), per launch, one box: 4096 x Inception-v3-shaped 6.05 -> 5.33 ms, 4096 x
// ResNet-101-shaped 11.3 -> 9.88, 1024 x NMT-shaped 66.7 -> 57.0, 1024 x AlexNet-shaped 0.175 -> 0.162, training iterations (1024 x Inception-v3-shaped) 16.3 -> 11.9,
// general strategies (777 x ResNet-101-shaped on 5 x 3 devices) 21.7 -> 17.4, with parameter traffic (4096 x Inception-v3-shaped) 10.3 -> 7.3.
// A step has more to find out now, so calls in which few events go together lose: general strategies and explicit devices of the AlexNet-shaped graph on 4 to 8
// devices 0.96 to 0.99x, chains of a few changes with parameter traffic on graphs of 6 and 12 ops 0.96 to 0.99x.
// L64: link rows are absolute 64-bit times (mem.lrow64); the form for what RESULT_RETRY leaves over, REG = false only.
template <bool RECORD, bool REG, bool STATS, int Q, int ROWL, bool L64 = false, class SimX, class PaceX = NoPace>
__device__ __forceinline__ u64 run_loop(SimX& m, const LoopMem& mem, LoopState& st, Counters& cnt, Recorder& rec, PaceX pace = PaceX()) {
    static_assert(!(REG && L64), "64-bit link rows go with the general form");
    constexpr bool EDGED = !SimX::kExt;      // without parameter traffic only ops with an edge have anything to release
    typedef typename std::conditional<L64, u64, uint32_t>::type T;      // times of transfers: absolute, or relative to the epoch
    const uint32_t lane = lane_id();
    PROF_DECL
    const SimDev& S = m.S;
    u64* words = mem.words;
    uint32_t latest_hi = 0;                  // per lane: high half of the latest time (see TIME_LIMIT)
    uint32_t latest_link = 0;                // per lane: latest time of a transfer relative to the epoch (all ones: a link row is booked beyond 32 bits)
    auto beyond_32 = [&]() { return !L64 && ballot(latest_link == 0xffffffffu) != 0; };
    const uint32_t G = m.gpn();
    const uint32_t n_links = S.n_rows - S.n_dev;
    // chosen per lane between the two of a pair: in vector registers, so that a select needs one scalar operand only
    const uint32_t m_near = vector_copy(S.near_link.m), m_far = vector_copy(S.far_link.m);
    const uint32_t k_near = vector_copy(S.near_link.k), k_far = vector_copy(S.far_link.k);
    const uint32_t l_near = vector_copy(S.near_link.lat1), l_far = vector_copy(S.far_link.lat1);
    const uint32_t elem_sh = vector_copy(S.elem_sh);
    Queue& q = st.q;
    // (uniform already, which the compiler does not always see where the state was rebuilt from memory)
    st.E = first_u64(st.E);
    q.n_spill = first_u32(q.n_spill);
    q.spill_min = first_u64(q.spill_min);
    if (RECORD) { rec.step = first_u64(rec.step); rec.next = first_u32(rec.next); rec.n_snaps = first_u32(rec.n_snaps); rec.check_below = first_u32(rec.check_below); }
    // Steps to the next look at the pace, and steps left behind that (every step deals with an event: a run that needs more has gone wrong).
    uint32_t max_steps = 2 * S.n_ops * WAVE + 8, last = 0;
    int32_t left = 0;
    uint32_t snap_key = KEY_NONE;            // RECORD: key of the next snapshot boundary
    auto set_snap_key = [&]() {
        if (RECORD) {
            const u64 at = (u64)rec.next * rec.step;
            snap_key = rec.next < rec.n_snaps ? (at <= 2 * st.E ? 0u : rel_key(at, st.E)) : KEY_NONE;
        }
    };
    set_snap_key();
    auto keys_min2 = [&](uint32_t& a, uint32_t& b) __attribute__((always_inline)) { if (Q == Q_OP16) row0_min2_u32(a, b); else wave_min2_u32(a, b); };
    auto keys_min = [&](uint32_t key) __attribute__((always_inline)) { return Q == Q_OP16 ? row0_min_u32(key) : wave_min_u32(key); };
    // The smallest keys of both kinds, and the first one at which something not known yet may have to be released (at most KEY_REFRESH; 0: to be found).
    uint32_t m_deq = keys_min(q.kd), m_rel = keys_min(q.kr), horizon = 0;
    uint32_t spill_key = KEY_NONE;           // of the smallest word on the spill list
    for (;;) {
        // ---- pop
        uint32_t kmin = m_deq < m_rel ? m_deq : m_rel;       // smallest key of the slots
        left--;
        if (__builtin_expect((int32_t)(kmin | (uint32_t)left | (Q == Q_SLOT ? 0u - q.n_spill : 0u)) < 0, 0)) {
            if (left < 0) {
                if (max_steps == 0 || left != -1) break;
                if (beyond_32()) break;
                if (PaceX::kOn) pace.at(first_u32(last));
                left = (int32_t)(PACE_STEPS < max_steps ? PACE_STEPS : max_steps);
                max_steps -= (uint32_t)left;
            }
            if (kmin >= KEY_REFRESH) {
                if (!advance_epoch<Q, ROWL, L64>(mem, st, n_links)) break;
                set_snap_key();
                m_deq = keys_min(q.kd);
                m_rel = keys_min(q.kr);
                kmin = m_deq < m_rel ? m_deq : m_rel;
                horizon = 0;
            }
            if (Q == Q_SLOT && q.n_spill) {
                for (uint32_t guard = 0; q.n_spill && guard < S.n_ops + WAVE; guard++) {
                    const u64 top = 2 * st.E + kmin;
                    if (q.spill_min > top) break;
                    if (q.spill_min == top) {
                        // equal keys: only needed if a spilled op comes first; bring in all of them
                        const uint32_t lo_op = wave_min_u32(slot_key(q) == kmin ? q.op : NO_OP);
                        uint32_t sop = NO_OP;
                        for (uint32_t t = lane; t < q.n_spill; t += WAVE)
                            if (mem.spill_key[t] == top && mem.spill_op[t] < sop) sop = mem.spill_op[t];
                        if (wave_min_u32(sop) > lo_op) break;
                    }
                    queue_unspill<ROWL>(mem, st);
                    m_deq = wave_min_u32(q.kd); m_rel = wave_min_u32(q.kr);
                    kmin = m_deq < m_rel ? m_deq : m_rel;
                }
                horizon = 0;                     // (ops on the list are not looked at: everything in the order of time)
                spill_key = q.n_spill ? rel_key(q.spill_min, st.E) : KEY_NONE;
                vector_loads_done();
            }
            if (kmin >= KEY_REFRESH) { left = LOST; break; }     // an event before the epoch
        }
        if (RECORD) {
            // the state before the first event at or after a multiple of `step` is a snapshot
            while (kmin >= snap_key) {
                if (save_loop_snapshot<ROWL, L64>(m, mem, st, rec, st.E + (kmin >> 1))) return beyond_32() ? RESULT_RETRY : RUN_CONVERGED;
                set_snap_key();
            }
        }
        // What is released next?  The first event if it is a release, else whatever comes before the horizon (and the next snapshot).
        const uint32_t ahead = RECORD && snap_key < horizon ? snap_key : horizon;
        const bool rel = m_rel < (m_deq > ahead ? m_deq : ahead);
        // the first op with that event (its slot: at), the smallest key of the others
        u64 at;
        uint32_t i, other_key;
        auto pop = [&](uint32_t key) __attribute__((always_inline)) {
            at = ballot(key == kmin);
            if (Q != Q_SLOT) {
                i = __builtin_ctzll(at);         // lowest op among equal keys
                at = ballot(lane == i);
            } else {
                if (at & (at - 1)) {
                    i = wave_min_u32(lanes_of(at) ? q.op : NO_OP);
                    at &= ballot(q.op == i);
                } else {
                    i = readlane_u32(q.op, __builtin_ctzll(at));
                }
            }
            if (PaceX::kOn) last = i;
            cnt.n_events++;
        };
        // An op whose words do not have the event that the queue has of it: noticed at the next pop.  (The step itself finds no part and changes no task
        // of the op; what a release does to its consumers goes no further than that pop either.  Asked behind the step's work, by a select: where the mask is
        // found, it costs 1024 x NMT-shaped 0.5 % and 1024 training iterations 0.9 % more, as a branch there training iterations 2 % and NMT-shaped 1 % less.)
        auto found = [&](u64 mask) __attribute__((always_inline)) { left = mask ? left : LOST + 1; };
        // A run: the events of the op up to the first event of another op of that kind, the first one of the other kind that may matter, the first one the
        // run itself may bring about, and the next snapshot.
        auto run_mask = [&](uint32_t d, uint32_t until, uint32_t first_new) __attribute__((always_inline)) {
            uint32_t b = other_key < until ? other_key : until;
            b = spill_key < b ? spill_key : b;
            if (RECORD) b = snap_key < b ? snap_key : b;
            b -= kmin;
            first_new = exe_span(first_new);
            b = b < first_new ? b : first_new;
            return ballot(d < (b > 1u ? b : 1u));
        };
        if (!rel) {
            // ---- dequeue READY tasks: start = max(readyTime, device free), end = start + exeTime
            pop(q.kd);
            const u64 K = 2 * st.E + kmin;       // the popped word
            PROF_MARK(1)
            // What depends only on i is requested together, and the smallest key of the other ops is found while that is on its way.
            u64 k0 = load_word<ROWL>(words, i);
            const uint4 h = mem.hdr[i];
            in_flight();
            other_key = keys_min(lanes_of(at) ? KEY_NONE : q.kd);
            in_flight();
            const uint32_t exe = first_u32(h.x), offs = first_u32(h.y), hflags = first_u32(h.w);
            OpCfg ci;
            ci.off = offs & 0xffffu; ci.stride = offs >> 16; ci.parts = hflags & 0xffffu;
            const uint32_t dev_p = m.template device_of<REG>(i, ci);
            PROF_MARK(1)
            PROF_VMWAIT(2)
            const uint32_t d = event_distance(k0, K);
            u64 mask = run_mask(d, m_rel, exe);
            const bool may_share = !REG && ((SimX::kExt && m.devmap != nullptr) || !(ci.stride == 1 && ci.parts <= S.n_dev));
            if (may_share) {
                // of the parts on one device only the first
                for (u64 t = mask & ballot(d != 0); t; t &= t - 1) {
                    const int p = __builtin_ctzll(t);
                    const uint32_t dp = readlane_u32(d, p), vp = readlane_u32(dev_p, p);
                    if (ballot(dev_p == vp) & ballot(d < dp)) mask &= ~(1ull << p);
                }
            }
            const bool in_mask = lanes_of(mask);
            u64 end;
            if (REG) {
                const u64 f = mem.crow[dev_p];               // (in range for every lane)
                const u64 r = k0 >> 1;
                end = (f > r ? f : r) + exe;
                if (in_mask) mem.crow[dev_p] = end;
                wave_sync();
            } else {
                end = fifo_commit(in_mask, dev_p, exe, k0 >> 1, may_share, m.L);
            }
            const u64 w = end << 1;
            const uint32_t dw = near_u32(w - K);
            const uint32_t none = (hflags & HDR_RELEASES) ? 0u : KEY_NONE;
            if (in_mask) {
                k0 = w | ((u64)none << 32 | none);           // (nothing to release: W_NONE)
                words[(size_t)i * ROWL + lane] = k0;
                latest_hi = (uint32_t)(end >> 32) > latest_hi ? (uint32_t)(end >> 32) : latest_hi;
                if (RECORD && rec.end_try) rec.end_try[(size_t)i * ROWL + lane] = rec.tag | end;
            }
            PROF_MARK(3)
            found(mask);
            // ---- the op's next events
            uint32_t nd = in_mask ? KEY_NONE : d, nr = in_mask ? dw | none : KEY_NONE;
            if (ROWL == 16) row0_min2_u32(nd, nr); else wave_min2_u32(nd, nr);
            const uint32_t nk = next_key(kmin, nd), new_rel = next_key(kmin, nr);
            const bool me = lanes_of(at);
            q.kd = me ? nk : q.kd;
            const uint32_t r = me ? new_rel : KEY_NONE;
            q.kr = r < q.kr ? r : q.kr;
            if (Q == Q_SLOT) q.op = me && (q.kd & q.kr) == KEY_NONE ? NO_OP : q.op;
            m_deq = nk < other_key ? nk : other_key;
            m_rel = new_rel < m_rel ? new_rel : m_rel;
            horizon = 0;
        } else {
            // ---- release the successors of finished tasks
            kmin = m_rel;
            pop(q.kr);
            const u64 K = 2 * st.E + kmin;
            PROF_MARK(1)
            // (the static record through the vector unit as well: a scalar load of it would be sunk below the wait for the words and be waited for once more)
            // (and ahead of the words: it is the same for all candidates and close by, the words are this candidate's and often are not.  Loads come back
            // in the order they were asked for in, so the first edge is asked for while the words are on their way:
            // with the minima in pairs 1024 x AlexNet-shaped 163.4 -> 157.9 us, 1024 x NMT-shaped 56.3 -> 55.7 ms, 4096 proposals 57.7 -> 55.7.)
            // With parameter traffic an op may have no edge to ask for, and the branch around it costs more than that gives: words first there.
            const uint4* lite_at = (const uint4*)mem.op_lite + 2 * (size_t)vector_copy(i);
            u64 k0;
            uint4 h, lite0, lite1;
            if (!EDGED) { k0 = load_word<ROWL>(words, i); h = mem.hdr[i]; }
            lite0 = lite_at[0]; lite1 = lite_at[1];
            in_flight();
            if (EDGED) { k0 = load_word<ROWL>(words, i); h = mem.hdr[i]; }
            in_flight();
            uint32_t x = __builtin_elementwise_add_sat(q.kd, q.ex);
            other_key = lanes_of(at) ? KEY_NONE : q.kr;
            keys_min2(other_key, x);
            horizon = (x < KEY_REFRESH ? x : KEY_REFRESH) - 1;
            in_flight();
            OpLite lite;
            lite.out_begin = first_u32(lite0.x); lite.out_end = first_u32(lite0.y); lite.param_bytes = first_u32(lite0.z);
            lite.first.word = first_u32(lite1.x); lite.first.in_pos = SimX::kOvr ? first_u32(lite1.y) : 0u; lite.first.row = first_u32(lite1.z);
            const uint32_t out_begin = lite.out_begin, out_end = lite.out_end;
            // What a release needs of an edge: the consumer's words and the kept rows of both sides.
            auto load_edge = [&](const EdgeLite& lit, uint32_t ei) __attribute__((always_inline)) {
                const uint32_t j = lit.word & EL_DST;
                const uint32_t* row = mem.rows + (size_t)lit.row * ROWL;
                if (SimX::kOvr && mem.priv) {
                    // a trial mutation's own edges have rows of their own
                    if (i == m.ov_op) row = mem.priv + (size_t)(m.ov_in + (ei - out_begin)) * (KEPT_ROWS * ROWL);
                    else if (j == m.ov_op) row = mem.priv + (size_t)lit.in_pos * (KEPT_ROWS * ROWL);
                }
                const uint32_t* p = row + (ROWL < WAVE ? (lane & (ROWL - 1)) : lane);
                EdgeLoad v;
                v.w = load_word<ROWL>(words, j);
                v.exe = mem.hdr[j].x;
                v.f = p[KR_F * ROWL]; v.clo = p[KR_CLO * ROWL]; v.chi = p[KR_CHI * ROWL]; v.plo = p[KR_PLO * ROWL]; v.phi = p[KR_PHI * ROWL];
                v.clo2 = 0; v.chi2 = 0; v.plo2 = 0; v.phi2 = 0; v.sortw = 0;
                if (lit.word & EL_FOUR) { v.clo2 = p[KR_CLO2 * ROWL]; v.chi2 = p[KR_CHI2 * ROWL]; v.plo2 = p[KR_PLO2 * ROWL]; v.phi2 = p[KR_PHI2 * ROWL]; }
                if (!REG) v.sortw = p[KR_SORT * ROWL];
                in_flight();
                return v;
            };
            // (from memory the first edge's are asked for now, and are there when it has been found out which parts are released)
            constexpr bool EARLY = Q == Q_SLOT;
            EdgeLite lit = lite.first;
            EdgeLoad ed;
            if (EARLY && EDGED) ed = load_edge(lit, out_begin);
            const uint32_t offs = first_u32(h.y), next_exe = first_u32(h.z), hflags = first_u32(h.w);
            OpCfg ci;
            ci.off = offs & 0xffffu; ci.stride = offs >> 16; ci.parts = hflags & 0xffffu;
            const uint32_t dev_p = m.template device_of<REG>(i, ci);
            PROF_MARK(1)
            PROF_VMWAIT(2)
            const uint32_t d = event_distance(k0, K);
            if (EARLY && !EDGED && out_end > out_begin) ed = load_edge(lit, out_begin);
            u64 mask = run_mask(d, horizon, next_exe);
            const uint32_t node_p = m.node_of(dev_p);
            // Transfers from one node (whose link rows are its own) go in the order of (time, edge, part), those from different nodes in any.  The edges
            // are gone through one after the other, each part by part, and parameters behind them: of the parts on a node only the first may go where there
            // is more than one edge to go through, and with one edge the parts are sorted where one on the same node before it is later.
            uint32_t sort = 0;
            {
                const u64 later = mask & ballot(d != 0);
                if (later) {
                    if (out_end - out_begin > 1 || (SimX::kExt && S.sync && lite.param_bytes)) {
                        for (u64 t = later; t; t &= t - 1) {
                            const int p = __builtin_ctzll(t);
                            const uint32_t dp = readlane_u32(d, p), np = readlane_u32(node_p, p);
                            if (ballot(node_p == np) & ballot(d < dp)) mask &= ~(1ull << p);
                        }
                    } else if (!REG) {
                        sort = 1;
                    } else {
                        // (the parts of a node are consecutive lanes; on a machine that the op goes all the way round they may come up once more at the end)
                        const uint32_t local = m.local_of(dev_p, node_p), mine = lanes_of(mask) ? d : KEY_NONE;
                        uint32_t before = lanes_of(mask) ? d : 0u, latest = 0;
                        for (uint32_t t = 1; t < G; t++) {
                            before = wave_shr1_u32(before);
                            before = local >= t ? before : 0u;
                            latest = before > latest ? before : latest;
                        }
                        if (ballot(latest > mine)) sort = 1;
                        if (ci.parts + G > S.n_dev) {
                            const uint32_t node0 = readlane_u32(node_p, 0);
                            const u64 same = mask & ballot(node_p == node0), again = same & ballot(dev_p < ci.off);
                            if (again && same != again) sort = 1;
                        }
                    }
                }
            }
            const bool in_mask = lanes_of(mask);
            // sorted: by (time, part); lane t then stands for the t-th part in what the passes read of the parts
            uint32_t order = lane;
            u64 parts_m = mask;
            if (sort) {
                uint32_t rank = 0;
                u64 t = mask;
                while (t) {
                    const int p = __builtin_ctzll(t);
                    t &= t - 1;
                    const uint32_t dp = readlane_u32(d, p);
                    rank = count_lanes(rank, ballot(dp < d) | (ballot(dp == d) & ~((2ull << p) - 1)));
                }
                const u64 rest = ~mask;
                const uint32_t behind = __builtin_amdgcn_mbcnt_hi((uint32_t)(rest >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)rest, (uint32_t)__popcll(mask)));
                order = scatter_u32(lane, in_mask ? rank : behind);
                parts_m = __popcll(mask) == 64 ? ~0ull : (1ull << __popcll(mask)) - 1;
            }
            uint32_t now_v = (kmin + d) >> 1, dev_v = dev_p;
            if (sort) { now_v = gather_u32(now_v, order); dev_v = gather_u32(dev_p, order); }
            // REG: what a pass needs of its producer part, ready to be read out of the part's lane
            const uint32_t node_v = m.node_of(dev_v);
            const uint32_t near_at_v = lds_addr(mem.lrow) + 4 * (dev_v * G), far_at_v = lds_addr(mem.lrow) + 4 * (S.n_nodes * G * G + node_v * S.n_nodes);
            // the records of the op's edges behind the first, a lane per edge, requested before the first edge is gone through
            uint4 lits = make_uint4(0, 0, 0, 0);
            auto load_lits = [&](uint32_t from) __attribute__((always_inline)) {
                const uint32_t t = from + lane < out_end ? from + lane : out_end - 1;
                lits = ((const uint4*)mem.edge_lite)[t];
            };
            if (out_end - out_begin > 1) load_lits(out_begin);
            auto next_edge = [&](uint32_t ei) __attribute__((always_inline)) {
                const uint32_t l = (ei - out_begin) & (WAVE - 1);
                if (l == 0) load_lits(ei);
                lit.word = readlane_u32(lits.x, l);
                lit.in_pos = SimX::kOvr ? readlane_u32(lits.y, l) : 0u;
                lit.row = readlane_u32(lits.z, l);
            };
            for (uint32_t ei = out_begin; EDGED || ei < out_end; ei++) {
                if (!EARLY) ed = load_edge(lit, ei);
                const uint32_t el = lit.word;
                const uint32_t j = el & EL_DST;
                const u64 w = ed.w;
                const uint32_t f = ed.f, sortw = ed.sortw, ed_exe = ed.exe;
                uint32_t clo = ed.clo, chi = ed.chi, plo = ed.plo, phi = ed.phi, clo2 = ed.clo2, chi2 = ed.chi2, plo2 = ed.plo2, phi2 = ed.phi2;
                if (ROWL < WAVE) {
                    // (no part there: an empty range)
                    chi = lane < (uint32_t)ROWL ? chi : 0u;
                    chi2 = lane < (uint32_t)ROWL ? chi2 : 0u;
                }
                const uint32_t dev_c = f & 1023u;
                const uint32_t node_c = SimX::kGpn == 4 ? dev_c >> 2 : (f >> 10) & 1023u;
                const uint32_t local_c = m.local_of(dev_c, node_c);
                const uint32_t far_base = S.n_nodes * G * G + node_c;
                u64 ready64 = w & (TIME_LIMIT - 1);
                T ready;                                    // relative to the epoch; what lies before it no longer matters
                if constexpr (L64) {
                    ready = ready64;
                } else {
                    const u64 rr = ready64 - st.E;
                    ready = (int32_t)(uint32_t)(rr >> 32) < 0 ? 0u : (uint32_t)rr;
                }
                const uint32_t pending = (uint32_t)(w >> 48) & PENDING_LIMIT;
                uint32_t c1 = 0, c2 = 0, c3 = 0, last_run = 0, first_len = 0;
                bool wrapped = false;
                if (REG) {
                    c1 = (uint32_t)((int32_t)(f << 11) >> 31);
                    c2 = (uint32_t)((int32_t)(f << 10) >> 31);
                    c3 = (uint32_t)((int32_t)(f << 9) >> 31);
                    last_run = (uint32_t)((int32_t)(f << 4) >> 31);
                    const uint32_t u = first_u32(f);         // the last two fields are the same in every lane
                    wrapped = (u >> 28) & 1u;
                    first_len = u >> 29;
                }
                const uint32_t local_c4 = 4 * local_c, node_c4 = 4 * node_c;
                const u64 dup_m = REG ? 0 : ballot((sortw >> 23) & 1u);
                PROF_MARK(4)
                PROF_VMWAIT(5)

                if (sort) {
                    plo = gather_u32(plo, order); phi = gather_u32(phi, order);
                    if (el & EL_FOUR) { plo2 = gather_u32(plo2, order); phi2 = gather_u32(phi2, order); }
                }
                uint32_t hits = 0;
                // One pass per producer part.  FORM 0: the parts' boxes meet in one pair of dims; 1: in one pair of dims, the
                // other contributes the same factor for every producer part (which does not split it); 2: in both.
                uint32_t factor = 1;
                // The regular form's passes avoid what a lone wavefront waits for: about 20 cycles wherever the scalar unit needs what
                // the vector unit has just found, 25 for a taken branch.  Lane masks are used as the comparisons leave them, or
                // combined long after; what the part brings is read from its lane ready for use, and the next part's
                // number is known a pass ahead.
                auto reg_passes = [&](auto form_) __attribute__((always_inline)) {
                    constexpr int FORM = decltype(form_)::value;
                    u64 todo = parts_m;
                    int next = __builtin_ctzll(todo);
                    do {
                        const int kp = next;
                        todo &= todo - 1;
                        next = __builtin_ctzll(todo);
                        uint32_t elems = pair_product(meet(clo, chi, readlane_u32(plo, kp), readlane_u32(phi, kp)));
                        if (FORM == 2) elems *= pair_product(meet(clo2, chi2, readlane_u32(plo2, kp), readlane_u32(phi2, kp)));
                        const uint32_t dev_a = readlane_u32(dev_v, kp), node_a = readlane_u32(node_v, kp), now_kp = readlane_u32(now_v, kp);
                        const u64 hit_m = ballot(elems != 0), near_m = ballot(node_c == node_a), diff_m = ballot(dev_c != dev_a);
                        const bool near = lanes_of(near_m);
                        if (FORM == 1) elems *= factor;
                        // Section 5.1: the link device between the two devices (in range for every lane); assumption A2: transfer time
                        const uint32_t near_at = readlane_u32(near_at_v, kp) + local_c4, far_at = readlane_u32(far_at_v, kp) + node_c4;
                        const uint32_t at_row = near ? near_at : far_at;
                        const uint32_t fr = *lds_at(at_row);
                        uint32_t lm = near ? m_near : m_far, lk = near ? k_near : k_far, ll = near ? l_near : l_far;
                        if (SimX::kExt && S.link_table) {
                            if (lanes_of(hit_m & diff_m & near_m)) { const uint4 e = mem.links[(dev_a - node_a * G) * G + local_c]; lm = e.x; lk = e.y; ll = e.z; }
                        }
                        if (SimX::kExt && S.node_table) {
                            if (lanes_of(hit_m & ~near_m)) { const uint4 e = mem.links[G * G + node_a * S.n_nodes + node_c]; lm = e.x; lk = e.y; ll = e.z; }
                        }
                        const uint32_t ns = (__umulhi((elems << elem_sh) - 1u, lm) >> lk) + ll;
                        // consumer parts on one node are consecutive lanes: a running sum along them is the FIFO order on the
                        // link row they share (rows between GPUs of one node are private)
                        uint32_t acc = lanes_of(mask_without(hit_m, near_m, ns)) ? ns : 0u;
                        uint32_t y = wave_shr1_u32(acc) & c1;
                        acc += y;
                        if (SimX::kGpn == 4) {
                            y = wave_shr1_u32(y) & c2; acc += y;
                            y = wave_shr1_u32(y) & c3; acc += y;
                        } else {
                            for (uint32_t s = 2; s < G; s++) { y = wave_shr1_u32(y) & (uint32_t)((int32_t)(f << (12 - s)) >> 31); acc += y; }
                        }
                        if (__builtin_expect(wrapped, 0)) acc += readlane_u32(acc, (int)first_len) & last_run;
                        const uint32_t end = __builtin_elementwise_add_sat(fr > now_kp ? fr : now_kp, near ? ns : acc);
                        row_max_of(at_row, end, hit_m, diff_m);
                        wave_sync();
                        uint32_t came = lanes_of(diff_m) ? end : now_kp;
                        came = lanes_of(hit_m) ? came : 0u;
                        ready = came > ready ? came : ready;
                        hits = count_lanes(hits, hit_m);
                        if (STATS) {
                            cnt.n_pairs += __popcll(hit_m);
                            cnt.n_comm += __popcll(hit_m & diff_m);
                            if (lanes_of(hit_m & diff_m)) cnt.sum_comm_ns += ns;     // per-lane partial sums, reduced by the caller
                        }
                    } while (todo);
                };
                auto passes = [&](auto form_) __attribute__((always_inline)) {
                    constexpr int FORM = decltype(form_)::value;
                    if constexpr (REG) {
                        if (FORM == 1) chi = factor ? chi : clo;         // (nothing is read)
                        reg_passes(form_);
                        return;
                    }
                    u64 todo = parts_m;
                    do {
                        const int kp = __builtin_ctzll(todo);
                        todo &= ~(1ull << kp);
                        uint32_t elems = pair_product(meet(clo, chi, readlane_u32(plo, kp), readlane_u32(phi, kp)));
                        if (FORM == 2) elems *= pair_product(meet(clo2, chi2, readlane_u32(plo2, kp), readlane_u32(phi2, kp)));
                        if (FORM == 1) elems *= factor;
                        const u64 hit_m = ballot(elems != 0);
                        if (!hit_m) continue;
                        const uint32_t dev_a = readlane_u32(dev_v, kp), now_kp = readlane_u32(now_v, kp);
                        const uint32_t node_a = SimX::kGpn == 4 ? dev_a >> 2 : m.node_of(dev_a);
                        const u64 comm_m = hit_m & ballot(dev_c != dev_a);
                        const T from = L64 ? (T)(st.E + now_kp) : (T)now_kp;
                        T arrive = from;
                        if (comm_m) {
                            // Section 5.1: the link device between the two devices; assumption A2: transfer time
                            const u64 near_m = ballot(node_c == node_a);
                            const bool near = lanes_of(near_m), comm = lanes_of(comm_m);
                            const uint32_t row_near = opaque(dev_a * G) + local_c, row_far = opaque(node_a * S.n_nodes) + far_base;
                            const uint32_t row = near ? row_near : row_far;
                            uint32_t lm = near ? m_near : m_far, lk = near ? k_near : k_far, ll = near ? l_near : l_far;
                            if (SimX::kExt && S.link_table) {
                                if (comm && near) { const uint4 e = mem.links[m.local_of(dev_a, node_a) * G + local_c]; lm = e.x; lk = e.y; ll = e.z; }
                            }
                            if (SimX::kExt && S.node_table) {
                                if (comm && !near) { const uint4 e = mem.links[G * G + node_a * S.n_nodes + node_c]; lm = e.x; lk = e.y; ll = e.z; }
                            }
                            const uint32_t ns = (__umulhi((elems << elem_sh) - 1u, lm) >> lk) + ll;
                            const u64 far_m = comm_m & ~near_m;
                            T end;
                            if constexpr (L64) {
                                end = fifo_commit(comm, row, ns, from, true, WaveLds{mem.lrow64, nullptr, nullptr, mem.tag});
                            } else {
                                // transfers to another node queue on the link row of the node pair in consumer-part order:
                                // a running sum along the consumer's parts taken in (node, part) order
                                end = 0;
                                if (far_m) {
                                    uint32_t incl = ns;
                                    const uint32_t fr = mem.lrow[row];
                                    if (far_m & (far_m - 1)) {
                                        const uint32_t x = gather_u32(lanes_of(far_m) ? ns : 0u, sortw & 63u);
                                        incl = gather_u32(seg_running_sum(x, (sortw >> 22) & 1u), (sortw >> 6) & 63u);
                                    }
                                    end = __builtin_elementwise_add_sat(fr > now_kp ? fr : now_kp, incl);
                                    row_max(mem.lrow, row, end, far_m);
                                    wave_sync();
                                }
                                const u64 here_m = comm_m & near_m;
                                if (here_m) {
                                    const bool here = lanes_of(here_m);
                                    const uint32_t e = fifo_links(here, row, ns, now_kp, (here_m & dup_m) != 0, mem);
                                    end = here ? e : end;
                                }
                            }
                            arrive = comm ? end : from;
                            if (STATS) {
                                cnt.n_comm += __popcll(comm_m);
                                if (comm) cnt.sum_comm_ns += ns;     // per-lane partial sums, reduced by the caller
                            }
                        }
                        const T came = lanes_of(hit_m) ? arrive : 0u;
                        ready = came > ready ? came : ready;
                        hits = count_lanes(hits, hit_m);
                        if (STATS) cnt.n_pairs += __popcll(hit_m);
                    } while (todo);
                };
                if (!(el & EL_FOUR)) {
                    passes(std::integral_constant<int, 0>{});
                } else if ((el & EL_CONTRIB) || (hflags & (HDR_SPLIT01 | HDR_SPLIT23)) == (HDR_SPLIT01 | HDR_SPLIT23)) {
                    passes(std::integral_constant<int, 2>{});
                } else {
                    if (hflags & HDR_SPLIT23) {
                        factor = pair_product(as_u16x2(chi) - as_u16x2(clo));
                        clo = clo2; chi = chi2; plo = plo2; phi = phi2;
                    } else {
                        factor = pair_product(as_u16x2(chi2) - as_u16x2(clo2));
                    }
                    passes(std::integral_constant<int, 1>{});
                }
                PROF_MARK(6)
                const bool touched = hits != 0;
                const u64 touched_m = ballot(touched);
                if (touched_m) {
                    const uint32_t left = pending - hits;
                    const u64 abs = L64 ? (u64)ready : st.E + ready;
                    const u64 zero_m = ballot(left == 0), ready_m = touched_m & zero_m;
                    const uint32_t abs_lo = (uint32_t)abs, abs_hi = (uint32_t)(abs >> 32);
                    // (both words, then a select: the compiler would put either side into a branch of its own)
                    uint32_t waits_hi = (left << 16) | 0x80000000u | (abs_hi & 0xffffu), ready_hi = __builtin_amdgcn_alignbit(abs_hi, abs_lo, 31);
                    asm("" : "+v"(waits_hi), "+v"(ready_hi));
                    const uint32_t w_lo = lanes_of(zero_m) ? (abs_lo << 1) | 1u : abs_lo;
                    const uint32_t w_hi = lanes_of(zero_m) ? ready_hi : waits_hi;
                    if (lanes_of(touched_m)) {
                        words[(size_t)j * ROWL + lane] = (u64)w_hi << 32 | w_lo;
                        latest_hi = abs_hi > latest_hi ? abs_hi : latest_hi;
                        if (!L64) latest_link = (uint32_t)ready > latest_link ? (uint32_t)ready : latest_link;
                    }
                    if (ready_m) {
                        uint32_t rel = (uint32_t)ready;
                        if constexpr (L64) { const u64 r = ready - st.E; rel = r >= KEY_FAR ? KEY_FAR : (uint32_t)r; }
                        const uint32_t first = part_min_of<ROWL>(rel, ready_m);
                        const uint32_t key = first >= KEY_REFRESH - 1 ? KEY_FAR : 2 * first + 1;
                        const uint32_t ex = exe_span(ed_exe);
                        queue_insert<Q, ROWL>(mem, st, j, key, KEY_NONE, ex);
                        m_deq = key < m_deq ? key : m_deq;
                        const uint32_t x = first_u32(__builtin_elementwise_add_sat(key, ex) - 1);
                        horizon = x < horizon ? x : horizon;
                    }
                }
                PROF_MARK(7)
                if (ei + 1 >= out_end) break;
                next_edge(ei + 1);
                if (EARLY) ed = load_edge(lit, ei + 1);
            }
            // (chains: code that inputs without parameters do not run is laid out behind the rest -- 64 chains x 16 changes with unequal links on the
            // AlexNet-shaped graph 3.42 -> 3.32 ms, and 0.5 % less with parameters; in batches it costs 1 % with parameters and gives nothing)
            if (SimX::kExt && (RECORD ? __builtin_expect(S.sync, 0) : S.sync)) {
                // parameter synchronisation (see run_events): a replica that has finished sends its gradient of the shard
                // to the owner's device, queued on its link row after the op's transfers to consumers
                const uint32_t pbytes = lite.param_bytes, now = (kmin + d) >> 1;      // (parts that share a link row are released at one time)
                if (pbytes) {
                    const OpCfg cfull = m.cfg(i);
                    const uint32_t pdims = m.T.ops[i].param_dims;
                    const uint32_t digits = part_digits(cfull, lane, m.magic_v);
                    uint32_t owner = 0, shards = 1;
#pragma unroll
                    for (int dd = 0; dd < 4; dd++) {
                        const bool indexes = (pdims >> dd) & 1u;
                        owner = owner * cfull.deg[dd] + (indexes ? (digits >> (8 * dd)) & 0xffu : 0u);
                        if (indexes) shards *= cfull.deg[dd];
                    }
                    const uint32_t shard_bytes = (pbytes - 1) / shards + 1;
                    const uint32_t dev_o = m.template device_of_part<REG>(i, ci, in_mask ? owner : 0u);
                    const bool act = in_mask && owner != lane && dev_o != dev_p;
                    if (ballot(act)) {
                        const uint32_t node_o = m.node_of(dev_o);
                        const uint32_t local_o = m.local_of(dev_o, node_o);
                        const bool same_node = node_o == node_p;
                        const uint32_t row_i = same_node ? dev_p * G + local_o : S.n_nodes * G * G + node_p * S.n_nodes + node_o;
                        uint32_t bw = same_node ? S.bw_intra : S.bw_inter, m_bw = same_node ? S.m_bw_intra : S.m_bw_inter;
                        uint32_t lat = same_node ? S.lat_intra : S.lat_inter;
                        if (S.link_table && act && same_node) {
                            const uint4 e = m.links[m.local_of(dev_p, node_p) * G + local_o];
                            bw = e.x; m_bw = e.y; lat = e.z;
                        }
                        if (S.node_table && act && !same_node) {
                            const uint4 e = m.node_links[node_p * S.n_nodes + node_o];
                            bw = e.x; m_bw = e.y; lat = e.z;
                        }
                        // (parameters may be larger than any tensor: the time of one transfer may take more than 32 bits)
                        const uint32_t send = ceil_div_u32(shard_bytes, bw, m_bw);
                        T ns;
                        if constexpr (L64) ns = (u64)send + lat;
                        else ns = __builtin_elementwise_add_sat(send, lat);
                        const u64 act_m = ballot(act);
                        if constexpr (L64) {
                            const u64 end = fifo_commit(act, act ? row_i : 0u, ns, st.E + now, true, WaveLds{mem.lrow64, nullptr, nullptr, mem.tag});
                            if (act) latest_hi = (uint32_t)(end >> 32) > latest_hi ? (uint32_t)(end >> 32) : latest_hi;
                        } else {
                            const uint32_t end = fifo_links(act, act ? row_i : 0u, ns, now, true, mem);
                            const uint32_t hi = (uint32_t)((st.E + end) >> 32);
                            if (act) { latest_link = end > latest_link ? end : latest_link; latest_hi = hi > latest_hi ? hi : latest_hi; }
                        }
                        if (STATS) {
                            cnt.n_comm += __popcll(act_m);
                            if (act) cnt.sum_comm_ns += ns;
                        }
                    }
                }
            }
            if (in_mask) {
                k0 = W_NONE;
                words[(size_t)i * ROWL + lane] = k0;
            }
            found(mask);
            // ---- the op's next event
            const uint32_t nd = part_min_u32<ROWL>(in_mask ? KEY_NONE : d);
            const uint32_t nk = next_key(kmin, nd);
            const bool me = lanes_of(at);
            q.kr = me ? nk : q.kr;
            if (Q == Q_SLOT) q.op = me && (q.kd & q.kr) == KEY_NONE ? NO_OP : q.op;
            m_rel = nk < other_key ? nk : other_key;
        }
        if (Q == Q_SLOT && q.n_spill) { m_deq = wave_min_u32(q.kd); m_rel = wave_min_u32(q.kr); }        // (what came up may have gone to the spill list)
        PROF_MARK(7)
    }
    PROF_STORE(cnt)
    if (beyond_32()) return RESULT_RETRY;
    if (ballot(latest_hi >= (uint32_t)(TIME_LIMIT >> 32))) return RESULT_OVERFLOW;
    if (left < -1 || (left < 0 && max_steps == 0)) { cnt.exit_code = 2; return RESULT_INTERNAL; }
    return 0;
}

}  // namespace ffsim

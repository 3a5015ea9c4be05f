// Replay kernels: one wavefront of 64 lanes replays one trace under one policy
// (a workgroup is one wavefront, or two that share nothing).  All allocator state of the trace lives in that wave's LDS
// and registers; scalar state (counters, byte totals) stays wave-uniform so the
// compiler keeps it in SGPRs.  Control flow is wave-uniform throughout: the 64
// lanes only ever split up to scan / shift / mark the pool arrays in parallel.
//
// A wave replays alone on its SIMD most of the time, so an event costs
//   4 cycles x instructions issued  +  ~130 cycles x dependent LDS round trips.
// The data layout below is chosen to keep both small on the two hot paths
// (an exact hit on a cached block, and a free): first search level in
// registers, slot table in registers, per-event results parked in lane j of
// four registers and digested once per tile of 64 events.
//
// Policies (GMLake, arXiv 2401.08156): the splitting caching allocator of
// Sec. 2.2 and the stitching allocator of Sec. 3 and Sec. 4.1 (Algorithm 1).
#pragma once
#include <type_traits>
#include "wave_ops.hpp"
#include "replay_plan.hpp"

enum { C_FREE = 0, C_EXACT = 1, C_SPLIT = 2, C_STITCH = 3, C_GROW = 4, C_OOM = 5, C_FREE_NOOP = 6, C_INVALID = 15 };
enum : u32 { B_SMALL = 1u << 4, B_SBLOCK = 1u << 5, B_6 = 1u << 6, B_7 = 1u << 7 };
enum { SLOT_UNBOUND = 0u, SLOT_OOM = 0xFFFFFFFFu };
enum { KIND_SMALL = 0u, KIND_PBLOCK = 1u, KIND_SBLOCK = 2u };
#define NONE32 0xFFFFFFFFu
#define WIT_NONE 32u            // a list entry with an empty mask (first bit 1, last bit 0 of word 0): "no witness"
#define ENT_WORD(e) ((e) >> 12)

// Scalars of one trace that live in LDS (stitching kernel): index k is the u32 at lds[4 k].  The
// first SC_STATE_COUNT are state that only the rare paths need (read when they start, written back
// when they end); the counters after them are only ever updated in place.
enum {
    SC_TOP, SC_LIVE, SC_NEXT_SID,                       // arena top, live list entries, next creation number
    SC_NP_ALL,                                          // fine-grained variant: pBlocks of any size
    SC_STATE_COUNT,
    SC_N_SPLIT = SC_STATE_COUNT, SC_N_CREATED, SC_N_EVICTED, SC_FIRST_OOM, SC_STATUS, SC_OVF_EVENT, SC_STOP,
    SC_HW_PBLOCKS, SC_HW_SBLOCKS, SC_HW_MEMBERS, SC_HW_RUNS, SC_HW_MULTI,
    SC_COUNT
};

// Event counters and high-water marks of one (trace, policy), addressed by the SC_* indices.
// Two holders with the same interface: registers (splitting kernel, everything inline) and the
// LDS scalars (rare paths of the stitching kernel: updated in place, nothing to load or store).
struct AcctRegs {
    u32 f[SC_COUNT];
    bool stop;
    DI void init()
    {
#pragma unroll
        for (u32 k = 0; k < SC_COUNT; k++) f[k] = 0;
        f[SC_FIRST_OOM] = f[SC_OVF_EVENT] = NONE32;
        stop = false;
    }
    DI void add(u32 k, u32 x) { f[k] += x; }
    DI void peak(u32 k, u32 v) { f[k] = max(f[k], v); }
    // An engine table is too small for this trace: stop replaying it.
    DI void overflow(u32 ev, u32 which)
    {
        f[SC_STATUS] |= VMS_ST_TABLE_OVERFLOW | which;
        if (f[SC_OVF_EVENT] == NONE32) f[SC_OVF_EVENT] = ev;
        stop = true;
    }
};

struct AcctLds {
    u32 *sc;
    u32 *idle;                  // 64 spare words: what the lanes other than lane 0 aim at
    // LDS atomics without a result: nothing to wait for.  Lane 0 updates the scalar, the other lanes
    // a spare word each (no lane is switched off, no two lanes meet at one address)
    DI void add(u32 k, u32 x) { atomicAdd(lane_id() == 0 ? &sc[k] : &idle[lane_id()], x); }
    DI void peak(u32 k, u32 v) { atomicMax(lane_id() == 0 ? &sc[k] : &idle[lane_id()], v); }
    DI void overflow(u32 ev, u32 which)
    {
        st_one(sc, (u32)SC_STATUS, ld_uni(sc, (u32)SC_STATUS) | VMS_ST_TABLE_OVERFLOW | which);
        st_one(sc, (u32)SC_OVF_EVENT, min(ld_uni(sc, (u32)SC_OVF_EVENT), ev));
        st_one(sc, (u32)SC_STOP, 1u);
        wave_sync();
    }
};

// ---------------------------------------------------------------------------
// Slot table: what each handle of the trace currently holds.
//   req  request size in units; 0 = unbound; 0xFFFFFFFF = its ALLOC hit OOM
//   a    splitting pools: the block's `at` (see SplitPool); pBlock: first chunk; sBlock: creation number
//   b    kind | chunks held << 2 (stitching policy only)
//   c    sBlock: where its list is (flat variant: offset << 16 | entries; fine-grained: its place)
// An event asks at() where its slot's record is (readable with get_*() until the event ends) and ends in one
// of free_done(), alloc_done(), failed() and not_done(), which also note what the decision word and the totals
// of the event are made of; tile_end() hands these over once per 64 events.
// With at most 64 slots (SLOTS_IN_REGS) the table is four registers, slot s in lane s.  Else a tile of events
// works on records in registers: lane j takes a copy of its event's record when the tile begins, keeps what the
// event makes of it, and knows the last lane before it with the same slot (`prev`), whose record is the current
// one then; the last event of each slot puts its record back when the tile ends.  So an event never waits for
// the table, and stores nothing; per event the look-ups cost three dependent LDS round trips and up to seven
// stores before (alone: the splitting kernel on LoRA 2048x20000 7.25 -> 6.18 ms, on one random trace 0.637 ->
// 0.529; the stitching kernel on ZeRO-3 1280x20000 13.4 -> 12.5, on LoRA 4096x50000 62 -> 58).
// The table itself is asked once per 64 events, so it need not be near: it is in global memory (SLOTS_IN_MEM),
// one record of 16 bytes (splitting policy: 8) per slot, read with one load per lane that is on its way while
// the lanes find their `prev`.  The 10 to 20 KB of LDS it took per wavefront leave room for others (whole pass:
// LoRA 4096x50000 75 -> 55 ms, 1024x20000 12.5 -> 7.8, ZeRO-3 1280x20000 12.6 -> 12.2, the splitting policy alone on
// LoRA 2048x20000 6.69 -> 6.50).  Where that room is not needed it stays in LDS (SLOTS_IN_LDS): the flat variant is 1 to
// 2 % faster so.
// ---------------------------------------------------------------------------
template <int WHERE, bool VMS, class LIST>
struct SlotsT {
    static constexpr bool REGS = WHERE == SLOTS_IN_REGS, MEM = WHERE == SLOTS_IN_MEM;
    struct alignas(VMS ? 16 : 8) Rec {
        u32 w[VMS ? 4 : 2];
    };
    u32 req, a, b, c;           // the table (REGS), or the records of the tile's events
    u32 v_dlo, v_dhi, v_req, v_act;         // the events' decision words and what they added to the totals
    u32 *t_req, *t_a, *t_b;     // the table in LDS
    LIST *t_c;
    Rec *tab;                   // the table in global memory
    u32 n_slots;
    u32 prev, slot, old_req;    // per lane: see above; the slot; what req was when the tile began
    // slice: which slice of the launch's tables in global memory is this wavefront's
    DI void init(char *lds, const KParams &P, u32 slice)
    {
        req = a = b = c = 0;
        n_slots = P.max_slots;
        if constexpr (MEM) {
            tab = (Rec *)(P.mem + (size_t)slice * P.mem_stride);
            for (u32 i = lane_id(); i < n_slots; i += 64) tab[i] = Rec{};
            wave_sync();
        } else if constexpr (!REGS) {
            t_req = (u32 *)(lds + P.off_slot_req);
            t_a = (u32 *)(lds + P.off_slot_a);
            t_b = (u32 *)(lds + P.off_slot_b);
            t_c = (LIST *)(lds + P.off_slot_c);
            for (u32 i = lane_id(); i < n_slots; i += 64) {
                t_req[i] = SLOT_UNBOUND;
                t_a[i] = 0;
                if constexpr (VMS) {
                    t_b[i] = 0;
                    t_c[i] = 0;
                }
            }
            wave_sync();
        }
    }
    // ev_lo, ev_hi: the tile's event words; n of them exist.  An event whose slot does not exist becomes an
    // ALLOC of nothing: it is as invalid as that.
    DI void tile_begin(u32 &ev_lo, u32 &ev_hi, u32 n)
    {
        const u32 lane = lane_id();
        const bool exists = ev_hi < n_slots;
        ev_lo = exists ? ev_lo : 0u;
        if constexpr (REGS) ev_hi = exists ? ev_hi : 0u;
        v_dlo = v_dhi = v_req = v_act = 0;
        if constexpr (!REGS) {
            slot = lane < n && exists ? ev_hi : n_slots;
            const u32 i = min(slot, n_slots - 1);
            Rec r;
            if constexpr (MEM) r = tab[i];      // (on its way while `prev` is found)
            // the last lane before this one with the same slot: key is slot * 128 + lane, so key - key' - 1 is
            // below 63 exactly for the same slot in an earlier lane, and smallest for the last of those
            const u32 key = (slot << 7) | lane;
            // (written out it is 3 % of the splitting kernel; the stitching kernels are 2 % faster with a loop of
            // nine a step, which leaves them the scalar registers)
            constexpr int STEP = VMS ? 9 : 63;
            u32 d = NONE32;
#pragma unroll STEP
            for (u32 i = 0; i < 63; i++) d = min(d, key - 1 - from_lane(key, i));
            prev = d < 63 ? lane - 1 - d : lane;
            if constexpr (MEM) {
                req = r.w[0];
                a = r.w[1];
                if constexpr (VMS) {
                    b = r.w[2];
                    c = r.w[3];
                }
            } else {
                req = t_req[i];
                a = t_a[i];
                if constexpr (VMS) {
                    b = t_b[i];
                    c = t_c[i];
                }
            }
            old_req = req;
        }
    }
    DI u32 at(u32 ev_hi, u32 j) const { return from_lane(REGS ? ev_hi : prev, j); }
    DI u32 get_req(u32 at) const { return from_lane(req, at); }
    DI u32 get_a(u32 at) const { return from_lane(a, at); }
    DI u32 get_b(u32 at) const { return from_lane(b, at); }
    DI u32 get_c(u32 at) const { return from_lane(c, at); }
    // a FREE: the slot held r units, d units of memory
    DI void free_done(u32 j, u32 at, u32 dlo, u32 dhi, u32 r, u32 d)
    {
        if constexpr (REGS) {
            req = write_lane(req, SLOT_UNBOUND, at);
            if constexpr (VMS) write_lane4(v_dlo, v_dhi, v_req, v_act, dlo, dhi, 0u - r, 0u - d, j);
            else write_lane3(v_dlo, v_dhi, v_req, dlo, dhi, 0u - r, j);
        } else {
            write_lane2(v_dlo, req, dlo, SLOT_UNBOUND, j);
        }
        wave_sync();
    }
    // an ALLOC of r units that was given d units of memory
    DI void alloc_done(u32 j, u32 at, u32 dlo, u32 dhi, u32 r, u32 d, u32 va, u32 vb, u32 vc)
    {
        if constexpr (VMS) {
            if constexpr (REGS) {
                write_lane4(req, a, b, c, r, va, vb, vc, at);
                write_lane4(v_dlo, v_dhi, v_req, v_act, dlo, dhi, r, d, j);
            } else {
                write_lane5(v_dlo, req, a, b, c, dlo, r, va, vb, vc, j);
            }
        } else {
            if constexpr (REGS) {
                write_lane2(req, a, r, va, at);
                write_lane3(v_dlo, v_dhi, v_req, dlo, dhi, r, j);
            } else {
                write_lane3(v_dlo, req, a, dlo, r, va, j);
            }
        }
        wave_sync();
    }
    // the slot is left with `r` as its req and nothing changes hands (out of memory, a FREE after that)
    DI void failed(u32 j, u32 at, u32 dlo, u32 r)
    {
        req = write_lane(req, r, REGS ? at : j);
        v_dlo = write_lane(v_dlo, dlo, j);
        wave_sync();
    }
    // an invalid event: the record stays as it is
    DI void not_done(u32 j, u32 at)
    {
        if constexpr (!REGS) {
            write_lane2(req, a, get_req(at), get_a(at), j);
            if constexpr (VMS) write_lane2(b, c, get_b(at), get_c(at), j);
        }
        v_dlo = write_lane(v_dlo, (u32)C_INVALID, j);
        wave_sync();
    }
    // the first `done` events have ended: v_dhi, v_req, v_act become theirs, and the table is up to date.
    // place(a): the address of a block of a splitting pool; shift: log2 of a chunk in units
    template <class Place>
    DI void tile_end(u32 done, u32 shift, Place place)
    {
        if constexpr (!REGS) {
            const u32 lane = lane_id(), code = v_dlo & 15;
            const bool freed = lane < done && code == C_FREE, given = lane < done && code - C_EXACT <= C_GROW - C_EXACT;
            // what a FREE let go of is the record it found: its own lane's or that of the event before it
            const u32 pa = other_lane(a, prev), pr = other_lane(req, prev);
            const u32 fa = freed ? pa : a, fr = freed ? (prev == lane ? old_req : pr) : req;
            u32 held = fr;
            bool whole = false;                                 // held in chunks
            if constexpr (VMS) {
                const u32 pb = other_lane(b, prev), fb = freed ? pb : b;
                whole = (fb & 3) != KIND_SMALL;
                held = whole ? (fb >> 2) << shift : fr;
            }
            const u32 sign = freed ? NONE32 : 0u, some = freed || given ? NONE32 : 0u;
            v_dhi = (VMS && whole ? fa : place(fa)) & some;
            v_req = ((fr ^ sign) - sign) & some;
            v_act = ((held ^ sign) - sign) & some;
            // a lane that a later one names as `prev` is not the last of its slot.  (No lane names lane 63: what
            // arrives there is from the lanes that name none)
            const u32 later = to_lane(prev != lane ? 1u : 0u, prev != lane ? prev : 63u);
            if (slot < n_slots && (lane == 63 || later == 0)) {
                if constexpr (MEM) {
                    Rec r;
                    r.w[0] = req;
                    r.w[1] = a;
                    if constexpr (VMS) {
                        r.w[2] = b;
                        r.w[3] = c;
                    }
                    tab[slot] = r;
                } else {
                    t_req[slot] = req;
                    t_a[slot] = a;
                    if constexpr (VMS) {
                        t_b[slot] = b;
                        t_c[slot] = (LIST)c;
                    }
                }
            }
            wave_sync();
        }
    }
    // The lists of the held sBlocks have moved: moved_to(a, b, c) is the place now of the list a record
    // describes (called by every lane, whatever its record holds).  Records that are no longer current get
    // something as well, which nothing reads.
    template <class MovedTo>
    DI void relist(MovedTo moved_to)
    {
        const u32 to = moved_to(a, b, c);
        c = req + 1u > 1u && (b & 3) == KIND_SBLOCK ? to : c;
        if constexpr (!REGS) {
            for (u32 base = 0; base < n_slots; base += 64) {
                const u32 i = min(base + lane_id(), n_slots - 1);
                u32 r, ta, tb, tc;
                if constexpr (MEM) {
                    const Rec x = tab[i];
                    r = x.w[0];
                    ta = x.w[1];
                    tb = x.w[2];
                    tc = x.w[3];
                } else {
                    r = t_req[i];
                    ta = t_a[i];
                    tb = t_b[i];
                    tc = t_c[i];
                }
                const u32 now = moved_to(ta, tb, tc);
                wave_lockstep();
                const u32 place = r + 1u > 1u && (tb & 3) == KIND_SBLOCK ? now : tc;
                if constexpr (MEM) tab[i].w[3] = place;
                else t_c[i] = (LIST)place;
            }
            wave_sync();
        }
    }
};

// ---------------------------------------------------------------------------
// Splitting pool (Sec. 2.2).  Only the inactive blocks are stored; an active block's place and size
// travel with the slot that holds it.
//
// They live in registers: place t * 64 + l of the array is at[t], h[t] of lane l: where the block is and
// its size; 0 in both = empty place.  The order of the array means nothing (best fit and the neighbour
// searches look at every block), so a block that leaves just zeroes its place and a new one takes the
// first empty place.  No LDS access at all: a request is compares, one or two wave-wide minima and a few
// lane selects.
// A table of more than 64 * TILES blocks has the rest in LDS: the tail, used only while every place in
// the registers is taken (most tables are sized for more blocks than their traces ever hold at once: the
// default holds 512, the random traces 63 to 115, the LoRA streams 250 to 300).  An earlier version kept
// every pool of a table of more than 320 (the small-request pool: 192) blocks in LDS as a whole and searched
// it four tiles at a time (the splitting kernel alone: one random trace 1.067 -> 0.637 ms, LoRA 64x20000 with
// a table of 1,024 blocks 12.05 -> 6.34; the stitching kernel, which had both kinds of pool in its code:
// random 1.567 -> 1.093, ZeRO-3 1280x20000 15.8 -> 13.7, LoRA 4096x50000 74.2 -> 63.6).  A kernel that can
// do without the tail is its own variant: with it the splitting kernel takes 7.75 instead of 7.25 ms on
// LoRA 2048x20000.
// at = address << 1 | segment parity (1 for the first segment, then 0, 1, ...).  Segments follow each
// other without a gap, so only neighbouring ones could touch, and theirs differ in the low bit: block x
// ends where y starts, in the same segment, iff at_x + 2 h_x == at_y.  One compare per side and place
// answers what took two segment flags their own tests, masks and merging before (the splitting kernel
// alone: LoRA 2048x20000 8.74 -> 7.22 ms, recomputation 1024x20000 6.33 -> 5.26; the stitching kernel on
// LoRA 4096x50000, most of whose requests are small, 80.2 -> 74.2 ms).  No block is at 0 (the block at
// address 0 has parity 1), so an empty place matches nothing.
// What bounds it is the chain of one event (two wavefronts per SIMD issue an instruction every nine
// cycles), so the halves are searched apart, all tiles side by side: 64-bit minima went through the
// tiles one after the other, compare, select, compare (the splitting kernel alone on LoRA streams, five
// tiles: 2048x20000 9.57 -> 8.84 ms, 4096x50000 35.6 -> 31.9 ms).
template <u32 TILES, bool TAIL>
struct SplitPool {
    u32 at[TILES], h[TILES];
    u64 *fl;                    // the tail: h << 32 | at
    u32 n, n_tail, cap, res, parity;        // n: blocks, those in the tail among them
    u32 hw;                     // the most blocks held at once (cuts and merges are counted off the decisions)
    DI void init(char *lds, const KParams &P)
    {
#pragma unroll
        for (u32 t = 0; t < TILES; t++) at[t] = h[t] = 0;
        fl = (u64 *)(lds + P.off_fl);
        n = n_tail = hw = 0;
        cap = P.cap_free;
        res = 0;
        parity = 1;
    }
    DI u32 reserved() const { return res; }
    DI u32 most() const { return hw; }
    static DI u32 addr(u32 ref) { return ref >> 1; }            // ref: `at` of a block, what its slot keeps
    // the block at `from` (one place holds it) takes a new place and size
    DI void swap_block(u32 from, u32 to, u32 size)
    {
#pragma unroll
        for (u32 q = 0; q < TILES; q++) {
            const bool here = at[q] == from;
            at[q] = here ? to : at[q];
            h[q] = here ? size : h[q];
        }
    }
    DI void place(u32 to, u32 size)             // into an empty place of the registers (there is one)
    {
        bool any = false;
#pragma unroll
        for (u32 q = 0; q < TILES; q++) any = any || h[q] == 0;
        bool todo = lane_id() == first_lane(ballot(any));       // the first lane with room, its first empty place
#pragma unroll
        for (u32 q = 0; q < TILES; q++) {
            const bool here = todo && h[q] == 0;
            at[q] = here ? to : at[q];
            h[q] = here ? size : h[q];
            todo = todo && !here;
        }
    }
    DI void insert(u32 to, u32 size)            // (n < cap)
    {
        if (!TAIL || LIKELY(n - n_tail < 64 * TILES)) place(to, size);
        else {
            st_one(fl, n_tail++, ((u64)size << 32) | to);
            wave_sync();
        }
        n++;
        hw = max(hw, n);
    }
    // block i of the tail leaves, the last one takes its place; where block `other` is now
    DI u32 tail_remove(u32 i, u32 other)
    {
        st_one(fl, i, ld_uni(fl, --n_tail));
        wave_sync();
        n--;
        return other == n_tail ? i : other;
    }
    // The tail's part of a request: a block there that fits better than the best in the registers (which
    // leaves `rest`) changes places with the one in this wavefront's first place, and the search is repeated
    DI bool fetch_from_tail(u32 size, u32 rest, const u32 (&d)[TILES])
    {
        u32 bd = NONE32, ba = NONE32, bi = 0;
        for (u32 base = 0; base < n_tail; base += 64) {
            const u32 i = base + lane_id();
            const u64 k = fl[i < n_tail ? i : 0u];
            const u32 x = i < n_tail ? (u32)(k >> 32) - size : NONE32;
            const bool better = x < bd || (x == bd && (u32)k < ba);
            bd = better ? x : bd;
            ba = better ? (u32)k : ba;
            bi = better ? i : bi;
        }
        const u32 left = wave_min_u32(bd);
        if ((int)left < 0 || left > rest) return false;
        const u32 ref = wave_min_u32(bd == left ? ba : NONE32);
        u32 c = NONE32;
#pragma unroll
        for (u32 t = 0; t < TILES; t++) c = min(c, d[t] == left ? at[t] : NONE32);
        if (left == rest && wave_min_u32(c) < ref) return false;        // of equal sizes the lowest address goes
        const u32 idx = from_lane(bi, first_lane(ballot(bd == left && ba == ref)));
        const u64 out = ((u64)from_lane(h[0], 0) << 32) | from_lane(at[0], 0);
        h[0] = write_lane(h[0], left + size, 0);
        at[0] = write_lane(at[0], ref, 0);
        if (out) st_one(fl, idx, out);
        else st_one(fl, idx, ld_uni(fl, --n_tail));             // that place was empty
        wave_sync();
        return true;
    }
    // The tail's part of a release: neighbours that are there leave it and are taken into the block
    DI void absorb_from_tail(u32 &ref, u32 &size, bool &ml, bool &mr)
    {
        u32 li = NONE32, ri = NONE32;
        for (u32 base = 0; base < n_tail; base += 64) {
            const u32 i = base + lane_id();
            const u64 k = fl[i < n_tail ? i : 0u];
            const u64 mL = ballot(i < n_tail && (u32)k + 2 * (u32)(k >> 32) == ref), mR = ballot(i < n_tail && (u32)k == ref + 2 * size);
            if (mL) li = base + first_lane(mL);
            if (mR) ri = base + first_lane(mR);
        }
        ml = li != NONE32;
        mr = ri != NONE32;
        if (mr) {
            size += (u32)(ld_uni(fl, ri) >> 32);
            li = tail_remove(ri, li);
        }
        if (ml) {
            const u64 k = ld_uni(fl, li);
            ref = (u32)k;
            size += (u32)(k >> 32);
            tail_remove(li, 0u);
        }
    }
    // Every outcome ends in a call of its own: done(code, ref, split) once the request is decided
    // (code C_OOM: it failed) or ovf() if the table is full.  Results handed back through one return
    // would meet again in flags that the caller has to test, event after event.
    template <class AcctT, class Done, class Ovf>
    DI void alloc(u32 size, u32 seg, bool may_grow, AcctT &A, u32 ev, Done done, Ovf ovf)
    {
        // step 1: best fit = smallest size not below the request.  Sizes have 31 bits, so what a block
        // has beyond the request has bit 31 set exactly if the block is too small (or the place empty)
        u32 d[TILES], mine, rest;
        do {
            mine = NONE32;
#pragma unroll
            for (u32 t = 0; t < TILES; t++) {
                d[t] = h[t] - size;
                mine = min(mine, d[t]);
            }
            rest = wave_min_u32(mine);
        } while (TAIL && UNLIKELY(n_tail != 0) && fetch_from_tail(size, rest, d));
        if (LIKELY((int)rest >= 0)) {
            u32 c = NONE32;                     // lowest address of that size in this lane
#pragma unroll
            for (u32 t = 0; t < TILES; t++) c = min(c, d[t] == rest ? at[t] : NONE32);
            const u64 m = ballot(mine == rest);
            const u32 ref = UNLIKELY(m & (m - 1)) ? wave_min_u32(c) : from_lane(c, first_lane(m));
            if (LIKELY(rest != 0)) {
                // step 2: cut off what is not needed; it stays cached as the right neighbour, in the
                // place the block had
                swap_block(ref, ref + 2 * size, rest);
                done((u32)C_SPLIT, ref, true);
                return;
            }
            swap_block(ref, 0u, 0u);
            n--;
            done((u32)C_EXACT, ref, false);
            return;
        }
        if (!may_grow) {
            done((u32)C_OOM, 0u, false);
            return;
        }
        const u32 ref = 2 * res + parity;       // "native allocation": a fresh segment
        res += seg;
        parity ^= 1;
        if (seg > size) {                       // the rest of a fresh segment
            if (n == cap) {
                A.overflow(ev, VMS_ST_OVF_FREE_BLOCKS);
                ovf();
                return;
            }
            insert(ref + 2 * size, seg - size);
            done((u32)C_GROW, ref, true);
            return;
        }
        done((u32)C_GROW, ref, false);
    }
    // steps 3 and 4: the block becomes inactive and absorbs inactive neighbours of its segment
    template <class AcctT, class Done, class Ovf>
    DI void release(u32 ref, u32 size, AcctT &A, u32 ev, Done done, Ovf ovf)
    {
        bool tl = false, tr = false;
        if (TAIL && UNLIKELY(n_tail != 0)) absorb_from_tail(ref, size, tl, tr);
        // at most one block ends where this one starts and at most one starts where it ends
        const u32 end = ref + 2 * size;
        bool l[TILES], r[TILES], any_l = false, any_r = false;
#pragma unroll
        for (u32 t = 0; t < TILES; t++) {
            l[t] = at[t] + 2 * h[t] == ref;
            r[t] = at[t] == end;
            any_l = any_l || l[t];
            any_r = any_r || r[t];
        }
        const u64 mL = ballot(any_l), mR = ballot(any_r);
        const bool ml = mL != 0, mr = mR != 0;
        if (mr) {
            u32 x = 0;                          // the right neighbour's size
#pragma unroll
            for (u32 t = 0; t < TILES; t++) x = r[t] ? h[t] : x;
            size += from_lane(x, first_lane(mR));
            if (UNLIKELY(ml)) {
                // the merged block takes the left neighbour's place
#pragma unroll
                for (u32 t = 0; t < TILES; t++) {
                    at[t] = r[t] ? 0u : at[t];
                    h[t] = r[t] ? 0u : (l[t] ? h[t] + size : h[t]);
                }
                n--;
            } else {
#pragma unroll
                for (u32 t = 0; t < TILES; t++) {
                    at[t] = r[t] ? ref : at[t];
                    h[t] = r[t] ? size : h[t];
                }
            }
        } else if (UNLIKELY(ml)) {
#pragma unroll
            for (u32 t = 0; t < TILES; t++) h[t] = l[t] ? h[t] + size : h[t];
        } else {
            if (n == cap) {
                A.overflow(ev, VMS_ST_OVF_FREE_BLOCKS);
                ovf();
                return;
            }
            insert(ref, size);
        }
        done(ml || tl, mr || tr);
    }
};

// ---------------------------------------------------------------------------
// Virtual memory pool (Sec. 3.2) in LDS.
//   pool[]   every pBlock (active or not) as key  size << 32 | ~first_chunk, sorted descending:
//            pool order = size descending, then first chunk ascending.  It changes only when
//            Alloc creates or Split cuts a pBlock.
//   bmp[]    one bit per physical chunk: set while the pBlock owning it is active.  A pBlock is
//            inactive iff the bit of its first chunk is clear; an sBlock is inactive iff all bits
//            of all its chunk runs are clear (Sec. 3.2: one active pBlock makes the sBlock active).
//            Handing out / releasing any block is therefore only bit-range work.
//   skey[]   sBlocks as key  size << 32 | ~creation_number, sorted descending (size descending,
//            then older first), with smeta[] = arena offset << 16 | entries, sstamp[] = last use,
//            swit[] = a "witness": the list entry that was seen active last (or WIT_NONE).  While the
//            witness is still active the sBlock is known to be active after one bitmap read.
//   arena[]  chunk runs of all cached sBlocks, bump-allocated, cut at bitmap word boundaries:
//            one 32-bit entry  word << 12 | first bit << 5 | last bit  per range of consecutive
//            chunks inside one bitmap word (bits 10-11 number the ranges of one word; unused).
//            Testing, setting or clearing an sBlock is one step over its entries, one lane per
//            entry: the test reads the words, set and clear are LDS atomics without a result, so
//            several ranges of one word need no ordering and a FREE waits for nothing but its list.
//   tmp[]    scratch bitmap of the same size as bmp[] (+ 64 spare words), zero between uses: a new list is OR-ed
//            together here and read back word by word, which merges touching runs.
//            Compacted through a global-memory buffer when full.
//   pp, sp   first level of the rank searches in pool[] and skey[], held in registers.
// ---------------------------------------------------------------------------
struct VmsT {
    typedef u32 meta_t;
    u64 *pool;
    u32 *bmp;
    u64 *skey;
    meta_t *smeta;
    u32 *sstamp, *swit, *tmp;
    u32 *idle;                  // 64 spare words behind tmp[]: targets of lanes that have nothing to update
    u32 *arena, *bounce;
    u32 np, ns, n_chunks, top, live_ent, next_sid, clock;
    u32 e_skip;                 // a list entry with an empty mask on the spare word behind the bitmap
    Probe pp, sp;
    static DI meta_t pack(u32 off, u32 cnt) { return (off << 16) | cnt; }
    static DI u32 off(meta_t m) { return m >> 16; }
    static DI u32 cnt(meta_t m) { return m & 0xFFFFu; }
    static DI meta_t pinm(meta_t m) { return pin(m); }      // pin() for a list place
};

DI u32 from_lane_any(u32 v, u32 l) { return from_lane(v, l); }
DI u64 from_lane_any(u64 v, u32 l) { return from_lane64(v, l); }

// bits of one list entry inside its bitmap word
DI u32 emask(u32 e) { return (2u << (e & 31)) - (1u << ((e >> 5) & 31)); }

DI u32 run_words(u32 start, u32 len) { return ((start + len - 1) >> 5) - (start >> 5) + 1; }

// entry q of the run [start, start + len)
DI u32 run_entry(u32 start, u32 len, u32 q)
{
    const u32 w0 = start >> 5, endm1 = start + len - 1, w = w0 + q;
    const u32 lo = q == 0 ? (start & 31) : 0u;
    const u32 hi = w == (endm1 >> 5) ? (endm1 & 31) : 31u;
    return (w << 12) | (lo << 5) | hi;
}

// write the entries of one run (wave-uniform arguments) at arena[at..]; returns how many
DI u32 arena_put(VmsT &V, u32 at, u32 start, u32 len)
{
    const u32 n = run_words(start, len);
    for (u32 qb = 0; qb < n; qb += 64) {
        // lanes past the run write its last entry again
        const u32 q = min(qb + lane_id(), n - 1);
        V.arena[at + q] = run_entry(start, len, q);
    }
    wave_sync();
    return n;
}

DI u32 word_mask(u32 w, u32 start, u32 end)    // bits of word w inside [start, end)
{
    u32 b0 = (w == (start >> 5)) ? (start & 31) : 0u;
    u32 b1 = (w == ((end - 1) >> 5)) ? ((end - 1) & 31) + 1u : 32u;
    u32 n = b1 - b0;
    return (n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u)) << b0;
}

// one run, the lanes take one bitmap word each; lanes past its end rewrite the spare word behind
// the bitmap (no divergent branch)
DI void bmp_fill(u32 *bmp, u32 spare, u32 start, u32 len, bool set)
{
    const u32 end = start + len, w0 = start >> 5, w1 = (end - 1) >> 5;
    for (u32 wb = w0; wb <= w1; wb += 64) {
        const u32 w = wb + lane_id();
        const bool in = w <= w1;
        const u32 mw = pin(word_mask(w, start, end));          // computed by every lane: no branch
        const u32 m = in ? mw : 0u, wi = in ? w : spare;
        const u32 old = pin(bmp[wi]);
        bmp[wi] = set ? (old | m) : (old & ~m);
    }
    wave_sync();
}

// One tile of list entries, one lane per entry (e, if live): their bits are set or cleared with LDS
// atomics that return nothing, so entries that share a bitmap word need no ordering and the wave
// does not wait for the result.  Lanes without an entry OR a zero into a spare word of their own.
DI void entries_apply(const VmsT &V, u32 e, bool live, bool set)
{
    u32 *t = live ? &V.bmp[ENT_WORD(e)] : &V.idle[lane_id()];
    const u32 m = live ? emask(e) : 0u;
    if (set) atomicOr(t, m);
    else atomicAnd(t, ~m);
}

// all entries of one sBlock
DI void bmp_fill_entries(const VmsT &V, u32 off, u32 cnt, bool set)
{
    for (u32 rb = 0; rb < cnt; rb += 64) {
        const u32 r = rb + lane_id();
        const u32 e = V.arena[off + (r < cnt ? r : 0u)];
        entries_apply(V, e, r < cnt, set);
    }
    wave_sync();
}

// A new list is collected in tmp[]: mark one run per lane (lanes with len == 0 mark nothing;
// wmin / wmax: per-lane range of the bitmap words touched so far) ...
DI void list_mark(const VmsT &V, u32 start, u32 len, u32 &wmin, u32 &wmax)
{
    const u32 end = start + len;
    const u32 w0 = len ? start >> 5 : NONE32, w1 = len ? (end - 1) >> 5 : 0u;
    for (u32 q = 0; ballot(len && w0 + q <= w1); q++) {
        // lanes with nothing left OR a zero into a word of their own
        const bool in = len && w0 + q <= w1;
        const u32 mw = pin(word_mask(w0 + q, start, end));
        atomicOr(in ? &V.tmp[w0 + q] : &V.idle[lane_id()], in ? mw : 0u);
    }
    wmin = min(wmin, w0);
    wmax = max(wmax, w1);
}

// ... and read back as entries at arena[at..], one per range of consecutive chunks inside a word
// (touching runs have merged), leaving tmp[] zero.  Returns the number of entries.
DI u32 list_extract(const VmsT &V, u32 wmin, u32 wmax, u32 at, u32 spare)
{
    u32 cnt = 0;
    for (u32 wb = wmin; wb <= wmax; wb += 64) {
        const u32 w = min(wb + lane_id(), wmax);     // lanes past the end: the last word again, taken as empty
        const u32 mw = pin(V.tmp[w]);
        u32 m = wb + lane_id() <= wmax ? mw : 0u;
        wave_sync();
        V.tmp[w] = 0;
        const u32 nr = (u32)__builtin_popcount(m & ~(m << 1));      // ranges start where a set bit follows a clear one
        u32 tot;
        const u32 incl = wave_scan_add(nr, &tot);
        const u32 o = at + cnt + incl - nr;
        for (u32 r = 0; ballot(m != 0); r++) {
            // a lane whose word is used up writes into the spare places behind the arena
            const bool some = m != 0;
            const u32 mm = some ? m : 1u;
            const u32 lo = (u32)__builtin_ctz(mm);
            const u32 rest = ~(mm >> lo);
            const u32 len = rest ? (u32)__builtin_ctz(rest) : 32u;
            const u32 hi = lo + len - 1;
            V.arena[some ? o + r : spare + lane_id()] = (w << 12) | ((r < 3 ? r : 3u) << 10) | (lo << 5) | hi;
            m = some ? m & ~((2u << hi) - (1u << lo)) : 0u;
        }
        cnt += tot;
    }
    wave_sync();
    return cnt;
}

template <class AcctT>
DI void pool_insert(VmsT &V, u32 size, u32 start, AcctT &A)
{
    u64 key = ((u64)size << 32) | (u32)~start;
    u32 pos = rank_desc(V.pool, V.np, key);
    shift_up(V.pool, pos, V.np);
    st_one(V.pool, pos, key);
    V.np++;
    A.peak(SC_HW_PBLOCKS, V.np);
    wave_sync();
}

// Split (Sec. 3.3.1): the pBlock at pool[idx] is replaced by its two pieces, both smaller and
// therefore further down in pool order.  Only the keys between the old place and the new
// places move: down by one up to the larger piece, up by one after the smaller piece.
template <class AcctT>
DI void pool_cut(VmsT &V, u32 idx, u32 size_a, u32 start_a, u32 size_b, u32 start_b, AcctT &A)
{
    u64 k1 = ((u64)size_a << 32) | (u32)~start_a, k2 = ((u64)size_b << 32) | (u32)~start_b;
    if (k1 < k2) {
        const u64 t = k1;
        k1 = k2;
        k2 = t;
    }
    u32 r1, r2;                                 // ranks among the old keys (the cut block counts in both)
    rank_desc2(V.pool, V.np, k1, k2, &r1, &r2);
    shift_down(V.pool, idx, r1);                // pool[idx+1 .. r1) -> pool[idx .. r1-1)
    shift_up(V.pool, r2, V.np);                 // pool[r2 .. np) -> pool[r2+1 .. np+1)
    st_one(V.pool, r1 - 1, k1);
    st_one(V.pool, r2, k2);
    V.np++;
    A.peak(SC_HW_PBLOCKS, V.np);
    wave_sync();
}

// skey[], smeta[], sstamp[] and swit[] move together: entries [pos, n) one place up (highest
// tile first) or entries (pos, n) one place down (lowest tile first), one LDS round trip per tile
DI void spool_shift_up(VmsT &V, u32 pos, u32 n)
{
    for (u32 hi = n; hi > pos;) {
        const u32 lo = hi - pos > 64 ? hi - 64 : pos;
        const u32 i = lo + lane_id(), src = i < hi ? i : i + 1;   // lanes above the part that moves: see shift_up
        const u64 k = V.skey[src];
        const auto m = V.smeta[src];
        const u32 st = V.sstamp[src], w = V.swit[src];
        wave_lockstep();
        V.skey[i + 1] = k;
        V.smeta[i + 1] = m;
        V.sstamp[i + 1] = st;
        V.swit[i + 1] = w;
        wave_lockstep();
        hi = lo;
    }
    wave_sync();
}

DI void spool_shift_down(VmsT &V, u32 pos, u32 n)
{
    for (u32 lo = pos + 1; lo < n; lo += 64) {
        const u32 i = lo + lane_id(), dst = i < n ? i - 1 : i;   // lanes past the end: see shift_down
        const u64 k = V.skey[i];
        const auto m = V.smeta[i];
        const u32 st = V.sstamp[i], w = V.swit[i];
        wave_lockstep();
        V.skey[dst] = k;
        V.smeta[dst] = m;
        V.sstamp[dst] = st;
        V.swit[dst] = w;
        wave_lockstep();
    }
    wave_sync();
}

// Stitch: the only creator of sBlocks (Sec. 3.3.1).  The entries are already in the arena.
// Returns the position of the new sBlock in skey[].
template <class AcctT>
DI u32 spool_insert(VmsT &V, u32 size, u32 off, u32 cnt, AcctT &A, bool probe_valid)
{
    u32 id = V.next_sid++;
    u64 key = ((u64)size << 32) | (u32)~id;
    // probe_valid: skey[] has not changed since its first search level was put into registers
    u32 pos = probe_valid ? rank_fast<false>(V.sp, V.skey, V.ns, key) : rank_desc(V.skey, V.ns, key);
    spool_shift_up(V, pos, V.ns);
    st_one(V.skey, pos, key);
    st_one(V.smeta, pos, V.pack(off, cnt));
    st_one(V.sstamp, pos, ++V.clock);
    // every sBlock starts out active (it is handed out, or the first part of the block it records
    // is): its first entry is a valid witness from the end of this event on
    st_one(V.swit, pos, ld_uni(V.arena, off));
    V.ns++;
    V.live_ent += cnt;
    A.add(SC_N_CREATED, 1);
    wave_sync();
    return pos;
}

DI void spool_remove(VmsT &V, u32 idx)
{
    V.live_ent -= V.cnt(ld_uni(V.smeta, idx));
    spool_shift_down(V, idx, V.ns);
    V.ns--;
    st_one(V.skey, V.ns, (u64)0);               // zero keys follow the live ones (see rank_fast)
    wave_sync();
}

// Squeeze the entries of evicted sBlocks out of the arena: copy the live lists to the
// global buffer in sPool order, then back.  Slots holding an sBlock learn its new place.
template <class Slots>
DI void arena_compact(VmsT &V, Slots &S, const KParams &P)
{
    u32 top = 0;
    for (u32 s = 0; s < V.ns; s++) {
        auto meta = ld_uni(V.smeta, s);
        u32 off = V.off(meta), cnt = V.cnt(meta);
        for (u32 rb = 0; rb < cnt; rb += 64) {          // lanes past the end copy the last entry again
            const u32 r = min(rb + lane_id(), cnt - 1);
            V.bounce[top + r] = V.arena[off + r];
        }
        st_one(V.smeta, s, V.pack(top, cnt));
        S.moved((u32)meta, (u32)V.pack(top, cnt), P);
        top += cnt;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");     // later reads are of other lanes' global writes
    wave_sync();
    for (u32 rb = 0; rb < top; rb += 64) {
        const u32 r = min(rb + lane_id(), top - 1);
        V.arena[r] = V.bounce[r];
    }
    V.top = top;
    wave_sync();
}

template <class Slots, class AcctT>
DI bool arena_reserve(VmsT &V, Slots &S, u32 need, const KParams &P, AcctT &A, u32 ev)
{
    if (UNLIKELY(V.top + need > P.cap_runs && V.live_ent < V.top)) arena_compact(V, S, P);
    if (UNLIKELY(V.top + need > P.cap_runs)) {
        A.overflow(ev, VMS_ST_OVF_RUNS);
        return false;
    }
    return true;
}

// Is any chunk of the list arena[off .. off + cnt) active?  All lanes work on the one list; if so,
// *witness receives an entry that was seen active.
DI bool list_busy(const VmsT &V, u32 off, u32 cnt, u32 *witness)
{
    for (u32 eb = 0; eb < cnt; eb += 64) {
        const u32 k = eb + lane_id();
        const u32 ek = pin(V.arena[off + (k < cnt ? k : 0u)]);
        const u32 e = k < cnt ? ek : V.e_skip;
        const u32 wk = pin(V.bmp[ENT_WORD(e)]);
        const u64 bm = ballot((wk & emask(e)) != 0);
        if (bm) {
            *witness = from_lane(e, first_lane(bm));
            return true;
        }
    }
    return false;
}

// StitchFree (Sec. 3.3.2, Sec. 4.2.3): while more sBlocks than the threshold are cached,
// release the least recently used one that is inactive.  One scan rules out, side by side, every
// sBlock whose witness is still active (three tiles at a time: all stamps and witnesses are loaded,
// then all witness words, two LDS round trips per 192 sBlocks) and leaves in every lane the two
// least recently used of the sBlocks it saw.  The oldest of all is tested with all lanes on its
// list and released if it is inactive; its lane falls back on its second and the search goes on
// without a new scan (a lane that runs out of its two forces one).  With a scan for each of the three sBlocks that
// a call of the threshold study releases, 64x20000 took 10.7 instead of 10.4 ms.
template <class AcctT>
DI bool stitch_free(VmsT &V, const KParams &P, AcctT &A)
{
    const u32 lane = lane_id();
    bool any = false, rescan = true;
    u32 b1 = NONE32, i1 = 0, b2 = NONE32, i2 = 0;
    bool spent = false;                         // this lane has given up its best once since the scan
    while (V.ns > P.spool_threshold) {
        if (rescan) {
            b1 = b2 = NONE32;
            i1 = i2 = 0;
            spent = false;
            for (u32 g = 0; g < V.ns; g += 192) {
                u32 st[3], wit[3], ww[3];
#pragma unroll
                for (u32 t = 0; t < 3; t++) {
                    const u32 i = g + t * 64 + lane, ic = i < V.ns ? i : 0u;
                    st[t] = V.sstamp[ic];
                    wit[t] = V.swit[ic];
                }
#pragma unroll
                for (u32 t = 0; t < 3; t++) ww[t] = pin(V.bmp[ENT_WORD(wit[t])]);
#pragma unroll
                for (u32 t = 0; t < 3; t++) {
                    const u32 i = g + t * 64 + lane;
                    const bool ok = (i < V.ns) & ((ww[t] & emask(wit[t])) == 0);
                    const u32 sv = ok ? st[t] : NONE32;
                    const bool lt1 = sv < b1, lt2 = sv < b2;
                    b2 = lt1 ? b1 : (lt2 ? sv : b2);
                    i2 = lt1 ? i1 : (lt2 ? i : i2);
                    b1 = lt1 ? sv : b1;
                    i1 = lt1 ? i : i1;
                }
            }
        }
        const u32 m = wave_min_u32(b1);
        if (m == NONE32) break;                 // everything cached is in use: the threshold stays exceeded
        const u32 owner = first_lane(ballot(b1 == m));
        const u32 c = from_lane(i1, owner);
        const auto meta = ld_uni(V.smeta, c);
        u32 witness;
        const bool busy = list_busy(V, V.off(meta), V.cnt(meta), &witness);
        // either way the lane falls back on its second
        rescan = from_lane(spent ? 1u : 0u, owner) != 0;
        const bool mine = lane == owner;
        b1 = mine ? b2 : b1;
        i1 = mine ? i2 : i1;
        b2 = mine ? NONE32 : b2;
        spent = spent || mine;
        if (busy) {
            st_one(V.swit, c, witness);         // active after all: remember where, look further
            wave_sync();
            continue;
        }
        spool_remove(V, c);
        i1 -= i1 > c ? 1u : 0u;                 // (the sBlocks behind it have moved down one place)
        i2 -= i2 > c ? 1u : 0u;
        A.add(SC_N_EVICTED, 1);
        any = true;
    }
    A.peak(SC_HW_SBLOCKS, V.ns);     // high-water marks as seen between events
    A.peak(SC_HW_RUNS, V.live_ent);
    return any;
}


// ---- S1 (Algorithm 1, first loop; Sec. 4.1 state S1), stitched blocks, oldest first.  The
// sBlocks of exactly bsize chunks start at the rank of (bsize, oldest) in skey[].  One lane per
// candidate reads its witness: a candidate whose witness is still active is out after two LDS
// round trips for the whole tile.  The others are tested in pool order with all lanes over the
// entries of one list; the first inactive one is handed out (ref = creation number, list = where
// its entries are).  This is the general route, from the tile that starts at `base`.
DI bool s1_sblock_from(VmsT &V, u32 bsize, u32 base, u32 &ref, u32 &list)
{
    const u32 lane = lane_id();
    for (;;) {
        // skey[] is followed by zero keys and swit[] by harmless entries: no index is clamped
        const u32 i = base + lane;
        const u64 key = V.skey[i];
        const u32 wit = V.swit[i];
        const auto meta = V.smeta[i];
        const u64 vm = ballot((u32)(key >> 32) == bsize);
        if (!vm) return false;
        const u32 wv = pin(V.bmp[ENT_WORD(wit)]);
        u64 unknown = vm & ~ballot((wv & emask(wit)) != 0);
        while (unknown) {
            const u32 l = first_lane(unknown);
            const auto m = from_lane_any(meta, l);
            const u32 off = V.off(m), cnt = V.cnt(m);
            // lanes past the end of the list hold an entry with an empty mask on the spare word
            const u32 e0 = pin(V.arena[off + lane]);
            u32 e = lane < cnt ? e0 : V.e_skip;
            const u32 word = pin(V.bmp[ENT_WORD(e)]);
            u64 bm = ballot((word & emask(e)) != 0);
            if (cnt > 64) {                     // long list: the rest of it, a tile at a time
                for (u32 eb = 64; eb < cnt && !bm; eb += 64) {
                    const u32 k = eb + lane;
                    const u32 ek = pin(V.arena[off + (k < cnt ? k : 0u)]);
                    e = k < cnt ? ek : V.e_skip;
                    const u32 wk = pin(V.bmp[ENT_WORD(e)]);
                    bm = ballot((wk & emask(e)) != 0);
                }
                if (!bm) {
                    bmp_fill_entries(V, off, cnt, true);
                    st_one(V.sstamp, base + l, ++V.clock);
                    ref = ~from_lane((u32)key, l);
                    list = (u32)m;
                    return true;
                }
            }
            if (!bm) {
                entries_apply(V, e, lane < cnt, true);      // inactive: hand it out
                st_one(V.sstamp, base + l, ++V.clock);
                ref = ~from_lane((u32)key, l);
                list = (u32)m;
                return true;
            }
            st_one(V.swit, base + l, from_lane(e, first_lane(bm)));
            unknown &= unknown - 1;
        }
        if (~vm) return false;                  // the run of equal sizes ended inside this tile
        base += 64;
    }
}

// (The usual route is written out in the replay loop and costs four dependent LDS round trips:
// the block of keys that the rank search reads, first level in registers, is taken as the first
// tile of candidates right away, together with their witnesses and list places; then the
// witnesses' bitmap words; then the list of the first candidate not ruled out; then the bitmap
// words of its entries.  Anything unusual - a long list, a candidate that turns out active, a run
// of equal sizes that leaves the tile - comes here.)

// ---- S1, primitive blocks: the first inactive pBlock of exactly bsize chunks in pool order.  As
// above, the block of the rank search doubles as the first tile of candidates.
DI bool s1_pblock(VmsT &V, u32 bsize, u32 &start)
{
    const u32 lane = lane_id();
    const u64 q = ((u64)bsize << 32) | 0xFFFFFFFFu;
    u32 base;
    if (V.pp.stride >= 64) {
        base = rank_fast<false>(V.pp, V.pool, V.np, q);
    } else {
        const u32 c = popc64(ballot(V.pp.v > q));
        base = dec_sat(c) * V.pp.stride;  // the first pBlock of bsize chunks lies inside this tile
    }
    for (;;) {
        const u32 i = base + lane;
        const u64 key = V.pool[i];                  // zero keys follow the pool
        const bool eq = (u32)(key >> 32) == bsize;
        const u64 vm = ballot(eq);
        if (!vm) return false;
        const u32 st = ~(u32)key;
        const u32 word = pin(V.bmp[eq ? st >> 5 : 0u]);
        const u64 m = ballot(eq && !((word >> (st & 31)) & 1u));
        if (LIKELY(m)) {
            start = from_lane(st, first_lane(m));
            return true;
        }
        if (~vm >> 63) return false;                // the run ended inside the tile
        base += 64;
    }
}

struct VmsRes {
    u32 dec_lo;                 // low decision word (code C_OOM alone when the request failed)
    u32 ref;                    // pBlock first chunk / sBlock creation number (= high decision word)
    u32 kind, held;             // what the slot now holds, chunks held
    u32 list;                   // sBlock: offset << 16 | entries of its list
};

// No block of exactly bsize chunks is free: BestFit's second loop and the post-processing of
// its state (Algorithm 1; Sec. 4.1, Fig. 9, states S2 to S5).  The rare path: a few per cent of
// the requests of a converged trace.
template <class Slots, class AcctT>
DI void vms_alloc_rest(VmsT &V, Slots &S, u32 bsize, u32 reserved_units, const KParams &P, AcctT &A, u32 ev,
                       VmsRes &R)
{
    const u32 lane = lane_id();
    R.kind = KIND_PBLOCK;
    R.held = bsize;
    R.ref = 0;
    R.list = 0;
    // pool[lo_p, hi_p) are the pBlocks of exactly bsize chunks (all active, or S1 had taken one)
    u32 lo_p, hi_p;
    {
        const u64 k1 = ((u64)bsize << 32) | 0xFFFFFFFFu, k2 = ((u64)bsize << 32) - 1;
        if (LIKELY(V.pp.stride <= 64)) {
            // the first search level is in registers and still describes the pool: one LDS round trip
            const u32 c1 = popc64(ballot(V.pp.v > k1)), c2 = popc64(ballot(V.pp.v > k2));
            const u32 b1 = dec_sat(c1) * V.pp.stride, b2 = dec_sat(c2) * V.pp.stride;
            const u64 v1 = V.pool[b1 + lane], v2 = V.pool[b2 + lane];
            lo_p = b1 + popc64(ballot(v1 > k1));
            hi_p = b2 + popc64(ballot(v2 > k2));
        } else {
            rank_desc2(V.pool, V.np, k1, k2, &lo_p, &hi_p);
        }
    }

    // ---- Algorithm 1, second loop.  Larger blocks are pool[0, lo_p): the last inactive one in
    // pool order is the single-block candidate (state 2).
    for (u32 hi = lo_p; hi > 0;) {
        u32 lo = hi > 64 ? hi - 64 : 0;
        const bool v = lane < hi - lo;
        const u64 key = V.pool[v ? hi - 1 - lane : 0u];
        const u32 fc = v ? ~(u32)key : 0u;                  // first chunk (chunk 0 for lanes without a block)
        const u32 kw = pin(V.bmp[fc >> 5]);
        const u64 m = ballot(v && !((kw >> (fc & 31)) & 1u));
        if (m) {
            u32 l = first_lane(m), idx = hi - 1 - l;
            u64 pk = from_lane64(key, l);
            u32 psize = (u32)(pk >> 32), pstart = ~(u32)pk;
            if (UNLIKELY(psize < P.frag_limit_chunks)) {
                // below the fragmentation limit: not worth cutting, hand it out whole (Sec. 4.2.3)
                bmp_fill(V.bmp, ENT_WORD(V.e_skip), pstart, psize, true);
                R.ref = pstart;
                R.held = psize;
                R.dec_lo = C_SPLIT | (1u << 8);
                return;
            }
            if (UNLIKELY(V.np + 1 > P.cap_pblocks || V.ns + 1 > P.cap_sblocks ||
                         !arena_reserve(V, S, run_words(pstart, psize), P, A, ev))) {
                A.overflow(ev, (V.np + 1 > P.cap_pblocks ? VMS_ST_OVF_PBLOCKS : 0u) | (V.ns + 1 > P.cap_sblocks ? VMS_ST_OVF_SBLOCKS : 0u));
                R.dec_lo = C_INVALID;
                return;
            }
            // S2: Split into the request and the rest; a stitched block keeps the uncut size on record
            pool_cut(V, idx, bsize, pstart, psize - bsize, pstart + bsize, A);
            A.add(SC_N_SPLIT, 1);
            u32 n = arena_put(V, V.top, pstart, psize);
            spool_insert(V, psize, V.top, n, A, true);
            V.top += n;
            bmp_fill(V.bmp, ENT_WORD(V.e_skip), pstart, bsize, true);
            R.ref = pstart;
            R.dec_lo = C_SPLIT | B_6 | (1u << 8);
            if (stitch_free(V, P, A)) R.dec_lo |= B_7;
            return;
        }
        hi = lo;
    }

    // Smaller blocks, largest first, until the request is covered (states 3 and 4).  Blocks
    // below the fragmentation limit sit at the tail of the pool and are never stitched.
    u32 lim = V.np;
    if (UNLIKELY(P.frag_limit_chunks > 1)) lim = rank_desc(V.pool, V.np, ((u64)P.frag_limit_chunks << 32) - 1);
    u32 sum = 0, k = 0, pos = NONE32;
    for (u32 base = hi_p; base < lim; base += 64) {
        const u32 i = base + lane;
        const u64 key = V.pool[i < lim ? i : 0u];
        const u32 fc = i < lim ? ~(u32)key : 0u;
        const u32 kw = pin(V.bmp[fc >> 5]);
        const bool inact = i < lim && !((kw >> (fc & 31)) & 1u);
        u32 tot, incl = wave_scan_add(inact ? (u32)(key >> 32) : 0u, &tot);
        u64 im = ballot(inact);
        if (sum + tot >= bsize) {
            u32 l = first_lane(ballot(inact && sum + incl >= bsize));
            pos = base + l;
            k += popc64(im & ((2ull << l) - 1));
            sum += from_lane(incl, l);
            break;
        }
        k += popc64(im);
        sum += tot;
    }
    const bool s3 = pos != NONE32;
    const u32 excess = s3 ? sum - bsize : 0, deficit = s3 ? 0 : bsize - sum;
    if (!s3) {
        // S4 needs new physical chunks; S5 if the device cannot provide them
        if (UNLIKELY(reserved_units + (deficit << P.chunk_shift) > P.capacity_units)) {
            R.dec_lo = C_OOM;
            return;
        }
        if (UNLIKELY(V.n_chunks + deficit > P.cap_chunks)) {
            A.overflow(ev, VMS_ST_OVF_CHUNKS);
            R.dec_lo = C_INVALID;
            return;
        }
    }
    if (!s3 && k == 0) {
        // nothing cached is usable: the new pBlock serves the request directly (no list, no sBlock)
        if (UNLIKELY(V.np + 1 > P.cap_pblocks)) {
            A.overflow(ev, VMS_ST_OVF_PBLOCKS);
            R.dec_lo = C_INVALID;
            return;
        }
        u32 start = V.n_chunks;
        pool_insert(V, deficit, start, A);
        V.n_chunks += deficit;
        bmp_fill(V.bmp, ENT_WORD(V.e_skip), start, deficit, true);
        R.ref = start;
        R.dec_lo = C_GROW;
        return;
    }
    // list entries created below: a run of L chunks touches at most L / 32 + 2 bitmap words
    const u32 need = 2u * k + 3u * (((sum > bsize ? sum : bsize) >> 5) + 2u);
    if (UNLIKELY(V.np + 2 > P.cap_pblocks || V.ns + 2 > P.cap_sblocks || !arena_reserve(V, S, need, P, A, ev))) {
        A.overflow(ev, (V.np + 2 > P.cap_pblocks ? VMS_ST_OVF_PBLOCKS : 0u) | (V.ns + 2 > P.cap_sblocks ? VMS_ST_OVF_SBLOCKS : 0u));
        R.dec_lo = C_INVALID;
        return;
    }
    // second pass: the candidates' chunk runs (and the new pBlock's) are collected in tmp[] and
    // read back as the list
    u32 cnt;
    {
        u32 wmin = NONE32, wmax = 0;
        const u32 endi = s3 ? pos + 1 : lim;
        for (u32 base = hi_p; base < endi; base += 64) {
            const u32 i = base + lane;
            const u64 key = V.pool[i < endi ? i : 0u];
            const u32 fc = i < endi ? ~(u32)key : 0u;
            const u32 kw = pin(V.bmp[fc >> 5]);
            const bool inact = i < endi && !((kw >> (fc & 31)) & 1u);
            u32 len = (u32)(key >> 32), start = ~(u32)key;
            if (i == pos) len -= excess;
            list_mark(V, start, inact ? len : 0u, wmin, wmax);
        }
        if (!s3) list_mark(V, V.n_chunks, lane == 0 ? deficit : 0u, wmin, wmax);
        wave_sync();
        cnt = list_extract(V, wave_min_u32(wmin), wave_max_u32(wmax), V.top, P.cap_runs);
    }
    u32 used = cnt;             // arena entries consumed, including a restore block's
    R.dec_lo = 0;
    if (s3) {
        if (excess) {
            // cut the last candidate so the sum is exact; remember its uncut size (Fig. 9, sBlock 2)
            u64 qk = ld_uni(V.pool, pos);
            u32 qsize = (u32)(qk >> 32), qstart = ~(u32)qk;
            pool_cut(V, pos, qsize - excess, qstart, excess, qstart + qsize - excess, A);
            A.add(SC_N_SPLIT, 1);
            u32 n = arena_put(V, V.top + cnt, qstart, qsize);
            spool_insert(V, qsize, V.top + cnt, n, A, true);
            used += n;
            R.dec_lo |= B_6;
        }
        R.dec_lo |= C_STITCH;
    } else {
        u32 start = V.n_chunks;                 // Alloc: exactly the missing chunks
        pool_insert(V, deficit, start, A);
        V.n_chunks += deficit;
        R.dec_lo |= C_GROW;
    }
    R.ref = V.next_sid;
    spool_insert(V, bsize, V.top, cnt, A, !(s3 && excess));
    bmp_fill_entries(V, V.top, cnt, true);
    R.list = (u32)V.pack(V.top, cnt);
    V.top += used;
    A.peak(SC_HW_MEMBERS, k + (s3 ? 0u : 1u));
    R.kind = KIND_SBLOCK;
    R.dec_lo |= B_SBLOCK | (k << 8);
    if (stitch_free(V, P, A)) R.dec_lo |= B_7;
}

// ---------------------------------------------------------------------------
// Hot and cold halves.  The replay loop keeps only what the two frequent paths need in registers
// (exact hit on a cached block, free).  The states S2 to S5 and the splitting pool for requests below
// one chunk sit behind unlikely branches and keep the scalars only they need in the first 256 bytes of
// LDS (SC_* above, one u32 each), where the event counters are updated in place as well.
// ---------------------------------------------------------------------------
#define LDS_SCALARS 0u
static_assert(SC_COUNT <= 64, "LDS header layout");

// stand-in for the slot table inside the rare paths: they only note that lists have moved
struct ColdSlots {
    bool compacted;
    DI void moved(u32, u32, const KParams &) { compacted = true; }
};

// the LDS scalars in registers, one LDS access for all of them: lane k holds scalar k
struct ColdState {
    u32 v;
    // pinned: every lane must load its scalar even if only one lane goes on to use them
    DI void load(const char *lds) { v = pin(((const u32 *)(lds + LDS_SCALARS))[lane_id()]); }
    DI u32 get(u32 k) const { return from_lane(v, k); }
};

DI void vms_bind(VmsT &V, char *lds, char *ws_slice, const KParams &P)
{
    V.pool = (u64 *)(lds + P.off_pool);
    V.bmp = (u32 *)(lds + P.off_bmp);
    V.skey = (u64 *)(lds + P.off_skey);
    V.smeta = (VmsT::meta_t *)(lds + P.off_smeta);
    V.sstamp = (u32 *)(lds + P.off_sstamp);
    V.swit = (u32 *)(lds + P.off_swit);
    V.tmp = (u32 *)(lds + P.off_tmp);
    V.idle = V.tmp + (P.cap_chunks + 31) / 32;
    V.e_skip = (((P.cap_chunks + 31) / 32) << 12) | WIT_NONE;
    V.bounce = (u32 *)ws_slice;                 // where arena_compact copies the lists
    V.arena = (u32 *)(lds + P.off_arena);
}

// A request for bsize chunks that no cached block fits exactly (states S2 to S5): inlined into the
// replay loop (a call would cost more in saved registers than the few per cent of the requests
// that come here can repay), working on the loop's own pool state; the three scalars that only
// this path needs (arena top, live entries, next creation number) wait in LDS in between.
// Returns false if an engine table overflowed (the trace ends).
DI bool vms_alloc_cold(char *lds, VmsT &V, const KParams &P, u32 bsize, u32 reserved_units, u32 ev, VmsRes &R,
                       bool &compacted)
{
    u32 *sc = (u32 *)(lds + LDS_SCALARS);
    ColdState C;
    C.load(lds);
    V.top = C.get(SC_TOP);
    V.live_ent = C.get(SC_LIVE);
    V.next_sid = C.get(SC_NEXT_SID);
    AcctLds A;
    A.sc = sc;
    A.idle = V.idle;
    ColdSlots S;
    S.compacted = false;
    vms_alloc_rest(V, S, bsize, reserved_units, P, A, ev, R);
    st_one(sc, (u32)SC_TOP, V.top);
    st_one(sc, (u32)SC_LIVE, V.live_ent);
    st_one(sc, (u32)SC_NEXT_SID, V.next_sid);
    wave_sync();
    compacted = S.compacted;
    return ld_uni(sc, (u32)SC_STOP) == 0;
}

// The per-tile work shared by the replay kernels: one event per lane.  An event parks what it changed
// (decision word, change of requested and active units) in its lane; the running totals, their peaks
// and the split and merge counts are taken from the 64 lanes once per tile.  Kept per event they cost
// eight scalar operations each time (4.4 cycles apiece on a wavefront alone) and four scalar registers
// that the stitching kernels had to keep in vector lanes; two prefix sums and two maxima per tile cost
// five cycles per event.  The stitching kernel alone: LoRA 4096x50000 92.7 -> 84.3 ms, scale-out
// 320x20000 17.0 -> 15.6 ms; on a single random trace, whose scalars were at hand, 1.58 -> 1.60 ms.
struct TileOut {
    u32 n_code[8];              // events of this lane per decision code ([7]: invalid)
    u64 dig;                    // this lane's share of the digest
    u32 requested, active;      // wave-uniform: after the tiles so far
    u32 peak_requested, peak_active;
    u32 n_split, n_merge;       // of the splitting pools: cuts and merges the decision words report
    DI void init()
    {
#pragma unroll
        for (u32 c = 0; c < 8; c++) n_code[c] = 0;
        dig = 0;
        requested = active = peak_requested = peak_active = n_split = n_merge = 0;
    }
};

// the last tile of a trace (or the tile in which a table overflowed): only the lanes below `done` store
__device__ __attribute__((noinline)) void emit_partial(u64 *dst, u64 dec, u32 done)
{
    if (lane_id() < done) dst[lane_id()] = dec;
}

// v_req / v_act: what each event added to the requested and active units (modulo 2^32; lanes that hold no
// event hold zeros), v_res: units reserved after it.  SAME: active is requested (splitting policy).
template <bool SAME>
DI void tile_emit(TileOut &T, u64 *dec_row, u32 base, u32 done, u32 v_dlo, u32 v_dhi, u32 v_req, u32 v_act, u32 v_res)
{
    const u32 lane = lane_id();
    const bool valid = lane < done;
    const u64 dec = ((u64)v_dhi << 32) | v_dlo;
    if (dec_row) {
        if (done == 64) dec_row[base + lane] = dec;         // a full tile: one coalesced store, no lane off
        else emit_partial(dec_row + base, dec, done);
    }
    const u32 code = v_dlo & 15, cidx = !valid ? 8u : (code == C_INVALID ? 7u : code);
#pragma unroll
    for (u32 c = 0; c < 8; c++) T.n_code[c] += cidx == c ? 1u : 0u;
    // the totals only rise on an allocation, so their maximum over all events is their peak
    u32 tot;
    const u32 req = T.requested + wave_scan_add(v_req, &tot);
    T.requested += tot;
    T.peak_requested = max(T.peak_requested, ~wave_min_u32(~req));
    u32 act = req;
    if (!SAME) {
        act = T.active + wave_scan_add(v_act, &tot);
        T.active += tot;
        T.peak_active = max(T.peak_active, ~wave_min_u32(~act));
    }
    const bool pool = valid && (SAME || (v_dlo & B_SMALL)) && code <= C_GROW;
    T.n_split += popc64(ballot(pool && code != C_FREE && (v_dlo & B_6)));
    T.n_merge += popc64(ballot(pool && code == C_FREE && (v_dlo & B_6))) + popc64(ballot(pool && code == C_FREE && (v_dlo & B_7)));
    // digest: sum over events i of (decision * K1 + (active << 32 | reserved)) * ((2 i + 1) * K2)
    const u64 term = (dec * 0x9E3779B97F4A7C15ull + (((u64)act << 32) | v_res)) *
                     ((2ull * (base + lane) + 1ull) * 0xD6E8FEB86659FD93ull);
    T.dig += valid ? term : 0ull;
}

// end of the trace: the lanes' shares become the totals (all lanes return the same values)
DI u64 tile_totals(const TileOut &T, u32 n_code[8])
{
#pragma unroll
    for (u32 c = 0; c < 8; c++) n_code[c] = (u32)wave_sum_u64(T.n_code[c]);
    return wave_sum_u64(T.dig);
}

// The second pass (vms_config.retry_traces): a launch of a few wavefronts with larger
// tables that replays every trace whose first replay ended in a table overflow.  The wavefronts
// share one counter over the trace numbers: each takes 64 numbers at a time, looks at their
// status words side by side and replays the flagged ones among them one after the other.
struct SecondPass {
    u64 flagged = 0;
    u32 first = 0;
    // the next flagged trace for this wavefront, or false when all have been handed out
    DI bool next(const KParams &P, const vms_trace_stats *__restrict__ st, u32 *counter, u32 &trace)
    {
        while (!flagged) {
            u32 b = 0;
            if (lane_id() == 0) b = atomicAdd(counter, 64u);
            first = from_lane(b, 0);
            if (first >= P.n_traces) return false;
            const u32 t = first + lane_id();
            flagged = ballot(t < P.n_traces && (st[t < P.n_traces ? t : 0u].status & VMS_ST_TABLE_OVERFLOW) != 0);
        }
        trace = first + first_lane(flagged);
        flagged &= flagged - 1;
        return true;
    }
};

// ---------------------------------------------------------------------------
// Replay under the stitching policy (Sec. 3, Sec. 4.1), one wavefront per trace.
// SLOTS: where the slot table is (SLOTS_IN_REGS: max_slots <= 64).
//
// Per event only the allocator runs; the decision word and what the event added to the requested
// and active units are parked in lane j of four registers, and where memory was reserved the lanes
// from j up take over the new reserved total.  Once per tile of 64 events the lanes store the
// decisions with one coalesced write, take the totals after each event and their peaks by prefix
// sums and maxima, count the decision codes and fold their event into the digest, all 64 events
// side by side (tile_emit).
// ---------------------------------------------------------------------------
template <int SLOTS>
DI void replay_vms_flat(char *lds, const KParams &P, const u64 *__restrict__ events, const u32 *__restrict__ n_events,
                        u64 *__restrict__ decisions, vms_trace_stats *__restrict__ stats, char *__restrict__ workspace)
{
    const u32 lane = lane_id();
    const u32 trace = blockIdx.x;
    char *ws_slice = workspace + (size_t)trace * P.ws_stride;
    // a second pass follows for traces that outgrow these tables: it counts the traces it takes on
    if (P.retry_slots && trace == 0) ((u32 *)&stats[2 * (size_t)P.n_traces])[1] = 0;     // the second pass counts from 0

    SlotsT<SLOTS, true, u32> S;
    S.init(lds, P, trace);
    ((u32 *)(lds + LDS_SCALARS))[lane] = lane == SC_FIRST_OOM || lane == SC_OVF_EVENT ? NONE32 : 0u;     // LDS header
    VmsT V;
    vms_bind(V, lds, ws_slice, P);
    V.np = V.ns = V.n_chunks = V.top = V.live_ent = V.next_sid = V.clock = 0;
    V.pp.v = V.sp.v = 0;
    V.pp.stride = V.sp.stride = 1;
    for (u32 i = lane; i < (P.cap_chunks + 31) / 32; i += 64) V.bmp[i] = V.tmp[i] = 0;
    V.tmp[(P.cap_chunks + 31) / 32 + lane] = 0;             // 64 spare words: where idle lanes OR their zeros
    // the searches read up to 64 places past the live part of pool[], skey[], swit[] and arena[]
    // without clamping: zero keys there, and witnesses / entries on words that exist
    SplitPool<SMALL_TILES, true> Q;                               // the pool for small requests
    Q.init(lds, P);
    for (u32 i = lane; i < P.cap_pblocks + 64; i += 64) V.pool[i] = 0;
    for (u32 i = lane; i < P.cap_sblocks + 64; i += 64) {
        V.skey[i] = 0;
        V.swit[i] = WIT_NONE;
        V.smeta[i] = 0;
    }
    for (u32 i = lane; i < P.cap_runs + 64; i += 64) V.arena[i] = WIT_NONE;
    st_one(V.bmp, (P.cap_chunks + 31) / 32, 0u);                // the spare word
    wave_sync();

    u32 lost = 0;               // request of a FREE that outgrew a table: the trace ends there, the request counts as gone
    u32 sp_reserved = 0;        // small-request pool: units reserved so far
    bool stop = false;
    TileOut T;
    T.init();
    const u32 chunk_units = 1u << P.chunk_shift;
    const u32 n_ev = n_events ? min(uni(n_events[trace]), P.max_events) : P.max_events;
    const u64 *ev_row = events + (size_t)trace * P.max_events;
    u64 *dec_row = decisions ? decisions + (size_t)trace * P.max_events : nullptr;

    u32 fast_limit = P.small_limit_units;   // requests from this size on take the usual S1 route (renewed with the probe)
    u64 ev = pin64(lane < n_ev ? ev_row[lane] : 0), ev_next = ev;
    for (u32 base = 0; base < n_ev; base += 64) {
        const u32 tile = min(64u, n_ev - base);
        u32 ev_lo = (u32)ev;
        u32 ev_hi = (u32)(ev >> 32);
        S.tile_begin(ev_lo, ev_hi, tile);
        if (base + 64 < n_ev) ev_next = ev_row[min(base + 64 + lane, n_ev - 1)];       // prefetch (see replay_split_kernel)
        u32 v_res = sp_reserved + (V.n_chunks << P.chunk_shift);
        u32 done = tile, todo = tile;       // todo drops to 0 when an engine table overflows: the trace ends there
        // every path of an event ends by noting its results and going on to the next event
        // memory was reserved: the events from this one on see the new total
#define RESERVED_NOW() v_res = lane >= j ? sp_reserved + (V.n_chunks << P.chunk_shift) : v_res
        for (u32 j = 0; j < todo; j++) {
            const u32 w = from_lane(ev_lo, j), at = S.at(ev_hi, j), req = S.get_req(at);
            if ((int)w < 0) {
                // ---- FREE.  Update (Sec. 3.3.2): only activity flips; memory stays with its pBlocks
                if (UNLIKELY(req + 1u <= 1u)) {             // unbound, or bound to a request that failed
                    if (req == SLOT_OOM) S.failed(j, at, (u32)C_FREE_NOOP, SLOT_UNBOUND);
                    else S.not_done(j, at);
                    continue;
                }
                const u32 a = S.get_a(at), b = S.get_b(at);
                const u32 kind = b & 3, held = (b >> 2) << P.chunk_shift;
                if (LIKELY((kind & KIND_SBLOCK) != 0)) {    // (a bit test: the usual case stays the fall-through)
                    const u32 list = S.get_c(at), off = list >> 16, cnt = list & 0xFFFFu;
                    // one list read, then the entries' bits cleared without waiting for anything
                    if (LIKELY(cnt <= 64)) entries_apply(V, V.arena[off + lane], lane < cnt, false);
                    else bmp_fill_entries(V, off, cnt, false);
                    S.free_done(j, at, C_FREE | B_SBLOCK, a, req, held);
                    continue;
                }
                if (kind == KIND_PBLOCK) {
                    bmp_fill(V.bmp, ENT_WORD(V.e_skip), a, b >> 2, false);
                    S.free_done(j, at, (u32)C_FREE, a, req, held);
                    continue;
                }
                AcctLds A;
                A.sc = (u32 *)(lds + LDS_SCALARS);
                A.idle = V.idle;
                Q.release(a, req, A, base + j,
                          [&](bool ml, bool mr) {
                              S.free_done(j, at, C_FREE | B_SMALL | (ml ? B_6 : 0u) | (mr ? B_7 : 0u), Q.addr(a), req, req);
                          },
                          [&]() {
                              lost = req;
                              stop = true;
                              done = j;
                              todo = 0;
                          });
                continue;
            }
            // ---- ALLOC
            const u32 size = w;
            if (UNLIKELY(size == 0 || req != SLOT_UNBOUND)) {
                S.not_done(j, at);
                continue;
            }
            if (LIKELY(size >= fast_limit)) {
                const u32 bsize = (size + chunk_units - 1) >> P.chunk_shift;
                u32 ref, list = 0;
                // Sec. 5.1: active memory is recorded at its peak; the totals only rise on an allocation
#define S1_SBLOCK_HIT                                                      \
    {                                                                      \
        S.alloc_done(j, at, C_EXACT | B_SBLOCK | (1u << 8), ref, size, bsize << P.chunk_shift, ref, KIND_SBLOCK | (bsize << 2), list); \
        continue;                                                          \
    }
                // S1 on stitched blocks, the usual way (see s1_sblock_from for the general route).  It is
                // written out here, not called, so that the hit leaves for the next event from where it
                // is found: returned through a function it would meet the other outcomes again and
                // cost a flag and two branches to tell them apart.
                u32 from = NONE32;              // where the general route goes on; NONE32: no inactive sBlock of this size
                switch (0) {
                default:
                    const u64 q = ((u64)bsize << 32) | 0xFFFFFFFFu;
                    // keys greater than q end at most `stride` < 64 places into the block: the first
                    // sBlock of bsize chunks, if there is one, lies inside the tile
                    const u32 c = popc64(ballot(V.sp.v > q));
                    const u32 b0 = dec_sat(c) * V.sp.stride;
                    const u32 i = b0 + lane;
                    // (pinned, after all three loads are on their way: one round trip, not the last two
                    // behind the branch)
                    const u64 key = V.skey[i];
                    const u32 wit0 = V.swit[i];
                    const auto meta0 = V.smeta[i];
                    const u32 wit = pin(wit0);
                    const auto meta = VmsT::pinm(meta0);
                    const u64 vm = ballot((u32)(key >> 32) == bsize);
                    if (UNLIKELY(!vm)) break;
                    const u32 wv = pin(V.bmp[ENT_WORD(wit)]);
                    const u64 unknown = vm & ~ballot((wv & emask(wit)) != 0);
                    if (UNLIKELY(!unknown)) {
                        if (~vm >> 63) break;   // the run of equal sizes ended inside the tile: all known active
                        from = b0 + 64;
                        break;
                    }
                    const u32 l = first_lane(unknown);
                    const auto m = from_lane_any(meta, l);
                    const u32 off = V.off(m), cnt = V.cnt(m);
                    const u32 e0 = pin(V.arena[off + lane]);
                    const u32 e = lane < cnt ? e0 : V.e_skip;
                    const u32 word = pin(V.bmp[ENT_WORD(e)]);
                    if (LIKELY(cnt <= 64 && !ballot((word & emask(e)) != 0))) {
                        entries_apply(V, e, lane < cnt, true);
                        st_one(V.sstamp, b0 + l, ++V.clock);
                        ref = ~from_lane((u32)key, l);
                        list = (u32)m;
                        S1_SBLOCK_HIT
                    }
                    from = b0 + l;
                }
                if (UNLIKELY(from != NONE32))
                    if (s1_sblock_from(V, bsize, from, ref, list)) S1_SBLOCK_HIT
#define S1_PBLOCK_TRY                                                      \
    if (s1_pblock(V, bsize, ref)) {                                        \
        bmp_fill(V.bmp, ENT_WORD(V.e_skip), ref, bsize, true);             \
        S.alloc_done(j, at, C_EXACT | (1u << 8), ref, size, bsize << P.chunk_shift, ref, KIND_PBLOCK | (bsize << 2), 0u); \
        continue;                                                          \
    }
                S1_PBLOCK_TRY
            } else if (UNLIKELY(size >= P.small_limit_units)) {
                // more than 4,032 sBlocks cached: their first search level no longer selects a single
                // tile (fast_limit keeps such a trace off the route above, at no cost to the others)
                const u32 bsize = (size + chunk_units - 1) >> P.chunk_shift;
                u32 ref, list = 0;
                const u32 from = rank_fast<false>(V.sp, V.skey, V.ns, ((u64)bsize << 32) | 0xFFFFFFFFu);
                if (s1_sblock_from(V, bsize, from, ref, list)) S1_SBLOCK_HIT
                S1_PBLOCK_TRY
            }
#undef S1_PBLOCK_TRY
#undef S1_SBLOCK_HIT
            // ---- the rare cases: no exact fit (states S2 to S5), or a request below one chunk
            wave_sync();
            if (size < P.small_limit_units) {
                const u32 seg = ((size + chunk_units - 1) >> P.chunk_shift) << P.chunk_shift;
                const u32 reserved = sp_reserved + (V.n_chunks << P.chunk_shift);
                AcctLds A;
                A.sc = (u32 *)(lds + LDS_SCALARS);
                A.idle = V.idle;
                Q.alloc(size, seg, reserved + seg <= P.capacity_units, A, base + j,
                        [&](u32 code, u32 ref, bool split) {
                            sp_reserved = Q.reserved();
                            if (UNLIKELY(code == C_OOM)) {
                                S.failed(j, at, (u32)C_OOM, SLOT_OOM);
                                ColdState C;                // rare: note the first failed request
                                C.load(lds);
                                if (C.get(SC_FIRST_OOM) == NONE32)
                                    st_one((u32 *)(lds + LDS_SCALARS), (u32)SC_FIRST_OOM, base + j);
                                return;
                            }
                            if (code == C_GROW) RESERVED_NOW();
                            S.alloc_done(j, at, code | B_SMALL | (split ? B_6 : 0u) | ((code == C_GROW ? 0u : 1u) << 8), Q.addr(ref),
                                         size, size, ref, (u32)KIND_SMALL, 0u);
                        },
                        [&]() {
                            stop = true;
                            done = j;
                            todo = 0;
                        });
                continue;
            }
            const u32 bsize = (size + chunk_units - 1) >> P.chunk_shift;
            VmsRes R;
            bool compacted;
            const bool went = vms_alloc_cold(lds, V, P, bsize, sp_reserved + (V.n_chunks << P.chunk_shift), base + j, R, compacted);
            // the pools may have changed: renew the first search level of both
            probe_refresh(V.sp, V.skey, V.ns);
            probe_refresh(V.pp, V.pool, V.np);
            fast_limit = V.sp.stride >= 64 ? NONE32 : P.small_limit_units;
            // lists have moved: every record of an sBlock looks its list up again
            if (UNLIKELY(compacted))
                S.relist([&](u32 sid, u32 b, u32) {
                    // by its key (creation number, chunks) in skey[0..ns), descending; every lane searches (13 halvings
                    // cover 4096 sBlocks), lanes without an sBlock for nothing: no lane is switched off
                    const u64 key = ((u64)(b >> 2) << 32) | (u32)~sid;
                    u32 lo = 0, hi = V.ns;          // first index whose key is not greater than key
#pragma unroll 1
                    for (u32 it = 0; it < 13; it++) {
                        const u32 mid = (lo + hi) >> 1;         // < ns while lo < hi; else a place that exists
                        const bool open = lo < hi, greater = V.skey[mid] > key;
                        lo = open && greater ? mid + 1 : lo;
                        hi = open && !greater ? mid : hi;
                    }
                    return pin(V.smeta[lo]);
                });
            if (UNLIKELY(!went)) {                                // an engine table overflowed: the trace ends here
                stop = true;
                done = j;
                todo = 0;
                continue;
            }
            if (UNLIKELY((R.dec_lo & 15) == C_OOM)) {
                S.failed(j, at, (u32)C_OOM, SLOT_OOM);
                ColdState C;                                // rare: note the first failed request
                C.load(lds);
                if (C.get(SC_FIRST_OOM) == NONE32) st_one((u32 *)(lds + LDS_SCALARS), (u32)SC_FIRST_OOM, base + j);
                continue;
            }
            if ((R.dec_lo & 15) == C_GROW) RESERVED_NOW();
            S.alloc_done(j, at, R.dec_lo, R.ref, size, R.held << P.chunk_shift, R.ref, R.kind | (R.held << 2), R.list);
        }
#undef RESERVED_NOW
        ev = pin64(ev_next);
        S.tile_end(done, P.chunk_shift, [&](u32 ref) { return Q.addr(ref); });
        tile_emit<false>(T, dec_row, base, done, S.v_dlo, S.v_dhi, S.v_req, S.v_act, v_res);
        if (stop) break;
    }

    wave_sync();
    u32 n_code[8];
    const u64 digest = tile_totals(T, n_code);
    ColdState C;
    C.load(lds);
    // (lane reads stay outside the one-lane block below: they are wave-wide operations)
    u32 sc[SC_COUNT];
#pragma unroll
    for (u32 k = 0; k < SC_COUNT; k++) sc[k] = C.get(k);
    if (lane == 0) {
        vms_trace_stats &s = stats[(size_t)P.n_traces + trace];
#pragma unroll
        for (u32 c = 0; c < 8; c++) s.n_code[c] = n_code[c];
        const u64 reserved = sp_reserved + (V.n_chunks << P.chunk_shift);
        s.peak_requested = (u64)T.peak_requested * 512;
        s.peak_active = (u64)T.peak_active * 512;
        s.peak_reserved = reserved * 512;           // reserved memory never shrinks: its peak is its final value
        s.final_requested = (u64)(T.requested - lost) * 512;
        s.final_active = (u64)T.active * 512;
        s.final_reserved = reserved * 512;
        s.digest = digest;
        s.n_split = sc[SC_N_SPLIT] + T.n_split;
        s.n_merge = T.n_merge;
        s.n_sblock_created = sc[SC_N_CREATED];
        s.n_sblock_evicted = sc[SC_N_EVICTED];
        s.first_oom_event = sc[SC_FIRST_OOM];
        s.status = sc[SC_STATUS] | (n_code[7] ? VMS_ST_INVALID_EVENT : 0u);
        s.max_pblocks = sc[SC_HW_PBLOCKS];
        s.max_sblocks = sc[SC_HW_SBLOCKS];
        s.max_free_blocks = Q.most();
        s.max_members = sc[SC_HW_MEMBERS];
        s.max_runs = sc[SC_HW_RUNS];
        s.overflow_event = sc[SC_OVF_EVENT];
        s.max_multi_pblocks = sc[SC_HW_MULTI];
        s.reserved1 = 0;
        // Sec. 5.1: fragmentation = 1 - utilisation, utilisation = peak active / peak reserved
        s.fragmentation = reserved ? 1.0 - (double)T.peak_active / (double)reserved : 0.0;
    }
}

template <int SLOTS>
__global__ __launch_bounds__(64) void replay_vms_kernel(KParams P, const u64 *__restrict__ events,
                                                        const u32 *__restrict__ n_events,
                                                        u64 *__restrict__ decisions, vms_trace_stats *__restrict__ stats,
                                                        char *__restrict__ workspace)
{
    WAVE_DYNAMIC_LDS(lds);
    replay_vms_flat<SLOTS>(lds, P, events, n_events, decisions, stats, workspace);
}

// ---------------------------------------------------------------------------
// Replay under the splitting policy (Sec. 2.2), one wavefront per trace.  Both of its paths are
// hot, so everything is inline and its few scalars stay in registers.
// ---------------------------------------------------------------------------
template <int SLOTS, u32 TILES, bool TAIL>
DI void replay_split(char *lds, const KParams &P, const u64 *__restrict__ events, const u32 *__restrict__ n_events,
                     u64 *__restrict__ decisions, vms_trace_stats *__restrict__ stats)
{
    const u32 lane = lane_id();
    u32 trace = blockIdx.x;
    u32 *taken = (u32 *)&stats[2 * (size_t)P.n_traces];     // [0]: trace numbers the second pass has handed out
    if (!P.retry && P.retry_slots && trace == 0) taken[0] = 0;
    SecondPass W;
    do {        // once; the second pass: once per flagged trace this wavefront takes on
    if (P.retry && !W.next(P, stats, &taken[0], trace)) return;

    SlotsT<SLOTS, false, u32> S;
    S.init(lds, P, blockIdx.x);
    SplitPool<TILES, TAIL> sp;
    sp.init(lds, P);

    AcctRegs A;
    A.init();
    TileOut T;
    T.init();
    const u32 chunk_units = 1u << P.chunk_shift;
    const u32 n_ev = n_events ? min(uni(n_events[trace]), P.max_events) : P.max_events;
    const u64 *ev_row = events + (size_t)trace * P.max_events;
    u64 *dec_row = decisions ? decisions + (size_t)trace * P.max_events : nullptr;

    u64 ev = pin64(lane < n_ev ? ev_row[lane] : 0), ev_next = ev;
    for (u32 base = 0; base < n_ev; base += 64) {
        const u32 tile = min(64u, n_ev - base);
        u32 ev_lo = (u32)ev;
        u32 ev_hi = (u32)(ev >> 32);
        S.tile_begin(ev_lo, ev_hi, tile);
        // the next tile, on its way while this one is replayed (the flat stitching kernel alone on
        // recomputation traces 1024x20000: 8.56 -> 8.45 ms): nothing touches the value (a select on it
        // would wait for memory here, once per 64 events) until this tile's results are stored, and it is
        // taken over before that store, which would have to be waited for too (one counter).  Lanes past
        // the end hold the last event, which no j reaches.
        if (base + 64 < n_ev) ev_next = ev_row[min(base + 64 + lane, n_ev - 1)];
        u32 v_res = sp.reserved();
        u32 done = tile, todo = tile;       // todo drops to 0 when the free list overflows: the trace ends there
        u32 w_next = from_lane(ev_lo, 0), at_next = S.at(ev_hi, 0);            // one event ahead
        for (u32 j = 0; j < todo; j++) {
            const u32 w = w_next, at = at_next;
            w_next = from_lane(ev_lo, (j + 1) & 63);
            at_next = S.at(ev_hi, (j + 1) & 63);
            // every path of an event ends by noting its results; none hands a result to a common tail
            // (that would cost flags to test)
            auto overflow = [&]() {
                done = j;
                todo = 0;
            };
            const u32 req = S.get_req(at);
            if ((int)w < 0) {
                if (UNLIKELY(req + 1u <= 1u)) {             // unbound, or bound to a request that failed
                    if (req == SLOT_OOM) S.failed(j, at, (u32)C_FREE_NOOP, SLOT_UNBOUND);
                    else S.not_done(j, at);
                    continue;
                }
                const u32 a = S.get_a(at);
                sp.release(a, req, A, base + j,
                           [&](bool ml, bool mr) {
                               S.free_done(j, at, C_FREE | (ml ? B_6 : 0u) | (mr ? B_7 : 0u), sp.addr(a), req, req);
                           },
                           overflow);
                continue;
            }
            const u32 size = w;
            if (UNLIKELY(size == 0 || req != SLOT_UNBOUND)) {
                S.not_done(j, at);
                continue;
            }
            const u32 seg = ((size + chunk_units - 1) >> P.chunk_shift) << P.chunk_shift;
            sp.alloc(size, seg, sp.reserved() + seg <= P.capacity_units, A, base + j,
                     [&](u32 code, u32 ref, bool split) {
                         if (code == C_OOM) {
                             S.failed(j, at, (u32)C_OOM, SLOT_OOM);
                             if (A.f[SC_FIRST_OOM] == NONE32) A.f[SC_FIRST_OOM] = base + j;
                             return;
                         }
                         // blocks are cut to the request: active bytes are the requested bytes
                         if (code == C_GROW) v_res = lane >= j ? sp.reserved() : v_res;
                         S.alloc_done(j, at, code | (split ? B_6 : 0u) | ((code == C_GROW ? 0u : 1u) << 8), sp.addr(ref), size, size,
                                      ref, 0u, 0u);
                     },
                     overflow);
        }
        ev = pin64(ev_next);
        S.tile_end(done, 0u, [&](u32 ref) { return sp.addr(ref); });
        tile_emit<true>(T, dec_row, base, done, S.v_dlo, S.v_dhi, S.v_req, 0u, v_res);
        if (A.stop) break;
    }

    wave_sync();
    u32 n_code[8];
    const u64 digest = tile_totals(T, n_code);
    if (lane == 0) {
        vms_trace_stats &s = stats[trace];
#pragma unroll
        for (u32 c = 0; c < 8; c++) s.n_code[c] = n_code[c];
        const u64 reserved = sp.reserved();
        s.peak_requested = (u64)T.peak_requested * 512;
        s.peak_active = (u64)T.peak_requested * 512;
        s.peak_reserved = reserved * 512;           // reserved memory never shrinks: its peak is its final value
        s.final_requested = (u64)T.requested * 512;
        s.final_active = (u64)T.requested * 512;
        s.final_reserved = reserved * 512;
        s.digest = digest;
        s.n_split = T.n_split;
        s.n_merge = T.n_merge;
        s.n_sblock_created = 0;
        s.n_sblock_evicted = 0;
        s.first_oom_event = A.f[SC_FIRST_OOM];
        s.status = A.f[SC_STATUS] | (n_code[7] ? VMS_ST_INVALID_EVENT : 0u);
        s.max_pblocks = 0;
        s.max_sblocks = 0;
        s.max_free_blocks = sp.most();
        s.max_members = 0;
        s.max_runs = 0;
        s.overflow_event = A.f[SC_OVF_EVENT];
        s.max_multi_pblocks = 0;
        s.reserved1 = 0;
        // Sec. 5.1: fragmentation = 1 - utilisation, utilisation = peak active / peak reserved
        s.fragmentation = reserved ? 1.0 - (double)T.peak_requested / (double)reserved : 0.0;
    }
    wave_sync();
    } while (P.retry);
}

template <int SLOTS, u32 TILES, bool TAIL>
__global__ __launch_bounds__(64) void replay_split_kernel(KParams P, const u64 *__restrict__ events,
                                                          const u32 *__restrict__ n_events, u64 *__restrict__ decisions,
                                                          vms_trace_stats *__restrict__ stats)
{
    WAVE_DYNAMIC_LDS(lds);
    replay_split<SLOTS, TILES, TAIL>(lds, P, events, n_events, decisions, stats);
}

// Both policies in one launch: a workgroup replays one trace, its first wavefront under the stitching policy (flat
// variant), its second under the splitting policy, each in a part of the LDS of its own.  Nothing passes between
// them.  Two launches need a second stream, which costs a fork and a join (3 traces x 61 events: 76 -> 53 us on the
// device, 110 -> 78 for the caller) and which HIP may put on the hardware queue of the first, where the two kernels
// then run in turn (one handle in three or four of a process that holds more than four streams: recomputation
// 1024x20000 13.2 instead of 8.1 ms).
template <int SLOTS, u32 TILES, bool TAIL>
__global__ __launch_bounds__(128) void replay_both_kernel(KParams P, KParams P_split, const u64 *__restrict__ events,
                                                          const u32 *__restrict__ n_events, u64 *__restrict__ dec_vms,
                                                          u64 *__restrict__ dec_split, vms_trace_stats *__restrict__ stats,
                                                          char *__restrict__ workspace)
{
    WAVE_DYNAMIC_LDS(lds);
    if (wave_of_group() == 0) {
        // (where four workgroups share a compute unit their first wavefronts share two of its SIMDs: ahead of the
        // short wavefronts beside them, recomputation 1024x20000 8.68 -> 8.02 ms)
        wave_priority<2>();
        replay_vms_flat<SLOTS>(lds, P, events, n_events, dec_vms, stats, workspace);
    } else {
        replay_split<SLOTS, TILES, TAIL>(lds + P.lds_bytes, P_split, events, n_events, dec_split, stats);
    }
}

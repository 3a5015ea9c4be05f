// Host-side planning of a replay: checks a vms_config, chooses the kernel variants and lays out
// the per-wavefront LDS arrays and the per-trace workspace slice.  Plain C++ with no device or
// runtime calls, so that the same code serves the library and host-only checks of the kernels.
#ifndef VMS_REPLAY_PLAN_HPP
#define VMS_REPLAY_PLAN_HPP
#include <stdint.h>
#include <string.h>

#include "../../include/vms_replay.h"

// places per lane of the stitching policy's pool for requests below one chunk (see SplitPool)
const uint32_t SMALL_TILES = 3;

// Launch-constant parameters (passed by value as a kernel argument).
struct KParams {
    uint32_t n_traces, max_events;
    uint32_t chunk_shift;            // log2(chunk in 512-byte units)
    uint32_t small_limit_units;
    uint32_t frag_limit_chunks;
    uint32_t spool_threshold;
    uint32_t capacity_units;         // at most 2^30 (512 GiB)
    uint32_t max_slots;
    uint32_t cap_free, cap_pblocks, cap_sblocks, cap_runs, cap_chunks;
    // byte offsets of the per-wave arrays inside dynamic LDS
    uint32_t off_slot_req, off_slot_a, off_slot_b, off_slot_c, off_fl, off_pool, off_bmp, off_skey, off_smeta,
        off_sstamp, off_swit, off_tmp, off_arena;
    uint32_t lds_bytes;
    uint32_t reserved_pad0;
    uint64_t ws_stride;              // workspace bytes per trace
    // fine-grained variant only (see replay_fine.hpp)
    uint32_t off_bnd, off_soff;      // block-start bitmap; list places of the sBlocks
    uint32_t bmp_words;              // words per bitmap that scans may read (a multiple of 4: they are read 16 bytes at a time)
    uint32_t gran_shift;             // a list starts on a multiple of 2^gran_shift 8-byte words of the arena
    uint32_t cap_grans;              // granules per arena half
    uint64_t ws_half;                // bytes of one arena half; the second starts there
    uint32_t ws_tbl_bytes;           // tables in the workspace: bytes of each (witnesses, list places), behind the halves; else 0
    uint32_t reserved_pad;
    // second pass over the traces whose tables overflowed (see ReplayPlan::retry)
    uint32_t retry;                  // this launch is that pass: traces without an overflow flag are left alone
    uint32_t retry_slots;            // traces it has workspace for
    uint64_t retry_ws_off;           // where that workspace starts (bytes from the start of the caller's workspace)
    // tables in global memory of the handle: a slice of mem_stride bytes per wavefront of the launch, the slot table
    // at its start, pool[] of the fine-grained variant mem_pool bytes behind
    char *mem;
    uint64_t mem_stride, mem_pool;
};

// Where the slot table of a trace is: in LDS, in registers (at most 64 slots), in global memory of the handle
enum { SLOTS_IN_LDS, SLOTS_IN_REGS, SLOTS_IN_MEM };

struct ReplayPlan {
    KParams kp[2];                   // [0] splitting kernel, [1] stitching kernel
    bool fine;                       // stitching kernel: the fine-grained variant (lists in the workspace)
    bool wide;                       // fine-grained variant with 32-bit chunk numbers (more than 65,000 chunks)
    int tbl_ws;                      // fine-grained variant: 0 the sBlock tables in LDS; 2 witnesses and list places in the workspace;
                                     // 3 sizes too; 4 and pool[] in global memory of the handle
    bool slot_regs;                  // at most 64 slots
    int slots;                       // SLOTS_IN_*
    uint32_t fl_tiles;               // splitting policy: places for inactive blocks in registers, per lane: 3 or 5 (see SplitPool)
    bool fl_tail;                    // ... and the rest of them in LDS
    size_t ws_bytes;
    bool has_retry;                  // a second pass with the plan below follows the first
    bool together;                   // both policies in one launch, a workgroup of two wavefronts per trace
};

namespace plan_detail {

const uint64_t UNIT = 512;
const uint64_t ENGINE_MAX_BYTES = 1ull << 39;       // 30-bit block addresses in 512-byte units
const uint64_t LDS_PER_CU = 160 * 1024;
const uint32_t TABLE_MAX = 1u << 24;                // upper bound of every per-trace table size

inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }
inline bool is_pow2(uint64_t x) { return x && !(x & (x - 1)); }

// what a pool whose blocks are not all in registers would take with all of them in LDS, beyond what it takes
// there: counted against the compute unit's LDS, so that no table size is refused or accepted for where it lives
inline uint64_t pool_bytes_saved(const KParams &k, int policy, const ReplayPlan &p)
{
    const uint32_t in_regs = 64 * (policy ? SMALL_TILES : p.fl_tiles);
    return k.cap_free <= in_regs ? 0 : (128ull + in_regs) * 8;
}
// ... and what a slot table outside it would take there
inline uint64_t slot_bytes_saved(uint32_t max_slots, int policy, const ReplayPlan &p)
{
    if (p.slots != SLOTS_IN_MEM) return 0;
    const uint64_t words = align_up(4ull * max_slots, 16);
    return policy ? 3 * words + align_up((p.fine ? 2ull : 4ull) * max_slots, 16) : 2 * words;
}
// bytes of a slot table in global memory, and of pool[] of the fine-grained variant
inline uint64_t slot_table_bytes(uint32_t max_slots, int policy) { return align_up((uint64_t)max_slots * (policy ? 16 : 8), 16); }
inline uint64_t pool_bytes(const KParams &k, const ReplayPlan &p) { return ((uint64_t)k.cap_pblocks + 80) * (p.wide ? 8 : 4); }
const uint64_t MEM_TABLES_MAX = 1ull << 30;         // bytes of global memory that the slot tables of a launch, or its pools, may take

// Per-wave LDS layout, in 64-bit arithmetic (a table size that would wrap a 32-bit offset must end
// as "too big", not as a small layout).  Returns the bytes needed.
inline uint64_t layout(KParams &k, int policy, const vms_config &c, const ReplayPlan &p)
{
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        uint64_t at = off;
        off = align_up(off + bytes, 16);
        return (uint32_t)(at <= 0xFFFFFFFFu ? at : 0xFFFFFFFFu);
    };
    k.off_slot_req = k.off_slot_a = k.off_slot_b = k.off_slot_c = 0;
    k.off_pool = k.off_bmp = k.off_skey = k.off_smeta = k.off_sstamp = k.off_swit = k.off_tmp = k.off_arena = 0;
    k.off_bnd = k.off_soff = 0;
    if (policy) take(256);      // scalars of the trace (see replay_kernels.hpp)
    if (p.slots == SLOTS_IN_LDS) {
        k.off_slot_req = take((uint64_t)c.max_slots * 4);
        k.off_slot_a = take((uint64_t)c.max_slots * 4);
        k.off_slot_b = policy ? take((uint64_t)c.max_slots * 4) : 0;
        k.off_slot_c = policy ? take((uint64_t)c.max_slots * (p.fine ? 2 : 4)) : 0;     // 16-bit list places, or offset and length
    }
    // inactive blocks of a splitting pool beyond those held in registers
    const uint32_t in_regs = 64 * (policy ? SMALL_TILES : p.fl_tiles);
    k.off_fl = k.cap_free <= in_regs ? 0 : take(((uint64_t)k.cap_free - in_regs) * 8);
    if (policy && p.fine) {
        const uint64_t idx = p.wide ? 4 : 2;                    // bytes of a chunk number
        if (p.tbl_ws != 4) k.off_pool = take(pool_bytes(k, p));      // 64 spare places, and moves of whole 16-byte blocks
        k.off_bmp = take(((uint64_t)k.bmp_words + 1) * 4);      // and one spare word
        k.off_bnd = take(((uint64_t)k.bmp_words + 1) * 4);      // scans read one word ahead
        k.off_tmp = take(((uint64_t)k.bmp_words + 64) * 4);     // and 64 spare words
        if (p.tbl_ws < 3) k.off_skey = take(((uint64_t)c.max_sblocks + 80) * idx);    // 64 spare places, and shifts move whole 16-byte blocks
        if (!p.tbl_ws) {
            k.off_swit = take(((uint64_t)c.max_sblocks + 80) * idx);
            k.off_soff = take(((uint64_t)c.max_sblocks + 80) * 2);
        }
    } else if (policy) {
        // 64 spare places behind each searched array: reads there need no bounds check
        k.off_pool = take(((uint64_t)c.max_pblocks + 64) * 8);
        k.off_bmp = take(((uint64_t)c.max_chunks + 31) / 32 * 4 + 4);     // and one spare bitmap word
        k.off_skey = take(((uint64_t)c.max_sblocks + 64) * 8);
        k.off_smeta = take(((uint64_t)c.max_sblocks + 64) * 4);
        k.off_sstamp = take(((uint64_t)c.max_sblocks + 64) * 4);
        k.off_swit = take(((uint64_t)c.max_sblocks + 64) * 4);
        k.off_tmp = take(((uint64_t)c.max_chunks + 31) / 32 * 4 + 256);   // and 64 spare words
        k.off_arena = take(((uint64_t)c.max_runs + 64) * 4);
    }
    k.lds_bytes = (uint32_t)(off <= 0xFFFFFFFFu ? off : 0xFFFFFFFFu);
    return off;
}

}  // namespace plan_detail

// The plan for cfg with the variant it names (0: flat unless the tables are too large for it).
// VMS_OK, VMS_EINVAL / VMS_ESTRUCT for a configuration that makes no sense, VMS_ETOOBIG for tables
// that do not fit a compute unit's LDS.  Touches no device.
// slots_in_mem: slot tables of more than 64 slots in global memory, unless they take too much of it (any_size: even
// then); pool_in_mem: with all sBlock tables in the workspace pool[] goes there too, likewise.
inline int replay_plan_for(const vms_config *cfg, ReplayPlan &p, bool slots_in_mem, bool pool_in_mem = false, bool any_size = false)
{
    using namespace plan_detail;
    if (!cfg) return VMS_EINVAL;
    if (cfg->struct_size != sizeof(vms_config)) return VMS_ESTRUCT;
    const vms_config &c = *cfg;
    if (c.n_traces == 0 || c.max_events == 0 || c.max_slots == 0) return VMS_EINVAL;
    if ((c.policy_mask & ~3u) || c.policy_mask == 0) return VMS_EINVAL;
    if (!is_pow2(c.chunk_bytes) || c.chunk_bytes < UNIT || c.chunk_bytes > (1ull << 30)) return VMS_EINVAL;
    if (c.small_limit_bytes > c.chunk_bytes || c.small_limit_bytes % UNIT) return VMS_EINVAL;
    if (c.frag_limit_bytes % c.chunk_bytes) return VMS_EINVAL;
    if (c.max_free_blocks == 0 || c.max_pblocks < 4 || c.max_runs < 4 || c.max_runs > TABLE_MAX || c.max_chunks == 0)
        return VMS_EINVAL;
    if (c.max_chunks > TABLE_MAX) return VMS_EINVAL;
    if (c.max_sblocks < c.spool_threshold + 3) return VMS_EINVAL;
    if ((uint64_t)c.max_chunks * c.chunk_bytes > ENGINE_MAX_BYTES) return VMS_EINVAL;
    if ((uint64_t)c.n_traces * c.max_events > (1ull << 40)) return VMS_EINVAL;
    if (c.max_small_blocks > 192) return VMS_EINVAL;            // that pool is held in registers
    // table sizes no LDS could hold: too big, whatever a 32-bit layout would make of them
    if (c.max_slots > TABLE_MAX || c.max_free_blocks > TABLE_MAX || c.max_pblocks > TABLE_MAX || c.max_sblocks > TABLE_MAX ||
        c.max_multi_pblocks > TABLE_MAX)
        return VMS_ETOOBIG;

    memset(&p, 0, sizeof p);
    if (c.variant > VMS_VARIANT_FINE || c.table_place > VMS_TABLES_WORKSPACE_ALL) return VMS_EINVAL;
    // tables beyond what flat sorted LDS arrays serve (lists of more than 64 KB, thousands of blocks)
    // need the fine-grained variant with its lists in the workspace
    const bool big = c.max_runs > 16384 || c.max_pblocks > 4096 || c.max_sblocks > 4096;
    if (big && c.variant == VMS_VARIANT_FLAT) return VMS_ETOOBIG;
    p.fine = big || c.variant == VMS_VARIANT_FINE;
    p.wide = c.max_chunks > 63000;
    p.tbl_ws = p.fine && !p.wide && c.table_place >= VMS_TABLES_WORKSPACE ? (int)c.table_place : 0;
    if (c.table_place >= VMS_TABLES_WORKSPACE && p.fine && p.wide) return VMS_EINVAL;
    p.slot_regs = c.max_slots <= 64;
    slots_in_mem = slots_in_mem && (any_size || c.n_traces * slot_table_bytes(c.max_slots, 1) <= MEM_TABLES_MAX);
    p.slots = p.slot_regs ? SLOTS_IN_REGS : slots_in_mem ? SLOTS_IN_MEM : SLOTS_IN_LDS;
    p.fl_tiles = c.max_free_blocks <= 192 ? 3u : 5u;
    p.fl_tail = c.max_free_blocks > 320;
    uint32_t shift = 0;
    while ((UNIT << shift) < c.chunk_bytes) shift++;
    const uint64_t cap = c.capacity_bytes ? (c.capacity_bytes < ENGINE_MAX_BYTES ? c.capacity_bytes : ENGINE_MAX_BYTES)
                                          : ENGINE_MAX_BYTES;
    for (int pol = 0; pol < 2; pol++) {
        KParams &k = p.kp[pol];
        k.n_traces = c.n_traces;
        k.max_events = c.max_events;
        k.chunk_shift = shift;
        k.small_limit_units = (uint32_t)(c.small_limit_bytes / UNIT);
        // (no block has more than max_chunks chunks; the kernels make keys of this limit, in as many bits as a chunk number has)
        const uint64_t limit = c.frag_limit_bytes / c.chunk_bytes;
        k.frag_limit_chunks = limit > c.max_chunks ? c.max_chunks + 1 : (uint32_t)limit;
        k.spool_threshold = c.spool_threshold;
        k.capacity_units = (uint32_t)(cap / UNIT);
        k.max_slots = c.max_slots;
        // the stitching policy's pool for small requests may be given a size of its own
        k.cap_free = pol && c.max_small_blocks ? c.max_small_blocks : c.max_free_blocks;
        k.cap_pblocks = c.max_pblocks;
        k.cap_sblocks = c.max_sblocks;
        k.cap_runs = c.max_runs;
        k.cap_chunks = c.max_chunks;
        k.ws_stride = 0;
        if (pol && p.fine) {
            // pool[] holds the pBlocks of two or more chunks only; its rank search covers 4096 keys,
            // the one over the sBlocks 8064
            k.cap_pblocks = c.max_multi_pblocks ? c.max_multi_pblocks : (c.max_pblocks < 4096 ? c.max_pblocks : 4096);
            if (k.cap_pblocks > 4096 || c.max_sblocks > 8000) return VMS_ETOOBIG;
            k.bmp_words = (uint32_t)align_up((uint64_t)c.max_chunks / 32 + 1, 4);
            // The arena holds 8-byte words: per sBlock two header words and at most one word per
            // run, rounded up to whole granules of 2^gran_shift words.  List places are 16-bit
            // granule numbers.
            const uint64_t words = (uint64_t)c.max_runs + 5ull * c.max_sblocks;
            k.gran_shift = 2;
            while ((words >> k.gran_shift) > 65535u) k.gran_shift++;
            k.cap_grans = (uint32_t)(words >> k.gran_shift);
            if (k.cap_grans < 4) return VMS_EINVAL;
            // two halves (the lists, and where compaction copies them), each followed by 64 spare words;
            // behind them the two 16-bit tables, if they are kept here
            k.ws_half = align_up((((uint64_t)k.cap_grans << k.gran_shift) + 64) * 8, 256);
            k.ws_tbl_bytes = p.tbl_ws ? (uint32_t)align_up(((uint64_t)c.max_sblocks + 80) * 2, 256) : 0u;
            k.ws_stride = 2 * k.ws_half + (p.tbl_ws < 3 ? 2ull : 3ull) * k.ws_tbl_bytes;
            if (pool_in_mem && p.tbl_ws == 3 && c.n_traces * pool_bytes(k, p) <= MEM_TABLES_MAX) p.tbl_ws = 4;
        } else if (pol) {
            k.ws_stride = align_up(((uint64_t)c.max_runs + 64) * 4, 256);     // where compaction copies the lists
        }
        k.mem_pool = p.slots == SLOTS_IN_MEM ? slot_table_bytes(c.max_slots, pol) : 0;
        k.mem_stride = k.mem_pool + (pol && p.tbl_ws == 4 ? align_up(pool_bytes(k, p), 16) : 0);
        const uint64_t lds = layout(k, pol, c, p), need = lds + pool_bytes_saved(k, pol, p) + slot_bytes_saved(c.max_slots, pol, p);
        // flat variant: the lists' places in a slot table in LDS are there for speed only and refuse no tables; where
        // there is no room for them the slot table is in global memory, whatever it takes there
        const uint64_t lists = pol && !p.fine && !p.slot_regs ? align_up(4ull * c.max_slots, 16) : 0;
        if ((c.policy_mask & (1u << pol)) && need - lists > LDS_PER_CU) return VMS_ETOOBIG;
        if ((c.policy_mask & (1u << pol)) && lds > LDS_PER_CU) return replay_plan_for(cfg, p, true, pool_in_mem, true);
    }
    p.ws_bytes = (c.policy_mask & VMS_POLICY_VMS) ? (size_t)p.kp[1].ws_stride * c.n_traces : 0;
    return VMS_OK;
}

// LDS is handed out in granules of 1,280 bytes, 128 of them per compute unit (measured: 31,680 B per
// wavefront gives five wavefronts per compute unit, 32,576 B four).
const uint32_t PLAN_CUS = 256, PLAN_GRANULES = 128;
inline uint32_t plan_granules(uint32_t lds_bytes) { return (lds_bytes + 1279) / 1280; }

// Wavefronts of the stitching kernel that share a compute unit.  By their vector registers: four per SIMD, but three where
// the fine-grained kernel has its slot table in global memory and tables in the workspace (130 registers) or just two
// tables there (129 to 135) ...
inline uint32_t plan_waves_by_registers(const ReplayPlan &x)
{
    return x.fine && x.tbl_ws && (x.slots == SLOTS_IN_MEM || x.tbl_ws == 2) ? 12 : 16;
}
// ... and by their LDS
inline uint32_t plan_waves_per_cu(const ReplayPlan &x)
{
    const uint32_t g = plan_granules(x.kp[1].lds_bytes), most = plan_waves_by_registers(x), w = g ? PLAN_GRANULES / g : most;
    return w < most ? w : most;
}

// What a batch costs under plan x, in tenths of what one round of wavefronts of the flat variant takes.
// A round of the fine-grained variant takes 1.25 to 1.6 of that on streams of many small requests (LoRA, ZeRO-3;
// 64 to 1,280 traces x 20,000: 8.8 to 12.2 ms against 7.1 to 7.7) and 2.3 to 2.9 where every request stitches
// (recomputation, 64 to 4,096 traces: 17.1 to 23.6 against 7.3 to 8.2); what is known beforehand of the two is
// that the former hold more than 64 blocks at once.  Sblock tables in the workspace: 5 to 10 % more (offloading
// 1024x20000 58.6 -> 64.7 ms, ZeRO-3 11.8 -> 12.4); with two tables there instead of three it is not less
// (offloading 4096x50000 391 against 366 ms), so that place is taken on request only; with pool[] in global memory too
// another 5 % (offloading 2500x20000, resident at once either way, 85.1 -> 89.7 ms).
// The splitting kernel beside it takes 0.65 of a round (5 of 7.5 ms) and runs in the LDS that the stitching
// wavefronts leave, or behind them; a batch of several rounds costs its wavefronts' share of the LDS times how
// long they hold it, and half a round for the tail, but whole rounds where at most two share a SIMD and so gain
// little from a round that is not full (ZeRO-3 1280x20000 on the flat variant, 1,024 of them at a time: 14.8 ms,
// fine-grained 12.0).
// A slot table in global memory costs the flat variant 1 to 2 % (one random trace 1.057 -> 1.069 ms, scale-out
// 320x20000 7.58 -> 7.75).
// (With four wavefronts per SIMD assumed everywhere, ZeRO-3 batches of 3,585 traces and more had their tables moved to
// the workspace for a fourth that the registers have no room for: 4096x20000 23.4 ms, 21.8 with them in LDS, where
// fourteen share a compute unit; 8,192 traces 42.7 and 38.9; LoRA 4096x50000 with pool[] in global memory 54.1, without
// 53.5.)
// What the model cannot know: a stream of more than 64 slots of which every request stitches costs the fine-grained
// variant 2.4 rounds, not 1.6 (recomputation 1536x8000 with 65 slots 8.8 ms, flat 6.7), and one of 64 or fewer with the
// default tables is charged more rounds than it takes (4096x8000 on the flat variant 20.7 ms, fine-grained 15.8).
inline uint64_t plan_cost(const ReplayPlan &x, const vms_config &c)
{
    const uint64_t round = !x.fine ? 100 + (x.slots == SLOTS_IN_MEM ? 2 : 0)
                                   : (x.slot_regs ? 260 : 160) * (x.tbl_ws == 4 ? 112 : x.tbl_ws ? 106 : 100) / 100;
    const uint64_t n = c.n_traces, w = plan_waves_per_cu(x), most = plan_waves_by_registers(x), all = (uint64_t)PLAN_CUS * PLAN_GRANULES;
    if (!w) return ~0ull;
    const uint64_t lds = plan_granules(x.kp[1].lds_bytes), g3 = lds * most > PLAN_GRANULES ? 3 * lds : 3 * PLAN_GRANULES / most;     // in thirds
    const uint64_t g_split = c.policy_mask & VMS_POLICY_SPLIT ? plan_granules(x.kp[0].lds_bytes) : 0;
    if (n > PLAN_CUS * w) {
        const uint64_t shares = n * (g3 * round + 3 * g_split * 65) / (3 * all) + round / 2, rounds = (n + PLAN_CUS * w - 1) / (PLAN_CUS * w);
        return w > 8 || shares > rounds * round ? shares : rounds * round;
    }
    if (!g_split) return round;
    const uint64_t room = n * lds < all ? (all - n * lds) / g_split : 0;
    const uint64_t behind = round + (n * g_split + all - 1) / all * 65, beside = room ? (n + room - 1) / room * 65 : behind;
    const uint64_t split = beside < behind ? beside : behind;
    return split > round ? split : round;
}

// Both policies in one launch where all its workgroups are resident at once: each holds the LDS of both its
// wavefronts until the longer one, the stitching one, is done, so a batch of several rounds goes in two launches.
inline bool plan_together(const ReplayPlan &x, const vms_config &c)
{
    const uint64_t lds = (uint64_t)x.kp[0].lds_bytes + x.kp[1].lds_bytes;
    if (c.policy_mask != (VMS_POLICY_SPLIT | VMS_POLICY_VMS) || x.fine || lds > plan_detail::LDS_PER_CU) return false;
    const uint32_t g = plan_granules((uint32_t)lds), w = PLAN_GRANULES / g;
    return c.n_traces <= PLAN_CUS * (w < 8 ? w : 8);
}

// Up to this many traces of the splitting policy alone keep their slot tables in LDS (LoRA 64 and 512 x 20,000: no
// difference; 1024: 5.84 ms there, 5.59 in global memory; 2048: 6.69 and 6.50)
const uint32_t SPLIT_SLOTS_IN_LDS = 512;

// The plan for cfg.  With variant 0 and tables that both variants serve the library chooses between them, and
// with table_place 0 whether the fine-grained variant keeps the tables of the sBlocks in LDS, in the workspace, or there
// with pool[] in global memory too: whichever plan the batch costs least under.  (Scale-out
// 320x20000 11.0 -> 7.5 ms, fragmentation limit study 64x20000 9.2 -> 7.1, both fine-grained before because their
// presets said so; recomputation 2048x20000 22.9 -> 15.8, fine-grained before because the batch did not fit at once.)
inline int replay_plan_choose(const vms_config *cfg, ReplayPlan &p)
{
    int rc = replay_plan_for(cfg, p, false);
    if (rc != VMS_OK || !cfg) return rc;
    const bool stitch = cfg->policy_mask & VMS_POLICY_VMS;
    if (!stitch) return cfg->n_traces > SPLIT_SLOTS_IN_LDS ? replay_plan_for(cfg, p, true) : rc;
    const bool other = cfg->variant == VMS_VARIANT_AUTO && !p.fine;
    uint64_t best = ~0ull;
    // takes the plan if it costs less
    auto consider = [&](uint32_t variant, uint32_t place, bool slots_in_mem, bool pool_in_mem = false) {
        vms_config alt = *cfg;
        alt.variant = variant;
        alt.table_place = place;
        ReplayPlan q;
        if (replay_plan_for(&alt, q, slots_in_mem, pool_in_mem) != VMS_OK) return;
        const uint64_t c = plan_cost(q, *cfg);
        if (c < best) {
            best = c;
            p = q;
        }
    };
    if (!p.fine) consider(cfg->variant, cfg->table_place, false);
    consider(cfg->variant, cfg->table_place, true);
    if (!other && !p.fine) return VMS_OK;
    if (cfg->table_place != VMS_TABLES_AUTO) {
        if (other) consider(VMS_VARIANT_FINE, cfg->table_place, true);
    } else {
        consider(VMS_VARIANT_FINE, VMS_TABLES_LDS, true);
        consider(VMS_VARIANT_FINE, VMS_TABLES_WORKSPACE_ALL, true);
        consider(VMS_VARIANT_FINE, VMS_TABLES_WORKSPACE_ALL, true, true);
    }
    return VMS_OK;
}

// in_lds: without tables in global memory (but for those the LDS has no room for), whatever that costs
inline int replay_plan_make(const vms_config *cfg, ReplayPlan &p, bool in_lds = false)
{
    const int rc = in_lds ? replay_plan_for(cfg, p, false) : replay_plan_choose(cfg, p);
    if (rc == VMS_OK) p.together = plan_together(p, *cfg);
    return rc;
}

// The plan of the second pass for cfg: every table doubled, as far as the fine-grained variant and a
// compute unit's LDS allow.  VMS_OK and q.has_retry = false if no larger plan exists.
inline int replay_plan_retry(const vms_config *cfg, const ReplayPlan &first, ReplayPlan &q)
{
    memset(&q, 0, sizeof q);
    if (!cfg->retry_traces) return VMS_OK;
    vms_config big = *cfg;
    auto twice = [](uint32_t x, uint32_t cap) -> uint32_t { return (uint64_t)x * 2 > cap ? cap : x * 2; };
    big.variant = VMS_VARIANT_FINE;
    big.max_free_blocks = twice(cfg->max_free_blocks, 1u << 14);
    big.max_small_blocks = 0;
    big.max_pblocks = twice(cfg->max_pblocks, 1u << 20);
    big.max_multi_pblocks = twice(first.fine ? first.kp[1].cap_pblocks : cfg->max_pblocks, 4096);
    big.max_sblocks = twice(cfg->max_sblocks, 8000);
    big.max_runs = twice(cfg->max_runs < (1u << 16) ? (1u << 16) : cfg->max_runs, plan_detail::TABLE_MAX);
    big.max_chunks = twice(cfg->max_chunks, plan_detail::TABLE_MAX);
    while ((uint64_t)big.max_chunks * big.chunk_bytes > plan_detail::ENGINE_MAX_BYTES) big.max_chunks /= 2;
    // shrink towards the first pass's sizes until the tables fit; that of the multi-chunk pBlocks, of which a handle may
    // name more than pBlocks, when the others have been
    const uint32_t multi = first.fine ? first.kp[1].cap_pblocks : 0;
    for (int tries = 0; tries < 11; tries++) {
        const int rc = replay_plan_for(&big, q, first.slots == SLOTS_IN_MEM);
        if (rc == VMS_OK) {
            q.has_retry = true;
            for (int pol = 0; pol < 2; pol++) {
                q.kp[pol].retry = 1;
                q.kp[pol].retry_slots = cfg->retry_traces;
                q.kp[pol].retry_ws_off = first.ws_bytes;
            }
            q.ws_bytes = (cfg->policy_mask & VMS_POLICY_VMS) ? (size_t)q.kp[1].ws_stride * cfg->retry_traces : 0;
            return VMS_OK;
        }
        if (rc != VMS_ETOOBIG) return rc;
        big.max_chunks = big.max_chunks / 2 > cfg->max_chunks ? big.max_chunks / 2 : cfg->max_chunks;
        big.max_sblocks = big.max_sblocks * 3 / 4 > cfg->max_sblocks ? big.max_sblocks * 3 / 4 : cfg->max_sblocks;
        big.max_free_blocks = big.max_free_blocks / 2 > cfg->max_free_blocks ? big.max_free_blocks / 2 : cfg->max_free_blocks;
        if (tries >= 7 && multi) big.max_multi_pblocks = big.max_multi_pblocks * 3 / 4 > multi ? big.max_multi_pblocks * 3 / 4 : multi;
    }
    memset(&q, 0, sizeof q);
    return VMS_OK;
}

// For a handle whose own plans need more than `room` bytes of workspace: those that need least, with first.ws_bytes 0
// if they need more than that too.
inline void replay_plan_small(const vms_config *cfg, uint64_t room, ReplayPlan &first, ReplayPlan &second)
{
    if (replay_plan_for(cfg, first, false) != VMS_OK || replay_plan_retry(cfg, first, second) != VMS_OK ||
        first.ws_bytes + second.ws_bytes > room)
        first.ws_bytes = 0;
}

// wavefronts of the second pass
inline uint32_t plan_second_pass_waves(const vms_config &c) { return c.retry_traces < c.n_traces ? c.retry_traces : c.n_traces; }

// The tables of a run that are in global memory, those of each launch behind those of the one before: returns their
// bytes, and with `mem` says where each launch finds its own.
inline uint64_t plan_place_tables(const vms_config &c, ReplayPlan &first, ReplayPlan &second, char *mem)
{
    uint64_t bytes = 0;
    for (int pass = 0; pass < (second.has_retry ? 2 : 1); pass++)
        for (int pol = 0; pol < 2; pol++) {
            if (!(c.policy_mask & (1u << pol))) continue;
            KParams &k = (pass ? second : first).kp[pol];
            if (mem) k.mem = mem + bytes;
            bytes += plan_detail::align_up(k.mem_stride * (pass ? plan_second_pass_waves(c) : c.n_traces), 256);
        }
    return bytes;
}

#endif

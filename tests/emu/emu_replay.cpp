// TEST INFRASTRUCTURE ONLY.  Compiles the replay kernels for the host on top of wave_hw_emu.hpp
// (64 lanes as cooperative fibers) so that their indexing and results can be checked on the CPU:
// every device buffer and the LDS get guard bands that are verified after each wavefront.  The
// product never loads this; it exists to find out-of-bounds accesses and wrong decisions without a GPU.
#include "wave_hw_emu.hpp"

#include "../../paper_2401_08156_amd/csrc/replay_kernels.hpp"
#include "../../paper_2401_08156_amd/csrc/replay_fine.hpp"
#include "../../paper_2401_08156_amd/csrc/selftest.hpp"

#include <vector>

namespace emu {
int cur;
u32 wave;
ucontext_t ctx[LANES], back;
u64 xchg[2][LANES];
u64 n_coll;
u64 coll_of[LANES];
bool trace_on = getenv("VMS_EMU_TRACE") != nullptr;
static std::vector<void *> g_sites[LANES];
void note(void *site) { g_sites[cur].push_back(site); }
static void (*g_body)(void *);
static void *g_arg;
static std::vector<char> g_stacks;

static void trampoline(int lane)
{
    g_body(g_arg);
    cur = lane + 1;         // this lane is done: the next one runs on from where it last switched
}

void launch(void (*body)(void *), void *arg, u32 block)
{
    const size_t STACK = 1 << 20;
    if (g_stacks.empty()) g_stacks.resize(STACK * LANES);
    g_body = body;
    g_arg = arg;
    blockIdx.x = block;
    for (int l = 0; l < LANES; l++) {
        coll_of[l] = 0;
        g_sites[l].clear();
        getcontext(&ctx[l]);
        ctx[l].uc_stack.ss_sp = g_stacks.data() + STACK * l;
        ctx[l].uc_stack.ss_size = STACK;
        ctx[l].uc_link = l + 1 < LANES ? &ctx[l + 1] : &back;
        makecontext(&ctx[l], (void (*)())trampoline, 1, l);
    }
    cur = 0;
    swapcontext(&back, &ctx[0]);
    for (int l = 1; l < LANES; l++)
        if (coll_of[l] != coll_of[0]) {
            if (trace_on) {
                size_t i = 0;
                while (i < g_sites[0].size() && i < g_sites[l].size() && g_sites[0][i] == g_sites[l][i]) i++;
                fprintf(stderr, "emu: first difference at operation %zu: lane 0 at %p, lane %d at %p (previous %p)\n", i,
                        i < g_sites[0].size() ? g_sites[0][i] : nullptr, l, i < g_sites[l].size() ? g_sites[l][i] : nullptr,
                        i ? g_sites[0][i - 1] : nullptr);
            }
            fprintf(stderr, "emu: lane %d passed %llu wave-wide operations, lane 0 %llu: divergent control flow\n", l,
                    (unsigned long long)coll_of[l], (unsigned long long)coll_of[0]);
            abort();
        }
}
}  // namespace emu

emu::Dim blockIdx;
const size_t LDS_MAX = 160 * 1024, GUARD = 4096;
alignas(16) char lds[LDS_MAX + GUARD];

namespace {

const unsigned char CANARY = 0xA5;

// a device buffer with guard bands on both sides
struct Guarded {
    std::vector<char> mem;
    size_t bytes;
    Guarded(size_t n) : mem(n + 2 * GUARD + 256, (char)CANARY), bytes(n) {}
    char *ptr() { return (char *)(((uintptr_t)mem.data() + GUARD + 255) & ~(uintptr_t)255); }
    bool intact()
    {
        char *p = ptr();
        for (char *q = mem.data(); q < p; q++)
            if ((unsigned char)*q != CANARY) return false;
        for (char *q = p + bytes; q < mem.data() + mem.size(); q++)
            if ((unsigned char)*q != CANARY) return false;
        return true;
    }
};

struct Args {
    KParams P, P_split;
    const u64 *events;
    const u32 *n_events;
    u64 *dec;
    vms_trace_stats *stats;
    char *ws;
    const ReplayPlan *plan;
};

// the kernel of a plan, as the library picks it
template <int SLOTS>
void vms_with(const ReplayPlan &p, Args &a)
{
    if (!p.fine) return replay_vms_kernel<SLOTS>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
    if (p.wide) return replay_vms_fine_kernel<SLOTS, u32, 0>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
    if (p.tbl_ws == 4) return replay_vms_fine_kernel<SLOTS, uint16_t, 4>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
    if (p.tbl_ws == 3) return replay_vms_fine_kernel<SLOTS, uint16_t, 3>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
    if (p.tbl_ws) return replay_vms_fine_kernel<SLOTS, uint16_t, 2>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
    replay_vms_fine_kernel<SLOTS, uint16_t, 0>(a.P, a.events, a.n_events, a.dec, a.stats, a.ws);
}
template <int SLOTS>
void split_with(const ReplayPlan &p, Args &a)
{
    if (p.fl_tiles == 3) return replay_split_kernel<SLOTS, 3, false>(a.P, a.events, a.n_events, a.dec, a.stats);
    if (p.fl_tail) return replay_split_kernel<SLOTS, 5, true>(a.P, a.events, a.n_events, a.dec, a.stats);
    replay_split_kernel<SLOTS, 5, false>(a.P, a.events, a.n_events, a.dec, a.stats);
}
// both policies in one launch: only the wavefront emu::wave of the workgroup runs
template <int SLOTS>
void both_with(const ReplayPlan &p, Args &a)
{
    if (p.fl_tiles == 3) return replay_both_kernel<SLOTS, 3, false>(a.P, a.P_split, a.events, a.n_events, a.dec, a.dec, a.stats, a.ws);
    if (p.fl_tail) return replay_both_kernel<SLOTS, 5, true>(a.P, a.P_split, a.events, a.n_events, a.dec, a.dec, a.stats, a.ws);
    replay_both_kernel<SLOTS, 5, false>(a.P, a.P_split, a.events, a.n_events, a.dec, a.dec, a.stats, a.ws);
}
#define BY_SLOTS(f)                                                        \
    {                                                                      \
        Args &a = *(Args *)x;                                              \
        const ReplayPlan &p = *a.plan;                                     \
        if (p.slots == SLOTS_IN_REGS) f<SLOTS_IN_REGS>(p, a);              \
        else if (p.slots == SLOTS_IN_MEM) f<SLOTS_IN_MEM>(p, a);           \
        else f<SLOTS_IN_LDS>(p, a);                                        \
    }
void body_vms(void *x) BY_SLOTS(vms_with)
void body_split(void *x) BY_SLOTS(split_with)
void body_both(void *x) BY_SLOTS(both_with)

u32 g_selftest_fail;
void body_selftest(void *tab) { selftest_kernel(&g_selftest_fail, (uint16_t *)tab); }

}  // namespace

enum { PLAN_OF_LIBRARY, PLAN_POOL_IN_MEM, PLAN_SMALL, PLAN_IN_LDS };
static int g_plan;

extern "C" {

// what tests ask of a plan
struct emu_plan_info {
    uint32_t fine, slots, tbl_ws, has_retry, lds_bytes[2];
    uint64_t mem_stride[2], cost;
};

// the plan that emu_replay runs (and emu_plan tells of, if it is the first or the last): the library's; the fine-grained variant with all its tables out of the LDS, which the
// library plans for large batches only; the one that needs least workspace; the one without
// tables in global memory
void emu_use_plan(int which) { g_plan = which; }

// Replays every trace under the policies of cfg->policy_mask with the kernels the library would
// launch.  dec_split / dec_vms: [n_traces][max_events] or NULL; stats: [2][n_traces].
// Returns 0, a VMS_E* code from planning, or -100 - k if guard band k was written
// (1 LDS, 2 decisions, 3 statistics, 4 workspace, 5 tables in global memory).
int emu_replay(const vms_config *cfg, const uint64_t *events, const uint32_t *n_events, uint64_t *dec_split,
               uint64_t *dec_vms, vms_trace_stats *stats)
{
    ReplayPlan plan, again;
    int rc = replay_plan_make(cfg, plan, g_plan == PLAN_IN_LDS);
    if (rc == VMS_OK && g_plan == PLAN_POOL_IN_MEM) rc = replay_plan_for(cfg, plan, true, true);
    if (rc == VMS_OK && g_plan != PLAN_SMALL) rc = replay_plan_retry(cfg, plan, again);
    if (rc == VMS_OK && g_plan == PLAN_SMALL) replay_plan_small(cfg, ~0ull, plan, again);
    if (rc != VMS_OK) return rc;
    if (again.has_retry)
        for (int pol = 0; pol < 2; pol++) plan.kp[pol].retry_slots = cfg->retry_traces;
    const size_t n = (size_t)cfg->n_traces * cfg->max_events, ws_bytes = plan.ws_bytes + again.ws_bytes;
    Guarded g_dec(n * 8), g_stats(sizeof(vms_trace_stats) * (2 * cfg->n_traces + 1)), g_ws(ws_bytes ? ws_bytes : 256);
    memset(g_stats.ptr(), 0, g_stats.bytes);
    Guarded g_mem(plan_place_tables(*cfg, plan, again, nullptr));
    plan_place_tables(*cfg, plan, again, g_mem.ptr());
    for (int pol = 0; pol < 2; pol++) {
        if (!(cfg->policy_mask & (1u << pol))) continue;
        Args a;
        a.P = plan.kp[pol];
        a.events = events;
        a.n_events = n_events;
        uint64_t *out = pol ? dec_vms : dec_split;
        a.dec = out ? (u64 *)g_dec.ptr() : nullptr;
        a.stats = (vms_trace_stats *)g_stats.ptr();
        a.ws = g_ws.ptr();
        if (out) memset(g_dec.ptr(), 0xFF, n * 8);
        for (int pass = 0; pass < (again.has_retry ? 2 : 1); pass++) {
            const ReplayPlan &pl = pass ? again : plan;
            a.P = pl.kp[pol];
            a.plan = &pl;
            const bool together = plan.together && !pass;
            if (together) {
                a.P = plan.kp[1];
                a.P_split = plan.kp[0];
                emu::wave = pol ? 0 : 1;
            }
            // this wavefront's part of the LDS
            const size_t lds_from = together && !pol ? plan.kp[1].lds_bytes : 0, lds_to = lds_from + pl.kp[pol].lds_bytes;
            // the second pass is a launch of retry_traces wavefronts that share out the flagged traces
            const u32 waves = pass ? std::min(cfg->retry_traces, cfg->n_traces) : cfg->n_traces;
            for (u32 t = 0; t < waves; t++) {
                memset(lds, CANARY, sizeof lds);
                emu::launch(together ? body_both : pol ? body_vms : body_split, &a, t);
                for (size_t i = 0; i < sizeof lds; i++)
                    if ((i < lds_from || i >= lds_to) && (unsigned char)lds[i] != CANARY) return -101;
            }
        }
        if (!g_dec.intact()) return -102;
        if (!g_stats.intact()) return -103;
        if (!g_ws.intact()) return -104;
        if (!g_mem.intact()) return -105;
        if (out) memcpy(out, g_dec.ptr(), n * 8);
    }
    memcpy(stats, g_stats.ptr(), sizeof(vms_trace_stats) * 2 * cfg->n_traces);
    return 0;
}

// What the library plans for cfg (has_retry: a second pass too); with tables_in_mem >= 0 instead the one plan of the variant
// and table place that cfg names, with its slot tables (bit 0) and pool[] (bit 1) in global memory.  Returns VMS_OK or a
// VMS_E* code.
int emu_plan(const vms_config *cfg, int tables_in_mem, emu_plan_info *out)
{
    ReplayPlan p, again;
    int rc = tables_in_mem < 0 ? replay_plan_make(cfg, p, g_plan == PLAN_IN_LDS) : replay_plan_for(cfg, p, tables_in_mem & 1, tables_in_mem & 2);
    if (rc == VMS_OK) rc = replay_plan_retry(cfg, p, again);
    if (rc != VMS_OK) return rc;
    out->has_retry = again.has_retry;
    out->cost = plan_cost(p, *cfg);
    out->fine = p.fine;
    out->slots = p.slots;
    out->tbl_ws = p.tbl_ws;
    for (int pol = 0; pol < 2; pol++) {
        out->lds_bytes[pol] = p.kp[pol].lds_bytes;
        out->mem_stride[pol] = p.kp[pol].mem_stride;
    }
    return VMS_OK;
}

// the wave primitives' self-test kernel on the host lanes: 0, its failure bits, or 0xFFFFFFFF if a guard band was written
unsigned emu_selftest(void)
{
    Guarded tab((size_t)SELFTEST_TABLES * SELFTEST_PLACES * sizeof(uint16_t));
    g_selftest_fail = 0xFFFFFFFFu;
    emu::launch(body_selftest, tab.ptr(), 0);
    return tab.intact() ? g_selftest_fail : 0xFFFFFFFFu;
}

}  // extern "C"

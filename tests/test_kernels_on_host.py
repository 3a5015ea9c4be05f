"""The replay kernels compiled for the host (tests/emu: 64 lanes as cooperative fibers, guard bands
around the LDS and every buffer) against the oracle: finds wrong indexing and wrong decisions
without a GPU.  The lanes run one after another between wave-wide operations, so what this checks
is the kernels' logic and memory accesses, not their timing; the GPU parity tests remain the
proof for the device."""
import glob
import os

import numpy as np
import pytest

import emu
import gpu_util
import oracle
from paper_2401_08156_amd import binding, workloads
from paper_2401_08156_amd import tracegen as tg
from test_oracle_examples import GOLDEN, load_fixture

MiB = 1 << 20


def check(ev, cfg, n_events=None, label="", **kw):
    ds, dv, st = emu.replay(ev, cfg, binding.STATS_DTYPE, n_events, **kw)
    P = gpu_util.oracle_params(cfg)
    for pol, gdec in ((0, ds), (1, dv)):
        if not (cfg.policy_mask & (1 << pol)):
            continue
        odec, ost = oracle.replay(ev, P, pol, n_events=n_events, threads=8)
        gst = st[pol]
        assert not (gst["status"] & binding.VMS_ST_TABLE_OVERFLOW).any(), (label, pol, gst["status"], gst["overflow_event"])
        valid = np.ones(ev.shape, dtype=bool) if n_events is None else np.arange(ev.shape[1])[None, :] < np.asarray(n_events)[:, None]
        same = (gdec == odec) | ~valid
        if not same.all():
            t, i = np.argwhere(~same)[0]
            raise AssertionError("%s policy %d trace %d event %d: kernel %#x oracle %#x" % (label, pol, t, i, int(gdec[t, i]), int(odec[t, i])))
        assert np.all(gdec[~valid] == np.uint64(0xFFFFFFFFFFFFFFFF)), "wrote past the end of a trace"
        for f in gpu_util.COMPARED_FIELDS:
            assert np.array_equal(gst[f], ost[f]), (label, pol, f, gst[f], ost[f])
    return st


def test_wave_primitives_on_host_lanes():
    assert emu.lib().emu_selftest() == 0


def test_worked_examples_fine_grained_variant():
    for path in sorted(glob.glob(os.path.join(GOLDEN, "*.txt"))):
        fx = load_fixture(path)
        ev = fx["events"][None, :]
        kw = dict(spool_threshold=int(fx["spool_threshold"])) if "spool_threshold" in fx else {}
        for place in (binding.VMS_TABLES_LDS, binding.VMS_TABLES_WORKSPACE, binding.VMS_TABLES_WORKSPACE_ALL):
            cfg = gpu_util.make_cfg(1, ev.shape[1], 16, variant=binding.VMS_VARIANT_FINE, table_place=place, policy_mask=2, **kw)
            check(ev, cfg, label=os.path.basename(path))


def test_splitting_kernels():
    ev, ms = tg.generate(1, n_traces=2, n_events=1500)
    check(ev, gpu_util.make_cfg(2, 1500, ms, policy_mask=1), label="pool in LDS")
    check(ev, gpu_util.make_cfg(2, 1500, ms, policy_mask=1, max_free_blocks=150), label="pool in registers")
    check(ev, gpu_util.make_cfg(2, 1500, ms, policy_mask=1, max_free_blocks=300), label="pool in five registers per lane")
    ev, ms = tg.generate(4, n_traces=1, n_events=2000)
    check(ev, gpu_util.make_cfg(1, 2000, ms, policy_mask=1), label="slot table in LDS")
    check(ev, gpu_util.make_cfg(1, 2000, ms, policy_mask=1, max_free_blocks=320), label="slot table in LDS, pool in five registers per lane")
    ev, ms = tg.generate(3, n_traces=1, n_events=2000)
    assert ms <= 64
    check(ev, gpu_util.make_cfg(1, 2000, ms, policy_mask=1, max_free_blocks=320), label="slot table and pool (five per lane) in registers")


@pytest.mark.parametrize("blocks,cap", [(1, 64), (63, 192), (65, 192), (192, 192), (193, 320), (320, 320)])
@pytest.mark.parametrize("small", [False, True])
def test_splitting_pool_of_equal_blocks(blocks, cap, small):
    ev, ms = gpu_util.equal_blocks_trace(blocks, small, seed=blocks)
    cap = max(cap, 192 if small else 0)
    cfg = gpu_util.make_cfg(1, ev.shape[1], ms, policy_mask=1, max_free_blocks=cap)
    check(ev, cfg, label="%d equal blocks" % blocks)
    if small and blocks <= 96:
        check(ev, gpu_util.make_cfg(1, ev.shape[1], ms, variant=2, max_free_blocks=cap), label="pool for small requests")


# whole segments freed side by side do not merge, their own pieces do; from 256 GiB on the address
# takes all its bits
@pytest.mark.parametrize("cap", [64, 320])
def test_segments_that_touch_do_not_merge(cap):
    rng, ops, live, n = np.random.default_rng(cap), [], [], 0
    for i in range(400):
        if live and rng.random() < (0.2 if i % 100 < 50 else 0.8):
            ops.append(("F", live.pop(rng.integers(len(live)))))
        else:
            ops.append(("A", n, int(rng.choice([1, 2, 8, 32, 64])) << int(rng.choice([21, 30]))))
            live.append(n)
            n += 1
    ev = tg.make_events(ops)[None, :]
    st = check(ev, gpu_util.make_cfg(1, ev.shape[1], n, policy_mask=1, max_free_blocks=cap), label="segments side by side")
    assert st["n_merge"][0, 0] > 20 and st["peak_reserved"][0, 0] > 256 << 30


# pools of more blocks than the registers hold (192 or 320): the rest is in LDS.  Rounds that fill the pool (every
# other one of a row of blocks is freed), churn and drain it, with few sizes (equal ones in the registers and in LDS
# at once) and with many
@pytest.mark.parametrize("pol,row,sizes", [(0, 900, 4), (0, 900, 600), (1, 600, 4), (1, 600, 600)])
def test_splitting_pool_beyond_the_registers(pol, row, sizes):
    rng, ops, live, slots = np.random.default_rng(row + sizes), [], [], list(range(2000))
    def alloc():
        live.append(slots.pop(0))
        ops.append(("A", live[-1], int(rng.integers(1, sizes + 1)) * 512))
    def free(i):
        slots.append(live.pop(i))
        ops.append(("F", slots[-1]))
    for _ in range(2):
        for _ in range(row):
            alloc()
        for s in rng.permutation(live[::2]):
            free(live.index(s))
        for _ in range(500):
            if rng.random() < 0.5:
                alloc()
            else:
                free(int(rng.integers(len(live))))
        while len(live) > 40:
            free(int(rng.integers(len(live))))
    ev = tg.make_events(ops)[None, :]
    cfg = gpu_util.make_cfg(1, ev.shape[1], 2000, policy_mask=1 << pol, variant=binding.VMS_VARIANT_FINE if pol else 0, max_free_blocks=1024)
    st = check(ev, cfg, label="a pool beyond the registers")
    assert st["max_free_blocks"][pol, 0] > (192 if pol else 320) + 30


# pools in three and five registers per lane and in LDS; the stitching policy's pool in registers and in LDS
@pytest.mark.parametrize("pol,blocks,small", [(0, 64, 0), (0, 190, 0), (0, 250, 0), (0, 400, 0), (1, 64, 64), (1, 190, 190), (1, 250, 0)])
def test_free_that_outgrows_the_splitting_pool(pol, blocks, small):
    ev, ms = gpu_util.alternate_frees_trace(blocks)
    cfg = gpu_util.make_cfg(1, ev.shape[1], ms, policy_mask=1 << pol, variant=binding.VMS_VARIANT_FINE if pol else 0,
                            max_free_blocks=blocks, max_small_blocks=small)
    gpu_util.assert_free_outgrows_pool(lambda e, c: emu.replay(e, c, binding.STATS_DTYPE), cfg, ev, pol, binding.VMS_ST_OVF_FREE_BLOCKS)


@pytest.mark.parametrize("kind,nt,ne,tables", [
    (1, 2, 2000, dict(max_runs=20000)),
    (2, 2, 3000, dict(max_runs=20000)),
    (3, 2, 4000, dict(max_pblocks=4096, max_sblocks=2048, max_runs=1 << 18, max_chunks=16384)),
    (3, 2, 3000, dict(max_pblocks=4096, max_sblocks=2048, max_runs=1 << 18, max_chunks=16384, spool_threshold=32)),
    (4, 1, 3000, dict(max_runs=20000, max_chunks=32768)),                       # slot table in LDS
    (1, 1, 1500, dict(max_runs=20000, max_chunks=70000)),                       # 32-bit chunk numbers
    (2, 1, 3000, dict(variant=2, max_runs=600, spool_threshold=40, max_sblocks=128)),   # small arena: lists are squeezed
    (1, 2, 1200, dict(variant=2, frag_limit_bytes=8 * MiB, small_limit_bytes=512)),
    (1, 2, 1200, dict(variant=2, capacity_bytes=256 * MiB)),
])
def test_fine_grained_variant(kind, nt, ne, tables):
    # the witness and list-place tables of the sBlocks in LDS, then in the workspace (16-bit chunk numbers only)
    ev, ms = tg.generate(kind, n_traces=nt, n_events=ne, seed=7 + kind)
    for place in (binding.VMS_TABLES_LDS, binding.VMS_TABLES_WORKSPACE, binding.VMS_TABLES_WORKSPACE_ALL):
        if place != binding.VMS_TABLES_LDS and tables.get("max_chunks", 0) > 63000:
            continue
        cfg = gpu_util.make_cfg(nt, ne, ms, policy_mask=2, **dict(dict(variant=2), table_place=place, **tables))
        check(ev, cfg, label="generator %d %s tables %d" % (kind, tables, place))


@pytest.mark.parametrize("kind,nt,ne,kw", [
    (1, 1, 2000, dict(spool_threshold=8)),
    (1, 2, 1200, dict(frag_limit_bytes=8 * MiB, small_limit_bytes=512)),
    (1, 2, 1200, dict(capacity_bytes=256 * MiB)),
    (2, 1, 3000, dict(max_runs=700, spool_threshold=40, max_sblocks=128)),             # small arena: lists are squeezed
    (4, 1, 14000, dict(max_runs=700, spool_threshold=16, max_sblocks=92)),             # the same under a slot table in LDS
])
def test_flat_variant(kind, nt, ne, kw):
    ev, ms = tg.generate(kind, n_traces=nt, n_events=ne, seed=7 + kind)
    check(ev, gpu_util.make_cfg(nt, ne, ms, policy_mask=2, variant=binding.VMS_VARIANT_FLAT, **kw), label="generator %d" % kind)


# both policies in one launch: slot table in registers and in LDS, the splitting pool in three and five registers per
# lane and beyond; the wavefronts' parts of the LDS are told apart by guard bytes
@pytest.mark.parametrize("kind,free", [(2, 192), (2, 320), (2, 512), (4, 192), (4, 320), (1, 512)])
def test_both_policies_in_one_launch(kind, free):
    ev, ms = tg.generate(kind, n_traces=2, n_events=1000, seed=3)
    ev = ev[:, :1000]
    check(ev, gpu_util.make_cfg(2, 1000, ms, variant=binding.VMS_VARIANT_FLAT, max_free_blocks=free, retry_traces=1),
          n_events=np.array([1000, 937], dtype=np.uint32), label="generator %d, %d free blocks" % (kind, free))


# The library's choice for the presets by the number of traces: flat while a batch fits the compute units at once beside
# its splitting kernel, then the fine-grained variant, then its tables in the workspace, where that was measured to be
# the fastest of the plans (with slot tables in global memory and tables in the workspace the vector registers allow three
# wavefronts per SIMD, not four: ZeRO-3 stays in LDS)
@pytest.mark.parametrize("config,slots,sizes", [
    (2, 64, [(1024, 40208), (2048, 40208), (3072, 8944), (4096, 8944)]),
    (3, 64, [(64, 31984), (1280, 31984), (1281, 16144), (2304, 16144), (2305, 4432), (2560, 4432), (4096, 4432)]),
    (4, 650, [(64, 49616), (512, 49616), (1024, 39184), (1280, 14320), (2560, 14320), (3584, 10384), (4096, 10384), (8192, 10384)]),
    (6, 1163, [(64, 50608), (512, 50608), (1024, 31984), (1280, 31984), (1281, 10464), (3585, 10464), (4096, 10464), (8192, 10464)])])
def test_plan_of_a_batch_by_its_size(config, slots, sizes):
    for n, lds in sizes:
        rc, out = emu.plan(workloads.make_config(binding, config, n, 20000, slots))
        assert rc == 0 and out.lds_bytes[1] == lds, (config, n, rc, out.lds_bytes[1])


# ... and it costs no more than any other plan there is
@pytest.mark.parametrize("config,slots", [(1, 110), (1, 650), (2, 64), (2, 65), (3, 64), (4, 650), (6, 1163)])
@pytest.mark.parametrize("policies", [2, 3])
def test_plan_of_a_batch_costs_least(config, slots, policies):
    for n in [1, 64, 300, 512, 768, 1024, 1281, 1600, 2048, 2305, 2561, 3072, 3585, 4096, 5461, 8192, 16384]:
        cfg = workloads.make_config(binding, config, n, 20000, slots, policy_mask=policies)
        costs = {}
        for variant, place, in_mem in [(1, 0, 0), (1, 0, 1), (2, 1, 1), (2, 3, 1), (2, 3, 3)]:
            rc, p = emu.plan(workloads.make_config(binding, config, n, 20000, slots, policy_mask=policies, variant=variant, table_place=place),
                             tables_in_mem=in_mem)
            if rc == 0:
                costs[variant, place, in_mem] = p.cost
        rc, p = emu.plan(cfg)
        assert rc == 0 and len(costs) == (3 if config == 3 else 5) and p.cost == min(costs.values()), (n, p.cost, costs)


# slot tables in registers (up to 64 slots), in LDS (flat variant) and in global memory; a capacity that is reached, and an arena that is squeezed often
@pytest.mark.parametrize("slots", [3, 64, 65, 300])
@pytest.mark.parametrize("kw", [dict(policy_mask=1), dict(variant=1), dict(variant=2, capacity_bytes=192 * MiB),
                                dict(variant=1, spool_threshold=4, max_sblocks=128, max_runs=900),
                                dict(variant=2, table_place=binding.VMS_TABLES_WORKSPACE_ALL, spool_threshold=4, max_sblocks=128, max_runs=160)])
def test_events_that_follow_each_other_on_a_slot(slots, kw):
    ev, n = gpu_util.slot_reuse_traces(slots, 64 * 9, seed=slots)
    st = check(ev, gpu_util.make_cfg(4, ev.shape[1], slots, **kw), n_events=n, label="%d slots" % slots)
    assert (st["n_code"][:, :, 7][st["n_code"].sum(axis=2) > 0] > 20).all()


def test_ragged_traces_and_nothing_written_past_the_end():
    ev, ms = tg.generate(1, n_traces=3, n_events=700, seed=11)
    check(ev, gpu_util.make_cfg(3, 700, ms, max_runs=20000), n_events=np.array([0, 333, 700], dtype=np.uint32), label="ragged")


def test_second_pass_replays_traces_that_outgrow_the_tables():
    # tables far too small for the first trace's pools (the other two fit): flagged without a second
    # pass, replayed in full with doubled tables with one
    ev, ms = tg.generate(1, n_traces=3, n_events=900, seed=13)
    ev[1:, 60:] = ev[1:, :1] * 0 + tg.make_events([("A", 0, 2 * MiB), ("F", 0)] * 420)[None, :]
    for variant in (binding.VMS_VARIANT_FINE, binding.VMS_VARIANT_FLAT):
        small = dict(variant=variant, max_free_blocks=24, max_pblocks=40, max_sblocks=560, max_runs=900, max_chunks=8192)
        _, _, st = emu.replay(ev, gpu_util.make_cfg(3, 900, ms, **small), binding.STATS_DTYPE)
        assert (st["status"][:, 0] & binding.VMS_ST_TABLE_OVERFLOW).all() and not (st["status"][:, 1:] & binding.VMS_ST_TABLE_OVERFLOW).any()
        check(ev, gpu_util.make_cfg(3, 900, ms, retry_traces=2, **small), label="second pass, first pass variant %d" % variant)
        # both passes with the sBlock tables in the workspace
        check(ev, gpu_util.make_cfg(3, 900, ms, retry_traces=2, table_place=binding.VMS_TABLES_WORKSPACE_ALL, **small),
              label="second pass, tables in the workspace")
    # more such traces than the second pass has wavefronts: one wavefront replays all three in turn
    ev, ms = tg.generate(1, n_traces=3, n_events=900, seed=13)
    cfg = gpu_util.make_cfg(3, 900, ms, policy_mask=2, variant=2, max_pblocks=40, max_sblocks=560)
    _, _, st = emu.replay(ev, cfg, binding.STATS_DTYPE)
    assert ((st["status"][1] & binding.VMS_ST_TABLE_OVERFLOW) != 0).sum() == 3
    check(ev, gpu_util.make_cfg(3, 900, ms, retry_traces=1, variant=2, max_pblocks=40, max_sblocks=560), label="second pass of one wavefront")
    # 70 traces, every third flagged: the wavefronts take their trace numbers 64 at a time
    ev, ms = tg.generate(1, n_traces=70, n_events=300, seed=21)
    ev[np.arange(70) % 3 != 0, 10:] = tg.make_events([("A", 0, 2 * MiB), ("F", 0)] * 145)[None, :]
    small = dict(variant=2, max_free_blocks=24, max_pblocks=24, max_sblocks=560, max_runs=900, max_chunks=8192)
    _, _, st = emu.replay(ev, gpu_util.make_cfg(70, 300, ms, **small), binding.STATS_DTYPE)
    assert 10 < (st["status"] & binding.VMS_ST_TABLE_OVERFLOW != 0).any(axis=0).sum() <= 24
    check(ev, gpu_util.make_cfg(70, 300, ms, retry_traces=3, **small), label="second pass over 70 traces")


def test_lists_are_compacted_under_a_slot_table_in_lds():
    # 650 slots (in LDS: list places are halfwords there), a StitchFree threshold of 16 and an arena
    # of 290 granules: the 408 sBlocks this trace stitches take more granules than that one after the
    # other, so their lists are squeezed together several times and the slots that hold one learn
    # its new place; every later FREE of such a slot must still find the right list
    ev, ms = tg.generate(4, n_traces=1, n_events=14000, seed=3)
    assert ms > 64
    for place in (binding.VMS_TABLES_LDS, binding.VMS_TABLES_WORKSPACE_ALL):
        cfg = gpu_util.make_cfg(1, 14000, ms, policy_mask=2, variant=binding.VMS_VARIANT_FINE, table_place=place, spool_threshold=16,
                                max_pblocks=1024, max_sblocks=92, max_runs=700, max_chunks=20480)
        st = check(ev, cfg, label="compaction, slot table in LDS, tables %d" % place)
        assert st["n_sblock_created"][1, 0] > 400 and st["n_sblock_evicted"][1, 0] > 300


# List places take all 16 bits, whatever the slots that hold them: lists of a thousand words each, until they reach
# behind granule 32,767 of an arena of 43,200, then hits on the sBlocks that have them
@pytest.mark.parametrize("place", [1, 3])
@pytest.mark.parametrize("in_lds", [False, True])
def test_list_places_of_sixteen_bits(place, in_lds):
    chunk, n = 2 * MiB, 1000
    ops = [op for i in range(n) for op in (("A", 2 * i, chunk), ("A", 2 * i + 1, 31 * chunk))] + [("F", 2 * i) for i in range(n)]
    sizes = [n - i for i in range(160)]
    ops += [op for size in sizes + sizes[::-1] for op in (("A", 0, size * chunk), ("F", 0))]
    ev = tg.make_events(ops)[None, :]
    cfg = gpu_util.make_cfg(1, ev.shape[1], 2 * n, policy_mask=2, variant=2, table_place=place, max_pblocks=8192, max_multi_pblocks=1100,
                            max_sblocks=2560, max_runs=160000, max_chunks=32000)
    st = check(ev, cfg, label="lists of a thousand words", in_lds=in_lds)
    assert st["n_code"][1, 0, 1] == 160 and st["max_runs"][1, 0] > 36000


@pytest.mark.parametrize("seed,trace", [(1, 300), (12345, 500)])
def test_zero3_preset_holds_its_traces_in_the_first_pass(seed, trace):
    # the traces with the most pBlocks of their seeds (534 and 527); without retry_traces an overflow stays flagged
    ev, ms = tg.generate(6, n_traces=1, n_events=20000, first_trace=trace, seed=seed)
    cfg = workloads.make_config(binding, 6, 1, 20000, ms, retry_traces=0, policy_mask=2)
    st = check(ev, cfg, label="seed %d trace %d" % (seed, trace))
    assert st["max_pblocks"][1, 0] > 512


# ... and traces of seeds that tables of 536 and 544 places sent through the second pass
@pytest.mark.parametrize("config,seed,trace,pblocks", [(6, 112, 500, 539), (6, 140, 930, 535), (2, 114, 463, 546)])
def test_presets_hold_traces_of_other_seeds_in_the_first_pass(config, seed, trace, pblocks):
    ev, ms = tg.generate(config, n_traces=1, n_events=20000, first_trace=trace, seed=seed)
    cfg = workloads.make_config(binding, config, 1, 20000, ms, retry_traces=0, policy_mask=2)
    st = check(ev, cfg, label="seed %d trace %d" % (seed, trace))
    assert st["max_pblocks"][1, 0] == pblocks


# Presets by the length of the traces: no pool of 320 traces outgrows its tables, and of the first 64 the trace with the
# most pBlocks is replayed on them without a second pass
@pytest.mark.parametrize("config,events,worst", [(6, 50000, 49), (2, 50000, 8), (6, 100000, None), (2, 100000, None), (2, 30000, None)])
def test_presets_hold_longer_traces_in_the_first_pass(config, events, worst):
    ev, ms = tg.generate(config, n_traces=320, n_events=events, seed=1)
    cfg = workloads.make_config(binding, config, 320, events, ms)
    _, st = oracle.replay(ev, gpu_util.oracle_params(cfg), oracle.VMS, want_decisions=False, threads=8)
    assert st["max_pblocks"].max() < cfg.max_pblocks and st["max_sblocks"].max() + 2 < cfg.max_sblocks
    assert st["peak_reserved"].max() <= cfg.max_chunks * cfg.chunk_bytes
    if worst is not None:
        assert st["max_pblocks"][:64].argmax() == worst
        cfg = workloads.make_config(binding, config, 1, events, ms, retry_traces=0, policy_mask=2)
        check(ev[worst : worst + 1], cfg, label="trace %d" % worst)


def test_table_overflow_is_flagged_not_fatal():
    ev, ms = tg.generate(3, n_traces=1, n_events=2500, seed=5)
    cfg = gpu_util.make_cfg(1, 2500, ms, policy_mask=2, variant=2, max_pblocks=64, max_sblocks=520, max_chunks=4096)
    _, _, st = emu.replay(ev, cfg, binding.STATS_DTYPE)
    assert st["status"][1, 0] & binding.VMS_ST_TABLE_OVERFLOW and st["overflow_event"][1, 0] < 2500


# pool[] of the fine-grained variant in global memory, all other tables in the workspace: one to several steps of its
# moves and scans (256 blocks each), cuts into pieces of one chunk and more, the fragmentation limit, an arena that is
# squeezed, a pool that is outgrown
@pytest.mark.parametrize("kind,events,kw", [
    (3, 2500, dict(max_runs=1 << 16, max_sblocks=2560, max_pblocks=8192, max_multi_pblocks=2848, max_chunks=10240)),
    (3, 1500, dict(max_runs=1 << 15, max_sblocks=1024, max_pblocks=8192, max_multi_pblocks=1030, max_chunks=10240, frag_limit_bytes=6 * MiB)),
    (1, 1500, dict(spool_threshold=8, max_sblocks=256, max_runs=700, max_chunks=8192)),
    (4, 3000, dict(max_pblocks=700, spool_threshold=16, max_sblocks=92, max_runs=700, max_chunks=20480)),
    (2, 2000, dict(max_pblocks=100, max_runs=4000, max_chunks=8192, retry_traces=1))])
def test_pool_in_global_memory(kind, events, kw):
    ev, ms = tg.generate(kind, n_traces=2, n_events=events, seed=11)
    cfg = gpu_util.make_cfg(2, events, ms, policy_mask=2, variant=2, table_place=binding.VMS_TABLES_WORKSPACE_ALL, **kw)
    check(ev, cfg, n_events=np.array([events, events - 37], dtype=np.uint32), label="generator %d" % kind, pool_in_mem=True)


# requests of more chunks than 16 bits count: no block of that size can exist, so they fail (a capacity) or outgrow the
# chunk table, and must not meet the blocks of the same size modulo 65,536
HUGE = [65534, 65535, 65536, 65537, 65541, 131077, (1 << 19) - 4096]


def assert_chunks_overflow(ev, cfg, chunks, n_events=None, **kw):
    """Up to the engine's own capacity of 512 GiB the first such request outgrows the chunk table: the replay ends before
    it, flagged."""
    at = 7
    if chunks * 2 * MiB > 512 << 30:
        check(ev, cfg, n_events=n_events, label="%d chunks" % chunks, **kw)
        return
    _, dv, st = emu.replay(ev, cfg, binding.STATS_DTYPE, n_events, **kw)
    P = gpu_util.oracle_params(cfg)
    odec, ost = oracle.replay(ev[-1:], P, 1, n_events=[at])
    g = st[1][-1]
    assert g["status"] == binding.VMS_ST_TABLE_OVERFLOW | binding.VMS_ST_OVF_CHUNKS and g["overflow_event"] == at
    assert np.array_equal(dv[-1, :at], odec[0, :at]) and (dv[-1, at:] == np.uint64(0xFFFFFFFFFFFFFFFF)).all()
    for f in ("peak_active", "peak_reserved", "final_active", "final_reserved", "n_code", "digest"):
        assert np.array_equal(g[f], ost[0][f]), f


@pytest.mark.parametrize("chunks", HUGE)
@pytest.mark.parametrize("place", [binding.VMS_TABLES_LDS, binding.VMS_TABLES_WORKSPACE, binding.VMS_TABLES_WORKSPACE_ALL, 4])
@pytest.mark.parametrize("frag", [0, 6 * MiB])
def test_request_of_more_chunks_than_16_bits_count(chunks, place, frag):
    ev = tg.make_events(gpu_util.huge_request_ops(chunks))[None, :]
    kw = dict(policy_mask=2, variant=binding.VMS_VARIANT_FINE, table_place=min(place, 3), frag_limit_bytes=frag)
    in_mem = dict(pool_in_mem=place == 4)
    st = check(ev, gpu_util.make_cfg(1, ev.shape[1], 16, capacity_bytes=4 << 30, **kw), label="%d chunks" % chunks, **in_mem)
    assert st["n_code"][1, 0, 5] == 3
    assert_chunks_overflow(ev, gpu_util.make_cfg(1, ev.shape[1], 16, **kw), chunks, **in_mem)


# the same where the library chooses the variant, in the flat variant, and in the second pass behind it
@pytest.mark.parametrize("chunks", [65536, 65541])
@pytest.mark.parametrize("traces,slots,kw", [(1, 16, {}), (800, 650, {}), (2, 16, dict(variant=1, retry_traces=1, max_chunks=9000)),
                                             (2, 16, dict(variant=2, retry_traces=1, max_chunks=9000))])
def test_request_of_more_chunks_than_16_bits_count_by_default(chunks, traces, slots, kw):
    one = tg.make_events(gpu_util.huge_request_ops(chunks))
    ev = np.repeat(one[None, :], traces, axis=0)
    n = np.full(traces, 0, dtype=np.uint32)
    n[-1] = ev.shape[1]
    check(ev, gpu_util.make_cfg(traces, ev.shape[1], slots, policy_mask=2, capacity_bytes=4 << 30, **kw), n_events=n, label="%d chunks" % chunks)
    assert_chunks_overflow(ev, gpu_util.make_cfg(traces, ev.shape[1], slots, policy_mask=2, **kw), chunks, n_events=n)


# limits of more chunks than 16 bits count, and of more than a trace has: no block is split or stitched
@pytest.mark.parametrize("chunks", [4096, 62999, 65535, 65536, 65537, 65541, 1 << 32])
@pytest.mark.parametrize("variant,place", [(1, 0), (2, 1), (2, 3), (2, 4)])
def test_fragmentation_limit_of_more_chunks_than_16_bits_count(chunks, variant, place):
    ev, ms = tg.generate(1, n_traces=1, n_events=300, seed=3)
    cfg = gpu_util.make_cfg(1, 300, ms, policy_mask=2, variant=variant, table_place=min(place, 3), max_chunks=4095,
                            frag_limit_bytes=chunks * 2 * MiB)
    st = check(ev, cfg, label="limit of %d chunks" % chunks, pool_in_mem=place == 4)
    assert st["max_members"][1, 0] <= 1


# The list places in the slot table of the flat variant are there for speed only: a slot table that leaves no room for
# them in LDS (up to about 12,500 slots of three words each beside the smallest other tables) is in global memory,
# whatever it takes there, and the tables are neither refused nor moved to the fine-grained variant.
@pytest.mark.parametrize("slots,traces,ok", [(9800, 1, True), (12400, 1, True), (12400, 1 << 16, True), (13700, 1, False)])
@pytest.mark.parametrize("variant", [binding.VMS_VARIANT_AUTO, binding.VMS_VARIANT_FLAT])
def test_plan_of_a_slot_table_as_large_as_the_lds(slots, traces, ok, variant):
    cfg = gpu_util.make_cfg(traces, 9, slots, variant=variant, max_free_blocks=8, max_small_blocks=8, max_pblocks=16, max_sblocks=520,
                            max_runs=64, max_chunks=640)
    rc, p = emu.plan(cfg)
    assert rc == (0 if ok else -6)
    if ok:
        assert p.slots == emu.SLOTS_IN_MEM and p.lds_bytes[1] < 20000
        assert not p.fine or variant == binding.VMS_VARIANT_AUTO


@pytest.mark.parametrize("small", [False, True])
def test_slot_table_as_large_as_the_lds(small):
    ev, n = gpu_util.slot_reuse_traces(11800, 64 * 9, seed=3)
    check(ev, gpu_util.make_cfg(4, ev.shape[1], 11800, variant=binding.VMS_VARIANT_FLAT, max_free_blocks=64, max_small_blocks=64,
                                max_pblocks=128, max_sblocks=520, max_runs=400, max_chunks=640, retry_traces=1),
          n_events=n, label="11,800 slots", small=small)


# The second pass shrinks its tables towards the first one's until they fit, the table of multi-chunk pBlocks among them
def test_second_pass_shrinks_the_table_of_multi_chunk_pblocks():
    cfg = gpu_util.make_cfg(1, 9, 10099, policy_mask=2, variant=binding.VMS_VARIANT_FINE, max_free_blocks=8, max_small_blocks=8,
                            max_pblocks=16, max_multi_pblocks=2855, max_sblocks=900, max_runs=64, max_chunks=64, retry_traces=1)
    rc, p = emu.plan(cfg)
    assert rc == 0 and p.fine and p.has_retry


# A batch whose tables are in global memory has a plan without them for a device that has no room left: in both passes,
# for each policy, whichever variant and place the handle names
@pytest.mark.parametrize("config,slots,traces", [(1, 120, 6000), (2, 64, 4096), (3, 64, 4096), (4, 650, 4096), (4, 650, 700), (6, 1163, 1280)])
@pytest.mark.parametrize("kw", [dict(), dict(variant=1), dict(variant=2), dict(table_place=3)])
def test_plan_without_tables_in_global_memory(config, slots, traces, kw):
    if config == 3 and kw.get("variant") == 1:
        return
    cfg = workloads.make_config(binding, config, traces, 20000, slots, **kw)
    rc, p = emu.plan(cfg, in_lds=True)
    assert rc == 0 and p.slots != emu.SLOTS_IN_MEM and list(p.mem_stride) == [0, 0] and max(p.lds_bytes) <= 160 * 1024
    again = emu.plan(workloads.make_config(binding, config, traces, 20000, slots, **kw))[1].has_retry
    assert p.has_retry == again


def test_replay_without_tables_in_global_memory():
    ev, ms = tg.generate(4, n_traces=3, n_events=1500, seed=9)
    cfg = workloads.make_config(binding, 4, 900, 1500, ms)
    ev = np.concatenate([ev, np.zeros((897, 1500), dtype=np.uint64)])
    assert emu.plan(cfg)[1].slots == emu.SLOTS_IN_MEM
    check(ev, cfg, n_events=np.array([1500, 1499, 1437] + [0] * 897, dtype=np.uint32), label="in LDS", in_lds=True)

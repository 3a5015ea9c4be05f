"""The synthetic workloads and the engine table sizes that fit them.

Table sizes (per trace) are capacity settings of the replay engine, not parameters of the
allocators: a trace that outgrows them is replayed a second time with doubled tables (up to
retry_traces traces per run), and flagged VMS_ST_TABLE_OVERFLOW, never replayed wrongly, if that
does not suffice.  The values below hold the high-water marks measured on the full workloads of the
default seed with headroom (what other seeds and longer traces need is said beside the tables where they were counted);
smaller tables mean less LDS per wavefront and therefore more resident wavefronts per compute unit.
"""
from . import tracegen

NAMES = {1: "config1-random", 2: "config2-recompute", 3: "config3-offload", 4: "config4-lora",
         5: "config5-mixture", 6: "config6-zero3-scaleout"}

TABLES = {
    # config: splitting free list (max_small_blocks: the stitching policy's own, smaller one), pBlocks, sBlocks,
    # chunk-run list entries, chunks (x 2 MiB)
    1: dict(max_free_blocks=512, max_pblocks=1024, max_sblocks=640, max_runs=4096, max_chunks=8192),
    # (40,208 B on the flat kernel: four wavefronts per compute unit have room for as much.  No trace of 120 seeds outgrows
    # these sizes at 20,000 events, nor of 13 at 50,000 (607 and 622 pBlocks); 544 pBlocks and 3,840 list entries were
    # too few in one seed of seven, whose batch of 1,024 traces then took 23 ms instead of 8)
    2: dict(max_free_blocks=192, max_pblocks=640, max_sblocks=576, max_runs=4992, max_chunks=4096),
    # offloading grinds pBlocks down to single chunks: thousands of pBlocks and sBlocks (the fine-grained kernel
    # variant: single chunks in bitmaps, a table for the pBlocks of two or more chunks, lists in the workspace)
    # (LDS is handed out in 1,280-byte granules, 128 per compute unit.  Multi-chunk pBlocks: 2,421 to 2,824 at most over
    # 13 seeds.  2,848 places are what five wavefronts per compute unit have room for with all tables in LDS, 31,984 B,
    # where the library puts them for up to 1,280 traces; up to 2,304 the tables of the sBlocks are in the workspace and
    # a wavefront takes 16,144 B; for more traces than that the table of the multi-chunk pBlocks is in global memory too,
    # 4,432 B, sixteen wavefronts.  2,592 places would hold 2,560 traces in one round without that, 2500x20000 in 81.8
    # instead of 88.2 ms, but at 50,000 events seven of the 13 seeds send one or two traces through the second pass)
    3: dict(max_free_blocks=64, max_pblocks=8192, max_multi_pblocks=2848, max_sblocks=2560, max_runs=1 << 18, max_chunks=10240),
    # (up to 512 traces on the flat kernel with the slot table in LDS, 49,616 B, up to 1,024 with it in global memory,
    # 39,184; the fine-grained one beyond that, 14,320 B, and with the tables of its sBlocks in the workspace 10,384,
    # beyond 2,560, where that saves a round; chunk tables for the 17,699 chunks the largest trace reserves)
    4: dict(max_free_blocks=320, max_small_blocks=192, max_pblocks=640, max_sblocks=576, max_runs=3840, max_chunks=18432),
    # (the same for the scale-out regime, 9,408 chunks at most; 50,608 / 31,984 / 10,464 B.  31,984 B are what five
    # wavefronts per compute unit have room for, so that the 1,280 traces of the workload are on the flat kernel at once:
    # 8.4 ms, 12.0 on the fine-grained one, which 3,072 list entries, 576 sBlocks, 9,728 chunks and 544 pBlocks made them
    # take.  Among what fits there these sizes were outgrown least: by one trace of 220 seeds, which puts the batch at
    # 21 ms; with 536 pBlocks, 544 sBlocks and 2,960 list entries by one in two seeds of 60)
    6: dict(max_free_blocks=192, max_pblocks=576, max_sblocks=540, max_runs=2912, max_chunks=9408),
}
# config 5 mixes the generators of configs 2, 3 and 4 (trace i uses kind 2 + i mod 3) with twice the
# events; replayed as three batches, one per kind, each with tables of its own
TABLES_5 = {
    2: dict(max_free_blocks=192, max_pblocks=640, max_sblocks=640, max_runs=5120, max_chunks=4096),
    # (the margins over the high-water marks are one to two per cent; a trace that outgrows a table is replayed
    # again by the second pass.  40,208 B of LDS per wavefront with every table in LDS, four wavefronts per compute
    # unit; for more traces than that the library moves the sBlock tables to the workspace, 14,960 B, ten, and beyond
    # 2,560 the table of the multi-chunk pBlocks too, 3,760 B, sixteen)
    3: dict(max_free_blocks=64, max_pblocks=8192, max_multi_pblocks=2720, max_sblocks=4128, max_runs=1 << 18, max_chunks=8480),
    # (18,055 chunks is the most a trace of this kind reserves; 10,768 B of LDS per wavefront for the 5,461 traces of the
    # workload)
    4: dict(max_free_blocks=320, max_small_blocks=192, max_pblocks=736, max_sblocks=576, max_runs=4224, max_chunks=18432),
}

# Tables of traces longer than the presets of workloads 2 and 6 are sized for: pBlocks are cut finer the longer a trace
# runs.  (events up to which the tables before hold its traces, the tables of longer ones.)  With tables for 20,000 events
# 202 of 1,280 ZeRO-3 traces x 50,000 were replayed again, in turns of retry_traces: 453 ms for the whole pass, 30.6 with
# these; at 100,000 events 2,475 and 55, recomputation 1,155 and 66.  No trace of 13 seeds outgrows them (ZeRO-3 721 pBlocks
# at most at 50,000 events, 867 at 100,000; recomputation 625).  Up to 23,000 events ZeRO-3 keeps the smaller ones, five
# traces per compute unit on the flat kernel: two of 40 seeds have a trace that is replayed again (22,000 events: 21.8
# against 13.3 ms), for the others the batch is that much faster (9.1 against 13.3).
LONGER = {
    2: [(50000, TABLES_5[2])],
    6: [(23000, dict(max_free_blocks=192, max_pblocks=768, max_sblocks=576, max_runs=4352, max_chunks=9408)),
        (50000, dict(max_free_blocks=192, max_pblocks=896, max_sblocks=688, max_runs=8448, max_chunks=9408))],
}


def shape(config):
    c = tracegen.CONFIGS[config]
    return c["n_traces"], c["n_events"]


def make_config(binding, config, n_traces, n_events, max_slots, kind=None, **overrides):
    """vms_config for a workload (kind: the generator of a config-5 batch)."""
    cfg = binding.vms_config_default(n_traces, n_events, max_slots)
    cfg.capacity_bytes = tracegen.CONFIGS[config]["capacity_bytes"]
    tables = TABLES_5[kind] if config == 5 else TABLES[config % 10]
    for events, longer in LONGER.get(config % 10, []):
        if n_events > events:
            tables = longer
    for k, v in tables.items():
        setattr(cfg, k, v)
    # the tables hold the high-water marks of the seeded workloads with little headroom; a trace of
    # another seed that outgrows one is replayed a second time with doubled tables
    cfg.retry_traces = min(32, n_traces)
    for k, v in overrides.items():
        assert hasattr(cfg, k), k
        setattr(cfg, k, v)
    return cfg

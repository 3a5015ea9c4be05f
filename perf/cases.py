"""The replay work that the measurements of this framework are taken on.

A case is a batch of allocation traces handed to one or more Replay handles: the workloads of
workloads.py at their own sizes (the mixture with shorter traces, so that its inputs are made in a
second), the two studies' batches, and small, odd and ragged batches with default tables.  One
pass replays the batch under the policies asked for and reads the per-trace statistics back, as
bench.py and the studies do; its outputs are every decision word and the statistics.

A case's values: `generator` (1 random, 2 recomputation, 3 offloading, 4 LoRA, 5 the mixture of
2 to 4 as three batches on three streams, 6 ZeRO-3 ranks), `traces`, `events` (per trace), `tables`
("preset": workloads.make_config, "roomy": the same with the studies' larger tables, "default":
vms_config_default), `policies` (VMS_POLICY_* mask), `decisions` (are decision words written),
`ragged` (trace lengths vary), `static` (vms_replay_run_static: the built-in workspace),
`threshold` / `frag_mib` (the allocator's knobs).
"""
import math

import numpy as np
import torch

from paper_2401_08156_amd import binding, workloads
from paper_2401_08156_amd import tracegen as tg

MiB = 1 << 20
# a statistics record as 32-bit words: everything up to max_members describes the allocators (the four
# words behind it are high-water marks of one kernel variant's own tables), the fragmentation comes last
RECORD_WORDS = binding.STATS_DTYPE.fields["max_runs"][1] // 4
SUMMARY_FIELDS = ("sum_peak_reserved", "sum_peak_active", "n_flagged", "max_fragmentation", "mean_fragmentation")
# the studies' table sizes (the knobs change how many blocks and chunks a trace needs)
ROOMY = dict(max_pblocks=2048, max_sblocks=1024, max_runs=16000, max_chunks=28672, max_free_blocks=1024)


def _case(generator, traces, events, tables="preset", policies=3, decisions=True, ragged=False, static=False,
          threshold=512, frag_mib=2, name=None):
    c = dict(generator=generator, traces=traces, events=events, tables=tables, policies=policies, decisions=decisions,
             ragged=ragged, static=static, threshold=threshold, frag_mib=frag_mib)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a handful of short streams, as in a serving loop that must not allocate: launches and waits
        _case(1, 3, 61, tables="default", static=True, name="static-3x61"),
        # workload 1: one trace, a latency figure (one wavefront per policy)
        _case(1, 1, 2000, name="random-1x2000"),
        # imported recordings: an odd batch of traces of different lengths, nothing known of them beforehand
        _case(1, 301, 1777, tables="default", ragged=True, name="ragged-301x1777"),
        # workload 2: as many traces as the device has SIMDs
        _case(2, 1024, 20000, name="recompute-1024x20000"),
        # the study of the StitchFree threshold: few traces, few cached blocks
        _case(2, 64, 20000, tables="roomy", threshold=64, name="threshold-64x20000"),
        # the study of the fragmentation limit on LoRA streams
        _case(4, 64, 20000, tables="roomy", frag_mib=8, name="fraglimit-64x20000"),
        # the scale-out study: statistics only, no decision words
        _case(6, 320, 20000, decisions=False, name="scaleout-320x20000"),
        # workload 6: ranks of a sharded job
        _case(6, 1280, 20000, name="zero3-1280x20000"),
        # the caching allocator alone, the baseline of every comparison
        _case(4, 2048, 20000, policies=1, name="splitting-2048x20000"),
        # workload 4: LoRA streams
        _case(4, 4096, 50000, name="lora-4096x50000"),
        # workload 3: offloading streams, thousands of blocks per trace
        _case(3, 4096, 50000, name="offload-4096x50000"),
        # workload 5: the mixture, three batches side by side
        _case(5, 16384, 20000, name="mixture-16384x20000"),
    ]


# what a pass costs at most, in seconds: per event of the whole batch, and per event of one trace
COST = {1: (1e-9, 2e-6), 2: (0.6e-9, 1e-6), 3: (2.2e-9, 6e-6), 4: (0.8e-9, 1.5e-6), 5: (1e-9, 6e-6), 6: (1e-9, 1.5e-6)}


def draw(rng):
    while True:
        g = rng.choice((1, 1, 2, 2, 3, 4, 4, 5, 6))
        lo, hi = (1, 16384) if g == 5 else (1, 4096)
        traces = max(3 if g == 5 else 1, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))
        events = round(math.exp(rng.uniform(math.log(48 if g == 1 else 700), math.log(2000 if g == 1 else 50000))))
        whole, single = COST[g]
        if max(traces * events * whole, events * single) > 0.4:
            continue
        c = _case(g, traces, events, ragged=rng.random() < 0.25)
        if g == 5:
            return c
        c["policies"] = rng.choice((3, 3, 3, 3, 1, 2))
        c["decisions"] = rng.random() < 0.8
        if g == 1:
            c["tables"] = "default" if rng.random() < 0.6 else "preset"
        elif g != 3 and traces <= 256 and rng.random() < 0.4:
            c["tables"] = "roomy"
            c["threshold"] = rng.choice((64, 128, 256, 512))
            c["frag_mib"] = rng.choice((2, 2, 8, 32))
        return c


def _lengths(case, traces, rng):
    if not case["ragged"]:
        return None
    n = rng.integers(0, case["events"] + 1, size=traces, dtype=np.int64)
    n[rng.integers(0, traces)] = case["events"]
    return n.astype(np.int32)


def _batch(case, seed, first, stride, kind, rng):
    g, n_events = case["generator"], case["events"]
    traces = len(range(first, case["traces"], stride))
    ev, max_slots = tg.generate(g, n_traces=traces, n_events=n_events, seed=seed & 0x7FFFFFFF, first_trace=first,
                                trace_stride=stride, threads=16)
    if case["tables"] == "default":
        cfg = binding.vms_config_default(traces, n_events, max_slots)
    else:
        over = dict(ROOMY) if case["tables"] == "roomy" else {}
        cfg = workloads.make_config(binding, g, traces, n_events, max_slots, kind=kind, **over)
    cfg.policy_mask = case["policies"]
    cfg.spool_threshold = case["threshold"]
    cfg.frag_limit_bytes = case["frag_mib"] * MiB
    d_ev = torch.from_numpy(ev.view(np.int64)).cuda()
    n = _lengths(case, traces, rng)
    b = dict(events=d_ev, lengths=None if n is None else torch.from_numpy(n).cuda(), split=None, vms=None, rep=binding.Replay(cfg))
    # (zeros: words past a trace's length are not written)
    if case["decisions"] and case["policies"] & 1:
        b["split"] = torch.zeros_like(d_ev)
    if case["decisions"] and case["policies"] & 2:
        b["vms"] = torch.zeros_like(d_ev)
    return b


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kinds = (2, 3, 4) if case["generator"] == 5 else (None,)
    batches = [_batch(case, seed, i, len(kinds), kind, rng) for i, kind in enumerate(kinds)]
    state = dict(batches=batches, static=case["static"], summary=case["generator"] == 5)
    if len(batches) > 1:
        state["streams"] = [torch.cuda.Stream() for _ in batches]
        state["order"] = (1, 0, 2)          # the long-running offloading batch first
    return state


def run(state):
    batches = state["batches"]
    if len(batches) > 1:
        main = torch.cuda.current_stream()
        for i in state["order"]:
            b, s = batches[i], state["streams"][i]
            s.wait_stream(main)
            b["rep"].run(b["events"], b["lengths"], b["split"], b["vms"], s)
        for s in state["streams"]:
            main.wait_stream(s)
    else:
        b = batches[0]
        go = b["rep"].run_static if state["static"] else b["rep"].run
        go(b["events"], b["lengths"], b["split"], b["vms"])
    out = []
    for b in batches:
        st = b["rep"].stats()
        o = dict(statistics=st.view("<i4").reshape(2, -1, st.itemsize // 4)[:, :, :RECORD_WORDS], fragmentation=st["fragmentation"])
        if b["split"] is not None:
            o["decisions_split"] = b["split"]
        if b["vms"] is not None:
            o["decisions_vms"] = b["vms"]
        if state["summary"]:
            s = b["rep"].summary()
            o["summary"] = [np.array([getattr(s, f)[p] for p in (0, 1)]) for f in SUMMARY_FIELDS] + [float(s.mem_reduction_ratio)]
        out.append(o)
    return out


def work(case):
    """Each event word read once, each decision word and statistics record written once (ragged traces are half as
    long on average); the path computes no floating-point results to speak of: integer compares, about thirty per event and policy."""
    pols = bin(case["policies"]).count("1")
    events = case["traces"] * case["events"] * (0.5 if case["ragged"] else 1.0)
    return {"bytes": events * 8 * (1 + (pols if case["decisions"] else 0)) + case["traces"] * 152 * pols, "flops": 0}


def tolerance(case):
    # decisions, byte counts and counters are whole numbers; the fragmentation is one division of two
    # of them and its mean is summed in trace order: every correct implementation gives the same bits
    return "exact"

"""Shared helpers of the GPU parity tests: run the HIP path through the C ABI and the
oracle on the same events, compare bit for bit."""
import numpy as np

import oracle
from paper_2401_08156_amd import binding

COMPARED_FIELDS = ["peak_requested", "peak_active", "peak_reserved", "final_requested", "final_active",
                   "final_reserved", "digest", "n_code", "n_split", "n_merge", "n_sblock_created",
                   "n_sblock_evicted", "first_oom_event", "status", "max_pblocks", "max_sblocks",
                   "max_free_blocks", "max_members", "fragmentation"]


def make_cfg(n_traces, max_events, max_slots, **kw):
    cfg = binding.vms_config_default(n_traces, max_events, max_slots)
    for k, v in kw.items():
        assert hasattr(cfg, k), k
        setattr(cfg, k, v)
    return cfg


def oracle_params(cfg):
    return oracle.Params(cfg.chunk_bytes, cfg.small_limit_bytes, cfg.frag_limit_bytes, cfg.capacity_bytes,
                         cfg.spool_threshold, cfg.max_slots)


def gpu_replay(events, cfg, n_events=None, want_decisions=True):
    """Returns (dec_split, dec_vms, stats[2, n_traces]) as numpy arrays."""
    import torch
    dev = torch.device("cuda:0")
    ev = torch.from_numpy(np.ascontiguousarray(events).view(np.int64)).to(dev)
    ne = None if n_events is None else torch.from_numpy(np.ascontiguousarray(n_events, dtype=np.uint32).view(np.int32)).to(dev)
    r = binding.Replay(cfg)
    ds = dv = None
    if want_decisions:
        # poison so that entries the kernel must write are distinguishable from untouched ones
        if cfg.policy_mask & 1:
            ds = torch.full_like(ev, -1)
        if cfg.policy_mask & 2:
            dv = torch.full_like(ev, -1)
    r.run(ev, ne, ds, dv)
    st = r.stats()
    out = [None if d is None else d.cpu().numpy().view(np.uint64) for d in (ds, dv)]
    r.close()
    return out[0], out[1], st


def assert_parity(events, cfg, n_events=None, threads=8, label=""):
    """Bit-exact comparison of decisions and statistics of both policies with the oracle."""
    ds, dv, st = gpu_replay(events, cfg, n_events)
    P = oracle_params(cfg)
    for pol, gdec in ((0, ds), (1, dv)):
        if not (cfg.policy_mask & (1 << pol)):
            continue
        odec, ost = oracle.replay(events, P, pol, n_events=n_events, threads=threads)
        gst = st[pol]
        bad = np.flatnonzero(gst["status"] & binding.VMS_ST_TABLE_OVERFLOW)
        assert bad.size == 0, "%s policy %d: table overflow in traces %s at events %s, status %s" % (
            label, pol, bad[:8].tolist(), gst["overflow_event"][bad[:8]].tolist(), gst["status"][bad[:8]].tolist())
        if n_events is None:
            same = gdec == odec
        else:
            valid = np.arange(events.shape[1])[None, :] < np.asarray(n_events)[:, None]
            same = (gdec == odec) | ~valid
            assert np.all(gdec[~valid] == np.uint64(0xFFFFFFFFFFFFFFFF)), "wrote past the end of a trace"
        if not same.all():
            t, i = np.argwhere(~same)[0]
            raise AssertionError("%s policy %d trace %d event %d: gpu %#x oracle %#x (event word %#x)" % (
                label, pol, t, i, int(gdec[t, i]), int(odec[t, i]), int(events[t, i])))
        for f in COMPARED_FIELDS:
            if not np.array_equal(gst[f], ost[f]):
                t = np.flatnonzero((gst[f] != ost[f]).reshape(len(gst), -1).any(axis=1))[0]
                raise AssertionError("%s policy %d trace %d field %s: gpu %s oracle %s" % (
                    label, pol, t, f, gst[f][t], ost[f][t]))
    return st


def equal_blocks_trace(blocks, small, seed):
    """Fills a splitting pool to `blocks` inactive blocks of three sizes (ties inside a lane and across lanes,
    every place taken), then allocates and frees at random: cuts, exact fits, merges to the left, to the right
    and on both sides.  small: sizes below one chunk (the stitching policy's own pool).  Returns (events, slots)."""
    from paper_2401_08156_amd import tracegen as tg
    rng = np.random.default_rng(seed)
    chunk = 2 << 20
    # a block of its own segment each; small ones: the request and the rest of the chunk are two blocks
    first = [("A", s, chunk - 512 * int(rng.integers(1, 4)) if small else chunk * int(rng.integers(1, 4))) for s in range(blocks)]
    ops, live = first + [("F", s) for s in rng.permutation(blocks)], set()
    for _ in range(1500):
        s = int(rng.integers(0, blocks))
        if s in live:
            ops.append(("F", s))
            live.discard(s)
        elif len(live) < blocks // 2:
            size = 512 * int(rng.choice((1, 2, 1024, 2047, 2048, 4095) if small else (1, 4096, 8192, 8191, 12288)))
            ops.append(("A", s, min(size, chunk - 512) if small else size))
            live.add(s)
    return tg.make_events(ops)[None, :], blocks


def slot_reuse_traces(slots, events, seed, traces=4):
    """Traces that keep coming back to a few slots, so that most events of 64 in a row follow another one on the same
    slot, with every kind of invalid event among them: slots that do not exist, an ALLOC of a held slot or of
    nothing, a FREE of an unbound slot.  Lengths end just before, at and after a tile of 64 events."""
    from paper_2401_08156_amd import tracegen as tg
    rng = np.random.default_rng(seed)
    out = np.zeros((traces, events), dtype=np.uint64)
    for t in range(traces):
        few = rng.choice(slots, size=min(slots, 3 + 12 * t), replace=False)
        held = set()
        ops = []
        while len(ops) < events:
            s = int(rng.choice(few)) if rng.random() < 0.8 else int(rng.integers(slots))
            x = rng.random()
            if x < 0.03:
                ops.append(("A", int(rng.choice((slots, slots + 1, 0x7FFFFFFF, 0xFFFFFFFF))), 4096))
            elif x < 0.05:
                ops.append(("F", int(rng.choice((slots, 0xFFFFFFFF)))))
            elif x < 0.07:
                ops.append(("A", s, 0))
            elif x < 0.10:
                ops.append((("A", s, 512) if s in held else ("F", s)))
            elif s in held:
                ops.append(("F", s))
                held.discard(s)
            else:
                big = int(rng.integers(1, 40)) << 20
                ops.append(("A", s, int(rng.integers(1, 3000)) * 512 if rng.random() < 0.5 else big))
                held.add(s)
        out[t] = tg.make_events(ops)
    return out, np.array([events, events - 1, events - 63, events - 64][:traces], dtype=np.uint32)


def huge_request_ops(chunks):
    """Cached blocks of as many chunks as the low 16 bits of `chunks` say (at least two), then three requests for about
    `chunks` chunks beside ordinary ones."""
    mib = 1 << 20
    low = max(chunks & 0xFFFF, 2) if chunks & 0xFFFF < 64 else 5
    return [("A", 0, low * 2 * mib), ("A", 1, 2 * mib), ("A", 2, 3 * 2 * mib), ("F", 0), ("F", 2),
            ("A", 3, (low + 2) * 2 * mib), ("F", 3), ("A", 4, chunks * 2 * mib), ("A", 0, low * 2 * mib), ("F", 0),
            ("A", 5, (chunks - 1) * 2 * mib + 512), ("F", 5), ("A", 2, 2 * mib), ("A", 6, chunks * 2 * mib), ("F", 1), ("F", 4)]


def alternate_frees_trace(n):
    """2 n requests of 1 KiB out of one chunk, then every second one back: each FREE adds a block to the splitting
    pool that merges with nothing, beside the rest of the chunk.  Returns (events, slots)."""
    from paper_2401_08156_amd import tracegen as tg
    ops = [("A", s, 1024) for s in range(2 * n)] + [("F", s) for s in range(0, 2 * n, 2)]
    return tg.make_events(ops + [("A", 0, 512)])[None, :], 2 * n


def assert_free_outgrows_pool(replay, cfg, ev, pol, flag):
    """The last FREE of alternate_frees_trace(n) needs a place more than the pool has: the replay ends before it,
    flagged, with the statistics of the events before it.  Under the stitching policy the request of that FREE is
    gone (its slot is unbound before the pool is asked), its memory is still held."""
    at = ev.shape[1] - 2
    ds, dv, st = replay(ev, cfg)
    dec, g = (ds, dv)[pol][0], st[pol][0]
    P = oracle_params(cfg)
    odec, ost = oracle.replay(ev, P, pol, n_events=[at])
    assert g["status"] == binding.VMS_ST_TABLE_OVERFLOW | flag and g["overflow_event"] == at
    assert np.array_equal(dec[:at], odec[0, :at]) and (dec[at:] == np.uint64(0xFFFFFFFFFFFFFFFF)).all()
    for f in COMPARED_FIELDS:
        if f not in ("status", "final_requested"):
            assert np.array_equal(g[f], ost[0][f]), (f, g[f], ost[0][f])
    assert g["final_requested"] == ost[0]["final_requested"] - (1024 if pol else 0)
    # with one place more the whole trace fits
    cfg.max_free_blocks += 1
    cfg.max_small_blocks += 1 if cfg.max_small_blocks else 0
    ds, dv, st = replay(ev, cfg)
    odec, ost = oracle.replay(ev, P, pol)
    assert np.array_equal((ds, dv)[pol], odec) and st[pol][0]["status"] == 0
    for f in COMPARED_FIELDS:
        assert np.array_equal(st[pol][0][f], ost[0][f]), f

"""The work whose speed counts: what a program that checks its transfers has this library do.

Every case goes through the C ABI's Python binding (paper_1310_0901_amd.xfercheck) the way a program calls it: the
context, the shadow and the records are in device memory before the call, one call checks the batch on the current
stream, and the verdicts (and, with propagation, the destination shadows) are what comes back.

Paths:
  staging    check_transfers, 1 to 256 uploads from a staging buffer (the plain, tiny configuration's sizes)
  requests   check_transfers, a few hundred to 16,000 requests of the serving mixture (90/9/1 of 64 B - 4 KiB,
             4 KiB - 1 MiB, 1 - 64 MiB) against a large allocation table
  full       check_transfers, one full-size upload per allocation (the plain-at-scale configuration)
  mixed      check_transfers, 16,384 records and more of all three kinds (the batched configuration)
  propagate  check_transfers with CG_PROPAGATE: verdicts and destination shadows, from one copy to many pieces
  rows       check_transfers_2d, pitched copies: tight rows on the host, pitched rows on the device
  join       check_concurrent over a program's copies on several streams
  pointers   check_pointers: kernel arguments against the live allocations
  serve      cg_serve_run: a log of requests with allocations and frees between them
"""
import math

import numpy as np
import torch

from paper_1310_0901_amd import workloads as W
from paper_1310_0901_amd import xfercheck as X

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30


def listed():
    return [
        # one hipMemcpy as the interposer checks it: verdict and shadow of a single small copy
        dict(name="one_copy", path="propagate", count=1, lo=12345, hi=12346, allocs=64, dense=True, only="h2d"),
        # a handful of uploads per step: the plain, tiny configuration
        dict(name="staging_64", path="staging", count=64, host=1 * MiB),
        # a serving tick's requests as one batch
        dict(name="requests_2000", path="requests", count=2000, allocs=100_000, host=1 * GiB),
        # a model's parameters uploaded: one full-size copy per allocation (plain at scale)
        dict(name="full_4096", path="full", count=4096, host=4 * GiB, hi=64 * MiB),
        # a whole trace checked at once: the batched configuration
        dict(name="mixed_1M", path="mixed", count=1_000_000, allocs=65536, host=4 * GiB, hi=16 * MiB),
        # partly defined structs carried to the device in one copy
        dict(name="hop_2GiB", path="propagate", count=1, lo=2 * GiB, hi=2 * GiB + 1, allocs=16, dense=True, only="h2d"),
        # many small unaligned copies of all kinds whose definedness is tracked
        dict(name="pieces_65k", path="propagate", count=65_536, lo=16, hi=64 * KiB, allocs=4096, dense=False, only=""),
        # images and matrices moved by hipMemcpy2D: check only, and with the shadow carried along
        dict(name="rows_check", path="rows", count=1500, width=4030, pitch=4096, rows=1200, host=1 * GiB, prop=False),
        dict(name="rows_track", path="rows", count=800, width=333, pitch=512, rows=2000, host=256 * MiB, prop=True),
        # a trace's copies on 8 streams joined for concurrent accesses, a synchronisation every 4,096 copies
        dict(name="join_1M", path="join", count=1_000_000, epoch=4096, streams=8),
        # a launch trace's pointer arguments against a table of a long-running server
        dict(name="pointers_1M", path="pointers", count=1_000_000, allocs=975_000),
        # a burst of requests with allocation churn, served to the end
        dict(name="serve_20k", path="serve", count=20_000, allocs=100_000, host=1 * GiB),
    ]


def draw(rng):
    def log(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    path = rng.choice(["staging", "requests", "full", "mixed", "propagate", "propagate", "rows", "rows", "join",
                       "pointers", "serve"])
    if path == "staging":
        return dict(path=path, count=log(1, 257), host=log(256 * KiB, 16 * MiB))
    if path == "requests":
        return dict(path=path, count=log(257, 16_000), allocs=log(2000, 200_000), host=log(256 * MiB, 2 * GiB))
    if path == "full":
        return dict(path=path, count=log(257, 4096), host=log(256 * MiB, 4 * GiB), hi=log(64 * KiB, 64 * MiB))
    if path == "mixed":
        return dict(path=path, count=log(16_384, 1_000_000), allocs=log(1024, 32_768), host=log(64 * MiB, 2 * GiB),
                    hi=log(1 * KiB, 4 * MiB))
    if path == "propagate":
        count = log(1, 200_000)
        hi = log(64, min(1 * GiB, 4 * GiB // count))
        return dict(path=path, count=count, lo=max(1, hi // log(2, 4096)), hi=hi, allocs=log(16, 8192),
                    dense=count < 16 or rng.random() < 0.3, only=rng.choice(["", "", "h2d", "d2d"]))
    if path == "rows":
        width = log(16, 16 * KiB)
        pitch = (width + 255) // 256 * 256
        rows = log(16, 4096)
        count = log(1, max(2, min(4096, 4 * GiB // (pitch * rows))))
        return dict(path=path, count=count, width=width, pitch=pitch, rows=rows, host=log(256 * MiB, 1 * GiB),
                    prop=rng.random() < 0.5)
    if path == "join":
        return dict(path=path, count=log(64, 1_000_000), epoch=log(128, 65_536), streams=log(2, 32))
    if path == "pointers":
        return dict(path=path, count=log(256, 2_000_000), allocs=log(256, 975_000))
    return dict(path=path, count=log(1000, 20_000), allocs=log(2000, 100_000), host=log(256 * MiB, 1 * GiB))


# ---- inputs ----------------------------------------------------------------------------------------------------
def _spread(start, length):
    """Every index of the ranges [start, start + length)."""
    start, length = np.asarray(start, np.int64), np.asarray(length, np.int64)
    ends = np.cumsum(length)
    return np.repeat(start - (ends - length), length) + np.arange(int(length.sum()), dtype=np.int64)


class World:
    """A host region, live device allocations and a batch of records.

    Undefined bytes are runs (start, length) of the host region and of device addresses; unaddressable host bytes are
    whole pages.  `dense` puts undefined padding at bytes 13-15 of every 16 of the host region and one undefined bit
    in 1 % of its 16-byte structs.  Allocations in `fresh` keep the shadow of a new allocation."""

    def __init__(self, seed, host, base, size, records, host_runs=(), holes=(), dev_runs=(), dense=False, fresh=None,
                 host_base=W.HOST_BASE):
        self.seed, self.host, self.hb, self.dense = seed, int(host), host_base, dense
        self.base, self.size = np.asarray(base, np.int64), np.asarray(size, np.int64)
        self.fresh = np.zeros(self.base.size, bool) if fresh is None else np.asarray(fresh, bool)
        self.records = records
        self.host_runs = np.asarray(host_runs, np.int64).reshape(-1, 2)
        self.dev_runs = np.asarray(dev_runs, np.int64).reshape(-1, 2)
        pages = np.unique(np.asarray(holes, np.int64) >> 12)
        self.pages = pages[(pages + 1) * 4096 <= self.host]

    def host_v(self):
        v = torch.zeros((self.host + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
        if self.dense:
            g = torch.Generator("cuda").manual_seed(self.seed)
            rows = v.view(-1, 16)
            hit = torch.randint(rows.shape[0], (rows.shape[0] // 100 + 1,), device="cuda", generator=g)
            byte = torch.randint(13, hit.shape, device="cuda", generator=g)
            bit = torch.randint(8, hit.shape, device="cuda", generator=g)
            # a struct hit twice has both bits: bits of one byte are summed apart, so that order does not matter
            for k in range(8):
                m = bit == k
                flat = torch.unique(16 * hit[m] + byte[m])
                v[flat] += 1 << k
            rows[:, 13:] = 0xFF
        if self.host_runs.size:
            v[torch.from_numpy(_spread(*self.host_runs.T)).cuda()] = 0xFF
        return v

    def host_a(self):
        a = torch.full(((self.host + 63) // 64,), -1, dtype=torch.int64, device="cuda")
        if self.pages.size:
            a[torch.from_numpy(_spread(self.pages * 64, np.full(self.pages.size, 64))).cuda()] = 0
        return a


def _from_workload(w, records, seed):
    live = w.dev.live_idx
    runs = np.asarray(w.dev.runs, np.int64).reshape(-1, 4)
    runs = runs[w.dev.live[runs[:, 0]]] if runs.size else runs
    dev_runs = np.stack([w.dev.base[runs[:, 0]].astype(np.int64) + runs[:, 1], runs[:, 2]], 1) if runs.size else ()
    host_runs = w.host.runs[:, :2] if len(w.host.runs) else [(p, 1) for p, _ in np.asarray(w.host.points).reshape(-1, 2)]
    return World(seed, w.host.length, w.dev.base[live], w.dev.size[live], records, host_runs,
                 np.asarray(w.host.holes, np.int64).reshape(-1, 2)[:, 0], dev_runs,
                 fresh=w.dev.init[live] == 0xFF, host_base=w.host.base)


def _requests(case, seed):
    w = W.config5(seed=seed, duration=1.1 * case["count"] / 50_000.0 + 0.002, n_alloc=case["allocs"],
                  host_len=case["host"], p_new=0.0)
    rq = w.requests[:case["count"]]
    return w, W.make_records(rq["kind"], rq["src"], rq["dst"], rq["n"])


def _check_world(case, seed):
    if case["path"] == "staging":
        w = W.config1(seed=seed, n_transfers=case["count"], host_len=case["host"])
        return _from_workload(w, w.records, seed)
    if case["path"] == "full":
        w = W.config2(seed=seed, host_len=case["host"], n_alloc=case["count"], max_size=case["hi"])
        return _from_workload(w, w.records, seed)
    if case["path"] == "mixed":
        w = W.config3(seed=seed, n_transfers=case["count"], n_alloc=case["allocs"], host_len=case["host"],
                      max_size=case["hi"])
        return _from_workload(w, w.records, seed)
    w, records = _requests(case, seed)
    return _from_workload(w, records, seed)


def _sparse(rng, total, density):
    count = max(1, int(density * total / 32))
    length = rng.integers(1, 65, size=count)
    return np.stack([rng.integers(0, max(1, total - 64), size=count), np.minimum(length, total)], 1)


def _packed(rng, length, gap=32):
    """Ascending starts of pieces that do not touch, up to gap - 1 bytes apart, and the end of the last."""
    skip = rng.integers(0, gap, size=length.size) if length.size > 1 else np.zeros(length.size, np.int64)
    ends = np.cumsum(length + skip)
    return ends - length, int(ends[-1]) if length.size else 0


def _tracked_world(case, seed):
    """Copies whose destinations do not meet any other copy's bytes: device destinations packed into one allocation
    (the last), host destinations into the end of the host region.  Sources are anywhere in the rest, 2 % of the
    device sources running past their allocation's end.  Lengths, kinds and packing are the case's own (so every
    seed fills as much shadow); order, sources and contents are the seed's."""
    rng, fixed = np.random.default_rng(seed), np.random.default_rng(W.SEED0)
    T, hi = case["count"], case["hi"]
    n = W.log_uniform_int(fixed, case["lo"], hi, T)
    kind = {"h2d": np.zeros(T, np.int64), "d2d": np.full(T, 2)}.get(case["only"])
    if kind is None:
        kind = fixed.choice(3, size=T, p=[0.6, 0.1, 0.3]).astype(np.int64)
    read = max(2 * hi, 16 * MiB) if T > 1 else max(hi, 1 * MiB)
    # several allocations to read from, at most 1 GiB of them
    many = max(2, min(case["allocs"], GiB // hi)) if (kind != 0).any() else case["allocs"]
    size = np.full(many, hi if (kind != 0).any() else 4 * KiB, np.int64)
    d, h = kind != 1, kind == 1
    dpos, dlen = _packed(fixed, n[d])
    hpos, hlen = _packed(fixed, n[h])
    base = W.place_allocations(rng, np.append(size, max(dlen, 1))).astype(np.int64)
    j = rng.integers(0, many, size=T)
    off = (rng.random(T) * (size[j] - np.minimum(n, size[j]) + 1)).astype(np.int64)
    over = (rng.random(T) < 0.02) & (n > 64) & (T > 1)
    off = np.where(over, size[j] - n + rng.integers(1, 64, size=T), off)
    src = np.where(kind == 0, W.HOST_BASE + (rng.random(T) * (read - n + 1)).astype(np.int64), base[j] + off)
    dst = np.empty(T, np.int64)
    dst[d] = base[-1] + dpos
    dst[h] = W.HOST_BASE + read + hpos
    order = rng.permutation(T)
    rec = W.make_records(kind[order], src[order].astype(np.uint64), dst[order].astype(np.uint64),
                         n[order].astype(np.uint64))
    a = rng.integers(0, many, size=max(1, many // 4))
    dev_runs = np.stack([base[a] + size[a] // 3, np.minimum(rng.integers(1, 65, size=a.size), size[a] // 3 + 1)], 1)
    w = World(seed, read + hlen + 64, np.append(base[:-1], base[-1]), np.append(size, max(dlen, 1)), rec,
              _sparse(rng, read, 1e-6 if read > 64 * MiB else 1e-4),
              () if case["dense"] else rng.integers(0, read - 8192, 2), dev_runs, case["dense"],
              np.append(np.zeros(many, bool), True))
    w.read, w.written_host = read, hlen
    return w


def _rows_world(case, seed):
    """Pitched copies: tight rows on the host, rows at `pitch` on the device, an allocation per device side."""
    rng, fixed = np.random.default_rng(seed), np.random.default_rng(W.SEED0)
    T, width, pitch = case["count"], case["width"], case["pitch"]
    rows = W.log_uniform_int(fixed, max(1, case["rows"] // 8), case["rows"] + 1, T)
    kind = fixed.choice(3, size=T, p=[0.6, 0.1, 0.3]).astype(np.int64)
    tight, span = rows * width, (rows - 1) * pitch + width
    read = case["host"]
    h, d = kind == 1, kind != 1
    hpos, hlen = _packed(fixed, tight[h])
    # device sources, then device destinations packed into one allocation
    ns = int((kind != 0).sum())
    size = np.append(np.repeat(rows[kind != 0] * pitch, 1), max(int((rows[d] * pitch).sum()), 1)).astype(np.int64)
    base = W.place_allocations(rng, size).astype(np.int64)
    src = np.empty(T, np.int64)
    src[kind != 0] = base[:ns]
    src[kind == 0] = W.HOST_BASE + (rng.random(T - ns) * (read - tight[kind == 0] + 1)).astype(np.int64)
    dst = np.empty(T, np.int64)
    dst[d] = base[-1] + np.cumsum(rows[d] * pitch) - rows[d] * pitch
    dst[h] = W.HOST_BASE + read + hpos
    rec = np.zeros(T, W.RECORD2D_DTYPE)
    rec["src"], rec["dst"], rec["width"], rec["rows"], rec["kind"] = src, dst, width, rows, kind
    rec["spitch"] = np.where(kind == 0, width, pitch)
    rec["dpitch"] = np.where(kind == 1, width, pitch)
    rec = rec[rng.permutation(T)]
    a = rng.integers(0, max(ns, 1), size=max(1, ns // 8))
    dev_runs = np.stack([base[a] + size[a] // 2, np.minimum(8, size[a] // 2 + 1)], 1) if ns else ()
    w = World(seed, read + hlen + 64, base, size, rec, _sparse(rng, read, 1e-6), rng.integers(0, read - 8192, 2), dev_runs,
              False, np.append(np.zeros(ns, bool), True))
    w.read, w.written_host = read, hlen
    return w


def _serve_log(case, seed):
    """The requests of the serving configuration with temporary allocations made and freed between them, one event
    per 10 requests; all are freed by the end, so that the log can be served again.  A tenth of the uploads go to a
    temporary allocation, some of them after it was freed."""
    w, records = _requests(case, seed)
    rng = np.random.default_rng(seed + 1)
    world = _from_workload(w, records, seed)
    T = records.size
    events, live, dead = [], [], []
    at = int(world.base[-1] + world.size[-1]) + MiB
    comps = W.REQ_COMPONENTS
    target = rng.random(T)
    for t in range(T):
        if t % 10 == 9:
            if live and rng.random() < 0.5:
                b, n = live.pop(int(rng.integers(len(live))))
                dead.append((b, n))
                events.append((X.CG_EV_FREE, 0, b, 0, 0))
            else:
                lo, hi = comps[int(rng.choice(3, p=[0.99, 0.009, 0.001]))]
                n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
                live.append((at, n))
                events.append((X.CG_EV_ALLOC, 0, at, n, 0))
                at += (n + 255) // 256 * 256 + 256
        r = records[t]
        dst, n = int(r["dst"]), int(r["n"])
        pool = live if target[t] < 0.09 else dead if target[t] < 0.1 else None
        if pool and r["kind"] == 0:
            dst, size = pool[int(rng.integers(len(pool)))]
            n = min(n, size)
        events.append((X.CG_EV_CHECK, int(r["src"]), dst, n, int(r["kind"])))
    events += [(X.CG_EV_FREE, 0, b, 0, 0) for b, _ in live]
    e = np.array(events, np.uint64)
    log = np.zeros(e.shape[0], W.SERVE_EVENT_DTYPE)
    log["type"], log["src"], log["dst"], log["n"], log["kind"] = e.T
    world.room = 256 * MiB
    world.slots = T // 10 + 16
    return world, log


def _join_batch(case, seed):
    w = W.config3(seed=seed, n_transfers=case["count"], n_alloc=16_384, host_len=1 * GiB, max_size=1 * MiB)
    return W.race_from_records(w.records, seed, case["streams"], case["epoch"])


# ---- state -----------------------------------------------------------------------------------------------------
class Context:
    """A checker context and the host region's shadow that it reads.  It lives as long as anything that views its
    memory: a state, or an output of a pass on it."""

    def __init__(self, pool, allocs):
        self.handle = X.cg_create(0, pool, allocs)

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            X.cg_destroy(self.handle)
            self.handle = None

    def shadow(self, addr, n):
        """The V bytes of [addr, addr + n), in the library's own memory."""
        t = torch.as_tensor(_Bytes(self, X.shadow_ptr(self.handle, addr), n), device="cuda")
        t.owner = self
        return t


class _Bytes:
    """Device bytes of a context, for torch.as_tensor."""

    def __init__(self, owner, ptr, n):
        self.owner = owner   # the memory is the context's
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "|u1", "data": (ptr, False), "version": 2}


class State:
    """A context and the device buffers of one call."""

    def __init__(self, context):
        self.context, self.ctx = context, context.handle


def _upload(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).cuda()


def _open(w):
    room = getattr(w, "room", 0) + 16 * MiB
    c = Context(int(((w.size + 255) // 256 * 256).sum()) + room, w.base.size + getattr(w, "slots", 16))
    c.hv, c.ha = w.host_v(), w.host_a()
    torch.cuda.synchronize()
    X.cg_host_register(c.handle, w.hb, w.host, c.hv.data_ptr(), c.ha.data_ptr())
    X.shadow_alloc_batch(c.handle, w.base, w.size)
    known = ~w.fresh
    if known.any():
        X.shadow_set_batch(c.handle, w.base[known], w.size[known], np.zeros(int(known.sum()), np.uint8))
    if w.dev_runs.size:
        X.shadow_set_batch(c.handle, w.dev_runs[:, 0], w.dev_runs[:, 1], np.full(len(w.dev_runs), 0xFF, np.uint8))
    X.cg_sync(c.handle)
    return State(c)


def prepare(case, seed):
    path = case["path"]
    if path == "pointers":
        p = W.pointer_batch(seed=seed, n_alloc=case["allocs"], n_ptrs=case["count"])
        s = State(Context(int(((p.sizes.astype(np.int64) + 255) // 256 * 256).sum()) + 16 * MiB, p.bases.size + 16))
        X.shadow_alloc_batch(s.ctx, p.bases, p.sizes)
        X.shadow_free_batch(s.ctx, p.bases[p.freed])
        X.cg_sync(s.ctx)
        s.rec, s.out = _upload(p.ptrs), torch.zeros((case["count"], 3), dtype=torch.int64, device="cuda")
    elif path == "join":
        b = _join_batch(case, seed)
        s = State(Context(16 * MiB, 16))
        s.rec, s.streams, s.epochs = _upload(b.records), _upload(b.streams), _upload(b.epochs)
        s.out = torch.zeros((case["count"], 2), dtype=torch.int64, device="cuda")
    elif path == "serve":
        w, s_log = _serve_log(case, seed)
        s = _open(w)
        s.log = s_log
        s.cfg = X.cg_serve_config(streams=4, max_batch=64, mem_cap=16 * GiB, plain=0, open_loop=0, blocks_per_cu=0)
    else:
        tracked = path == "propagate" or (path == "rows" and case["prop"])
        w = _rows_world(case, seed) if path == "rows" else \
            _tracked_world(case, seed) if tracked else _check_world(case, seed)
        s = _open(w)
        s.rec, s.out = _upload(w.records), torch.zeros((case["count"], 4), dtype=torch.int64, device="cuda")
        s.mode = X.CG_CHECK | (X.CG_PROPAGATE if tracked else 0)
        s.result = {"verdicts": s.out}
        if tracked:
            # the shadows that the copies write: of the one allocation they fill, and of the end of the host region
            s.result["device"] = s.context.shadow(int(w.base[-1]), int(w.size[-1]))
            if w.written_host:
                s.result["host"] = s.context.hv[w.read:w.read + w.written_host]
    s.path, s.count = path, case["count"]
    return s


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if s.path == "serve":
        res, _ = X.cg_serve_run(s.ctx, s.log, s.cfg)
        return {k: res[k].astype(np.int64) for k in ("flags", "first_bad", "undef_bytes", "avail", "epoch")}
    if s.path == "join":
        X.check_concurrent(s.ctx, s.rec.data_ptr(), s.streams.data_ptr(), s.epochs.data_ptr(), s.count,
                           s.out.data_ptr(), stream)
        return {"flags": s.out[:, 0], "partner": s.out[:, 1]}
    if s.path == "pointers":
        X.check_pointers(s.ctx, s.rec.data_ptr(), s.count, s.out.data_ptr(), stream)
        return s.out
    if s.path == "rows":
        X.check_transfers_2d(s.ctx, s.rec.data_ptr(), s.count, s.out.data_ptr(), s.mode, stream)
    else:
        X.check_transfers(s.ctx, s.rec.data_ptr(), s.count, s.out.data_ptr(), s.mode, stream)
    return s.result


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def _union(lo, n):
    if lo.size == 0:
        return 0
    o = np.argsort(lo, kind="stable")
    lo = lo[o]
    hi = np.maximum.accumulate((lo + n[o]))
    before = np.concatenate([[lo[0]], hi[:-1]])
    return int(np.maximum(hi - np.maximum(before, lo), 0).sum())


def _touched(records):
    """Shadow bytes that the records read: each V byte once, an A bit with each host byte."""
    k, n = records["kind"], records["n"].astype(np.int64)
    src, dst = records["src"].astype(np.int64), records["dst"].astype(np.int64)
    up, down = _union(src[k == 0], n[k == 0]), _union(dst[k == 1], n[k == 1])
    return up * 9 / 8 + down / 8 + _union(src[k != 0], n[k != 0])


def work(case):
    path, T = case["path"], case["count"]
    if path == "pointers":
        return {"bytes": 32 * T + 24 * case["allocs"], "flops": 0}
    if path == "join":
        return {"bytes": 56 * T, "flops": 0}
    if path == "serve":
        w, log = _serve_log(case, 0)
        return {"bytes": 104 * T + _touched(log[log["type"] == X.CG_EV_CHECK]), "flops": 0}
    if path == "rows":
        r = _rows_world(case, 0).records
        n = (r["rows"] * r["width"]).astype(np.int64)
        flat = W.make_records(r["kind"], r["src"], r["dst"], n.astype(np.uint64))  # tight on the host: the rows' bytes
        dev = int(n[r["kind"] != 0].sum())
        host = _touched(flat[flat["kind"] == 0]) + int(n[r["kind"] == 1].sum()) / 8
        return {"bytes": 96 * T + host + dev + (int(n.sum()) if case["prop"] else 0), "flops": 0}
    if path == "propagate":
        r = _tracked_world(case, 0).records
        return {"bytes": 64 * T + _touched(r) + int(r["n"].sum()), "flops": 0}
    return {"bytes": 64 * T + _touched(_check_world(case, 0).records), "flops": 0}


# ---- the results from their definitions ------------------------------------------------------------------------
def _t(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a).astype(np.int64))).cuda()


def _verdicts(w, kind, src, dst, n):
    """[flags, first_bad, undef_bytes, avail] of transfers inside the host region or anywhere on the device."""
    none = torch.full_like(n, -1)
    big = torch.full_like(n, (1 << 63) - 1)
    base, end = _t(w.base), _t(w.base + w.size)
    host, down, d2d = kind == 0, kind == 1, kind == 2

    def owner(p):
        j = torch.searchsorted(base, p, right=True) - 1
        k = j.clamp(min=0)
        ok = (j >= 0) & (p < end[k])
        return ok, torch.where(ok, end[k] - p, torch.zeros_like(p))

    s_ok, s_av = owner(src)
    d_ok, d_av = owner(dst)
    first, flags = big.clone(), torch.zeros_like(n)

    def flag(where, bit, at):
        flags.add_(where.to(torch.int64) * bit)
        first.copy_(torch.where(where, torch.minimum(first, at), first))

    zero = torch.zeros_like(n)
    flag(~host & ~s_ok, X.CG_SRC_UNALLOC, zero)
    flag(~host & s_ok & (n > s_av), X.CG_SRC_OVERRUN, s_av)
    flag(~down & ~d_ok, X.CG_DST_UNALLOC, zero)
    flag(~down & d_ok & (n > d_av), X.CG_DST_OVERRUN, d_av)
    apart = torch.where(src < dst, dst - src, src - dst)
    flag(d2d & (apart < n), X.CG_OVERLAP, big)
    # host bytes without address: whole pages
    page = _t(w.hb + w.pages * 4096)
    for where, p, bit in ((host, src, X.CG_SRC_UNADDR), (down, dst, X.CG_DST_UNADDR)):
        if page.numel():
            j = torch.searchsorted(page + 4096, p, right=True)
            at = torch.maximum(torch.where(j < page.numel(), page[j.clamp(max=page.numel() - 1)], big), p) - p
            flag(where & (at < n), bit, at)
    # undefined bytes
    hu = torch.cat([torch.nonzero(v).reshape(-1) + i * GiB for i, v in enumerate(w.host_v()[:w.host].split(GiB))])
    if page.numel() and hu.numel():
        hu = hu[~torch.isin(hu >> 12, _t(w.pages))]
    hu = hu + w.hb
    du = _t(np.unique(_spread(*w.dev_runs.T))) if w.dev_runs.size else _t([])
    valid = torch.where(host, n, torch.minimum(n, s_av))
    undef = zero.clone()
    for where, u in ((host, hu), (~host, du)):
        if u.numel():
            a, b = torch.searchsorted(u, src), torch.searchsorted(u, src + valid)
            c = torch.where(where, b - a, zero)
            undef += c
            flag(c > 0, X.CG_SRC_UNDEF, u[a.clamp(max=u.numel() - 1)] - src)
    avail = torch.where(host, d_av, torch.where(down, s_av, torch.minimum(s_av, d_av)))
    return torch.stack([flags, torch.where(first == big, none, first), undef, avail], 1)


def _carry(w, out_v, host_v, kind, src, dst, n, reach):
    """The shadow that one copy of n bytes carries to its destination; `reach`: valid bytes of a device source."""
    if kind == 0:
        o = src - w.hb
        v = host_v[o:o + n].clone()
        for p in w.pages[(w.pages * 4096 < o + n) & ((w.pages + 1) * 4096 > o)].tolist():
            v[max(p * 4096 - o, 0):max((p + 1) * 4096 - o, 0)] = 0xFF
    else:
        v = torch.zeros(n, dtype=torch.uint8, device="cuda")
        v[reach:] = 0xFF
        for a, k in w.runs_of(src, src + n):
            v[max(a - src, 0):max(min(a + k - src, reach), 0)] = 0xFF
    if kind == 1:
        host_v[dst - w.hb:dst - w.hb + n] = v
    else:
        o = dst - int(w.base[-1])
        out_v[o:o + n] = v


def exact(case, seed):
    path = case["path"]
    if path == "serve":
        return None   # every request has a table of its own
    if path == "join":
        b = _join_batch(case, seed)
        if min(case["epoch"], case["count"]) > 16_384:
            return None
        flags = torch.zeros(case["count"], dtype=torch.int64, device="cuda")
        r, st, ep = b.records, _t(b.streams), b.epochs.astype(np.int64)
        cut = np.flatnonzero(np.diff(ep)) + 1
        for lo, hi in zip(np.append(0, cut), np.append(cut, ep.size)):
            s, d, n, q = _t(r["src"][lo:hi]), _t(r["dst"][lo:hi]), _t(r["n"][lo:hi]), st[lo:hi]
            apart = q[:, None] != q[None, :]

            def meet(a, c):
                return ((a[:, None] < (c + n)[None, :]) & (c[None, :] < (a + n)[:, None]) & apart).any(1)

            flags[lo:hi] = meet(s, d).to(torch.int64) * X.CG_RACE_SRC + (meet(d, s) | meet(d, d)) * X.CG_RACE_DST
        return {"flags": flags, "partner": None}   # any conflicting record may be named
    if path == "pointers":
        p = W.pointer_batch(seed=seed, n_alloc=case["allocs"], n_ptrs=case["count"])
        keep = np.ones(p.bases.size, bool)
        keep[p.freed] = False
        base, size, q = _t(p.bases[keep]), _t(p.sizes[keep]), _t(p.ptrs)
        j = (torch.searchsorted(base, q, right=True) - 1)
        k = j.clamp(min=0)
        ok = (j >= 0) & (q <= base[k] + size[k])
        zero = torch.zeros_like(q)
        return torch.stack([(~ok).to(torch.int64), torch.where(ok, base[k], zero),
                            torch.where(ok, base[k] + size[k] - q, zero)], 1)
    if path == "rows":
        w = _rows_world(case, seed)
        r = w.records
        rows, T = _t(r["rows"]), case["count"]
        of = torch.repeat_interleave(torch.arange(T, device="cuda"), rows)
        at = torch.arange(of.numel(), device="cuda") - (torch.cumsum(rows, 0) - rows)[of]
        width = torch.full_like(of, case["width"])
        v = _verdicts(w, _t(r["kind"])[of], _t(r["src"])[of] + at * _t(r["spitch"])[of],
                      _t(r["dst"])[of] + at * _t(r["dpitch"])[of], width)
        big = (1 << 63) - 1
        first = torch.where(v[:, 1] < 0, torch.full_like(at, big), v[:, 1] + at * case["width"])
        first = torch.full((T,), big, device="cuda").scatter_reduce(0, of, first, "amin")
        flags = sum(torch.zeros(T, dtype=torch.int64, device="cuda").scatter_reduce(0, of, v[:, 0] & (1 << k), "amax")
                    for k in range(10))
        undef = torch.zeros(T, dtype=torch.int64, device="cuda").scatter_add(0, of, v[:, 2])
        out = {"verdicts": torch.stack([flags, torch.where(first == big, torch.full_like(first, -1), first), undef,
                                        v[(torch.cumsum(rows, 0) - rows), 3]], 1)}
        tracked = case["prop"]
        if tracked and (int(r["rows"].sum()) > 100_000):
            return dict(out, device=None, host=None)   # too many rows to carry one by one
        pieces = [(int(x["kind"]), int(x["src"]) + i * int(x["spitch"]), int(x["dst"]) + i * int(x["dpitch"]),
                   case["width"]) for x in r for i in range(int(x["rows"]))] if tracked else []
    else:
        tracked = path == "propagate"
        w = _tracked_world(case, seed) if tracked else _check_world(case, seed)
        r = w.records
        out = {"verdicts": _verdicts(w, _t(r["kind"]), _t(r["src"]), _t(r["dst"]), _t(r["n"]))}
        pieces = list(zip(r["kind"].tolist(), r["src"].tolist(), r["dst"].tolist(), r["n"].tolist())) if tracked else []
    if tracked:
        starts = np.sort(w.dev_runs[:, 0])
        length = w.dev_runs[np.argsort(w.dev_runs[:, 0]), 1]
        w.runs_of = lambda a, b: [(int(starts[i]), int(length[i])) for i in
                                  range(np.searchsorted(starts, a - 64), np.searchsorted(starts, b))]
        ends = w.base + w.size
        hv = w.host_v()
        device = torch.full((int(w.size[-1]),), 0xFF, dtype=torch.uint8, device="cuda")
        for kind, src, dst, n in pieces:
            reach = n if kind == 0 else min(n, int(ends[np.searchsorted(w.base, src, side="right") - 1]) - src)
            _carry(w, device, hv, kind, src, dst, n, reach)
        out["device"] = device
        if w.written_host:
            out["host"] = hv[w.read:w.read + w.written_host]
    return out

"""Edges of the device paths: sizes where a kernel's split, its remainder or
the rule that chooses it changes, against the oracle or a plain host model."""
import numpy as np
import pytest

from paper_1310_0901_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def X():
    from paper_1310_0901_amd import xfercheck
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    xfercheck.lib()
    return xfercheck


@pytest.mark.parametrize("n0", [0, 1, 63, 255, 256, 257, 5000])
@pytest.mark.parametrize("words", [1, 3, 95, 96, 97, 400])
def test_table_change_by_merge(X, n0, words):
    """A table version made from the one before by `words` words of frees and
    allocations (up to 96 travel in the launch's arguments, more through
    device memory): every entry and the top level equal the sorted list.
    Allocations go before, between, after and in place of the old entries."""
    rng = np.random.default_rng(1000 * n0 + words)
    step = 4096
    base = W.DEV_BASE + step * 8 * np.arange(1, n0 + 1, dtype=np.int64)
    ctx = X.cg_create(0, 64 << 20, n0 + 512)
    try:
        live = {int(b): 300 for b in base}
        if n0:
            X.shadow_alloc_batch(ctx, base, np.full(n0, 300))
        X.cg_table_read(ctx, n0 + 16)                       # the version to change
        nfree = min(words % 3 + 3 * int(rng.integers(0, words // 6 + 1)), n0)
        nins = (words - nfree) // 3
        nfree = min(words - 3 * nins, n0)
        kill = rng.choice(base, nfree, replace=False) if nfree else []
        for b in kill:
            X.shadow_free(ctx, int(b))
            live.pop(int(b))
        slots = np.setdiff1d(W.DEV_BASE + step * np.arange(0, 8 * n0 + 520, dtype=np.int64), np.array(list(live)))
        again = list(kill[: nins // 3])
        new = np.unique(np.concatenate([again, rng.choice(slots, nins, replace=False)]).astype(np.int64))[:nins]
        for b in new:
            live[int(b)] = int(rng.integers(1, 300))
            X.shadow_alloc(ctx, int(b), live[int(b)])
        t = X.cg_table_read(ctx, n0 + 512)
        keys = np.array(sorted(live), np.uint64)
        sizes = np.array([live[int(k)] for k in keys], np.uint64)
        assert np.array_equal(t["base"], keys) and np.array_equal(t["end"], keys + sizes)
        assert np.array_equal(t["top"], keys[:: 1 << t["shift"]])
        for b, o in zip(t["base"], t["off"]):
            assert X.shadow_ptr(ctx, int(b)) == t["pool"] + int(o)
    finally:
        X.cg_destroy(ctx)


@pytest.mark.parametrize("count", [1, 63, 64, 65, 200])
def test_fills_of_many_ranges(X, count):
    """shadow_set_batch of up to 64 ranges (in the launch's arguments) and of
    more (uploaded), at every start and length modulo 16: each byte set has
    the last value written to it, every other keeps its own."""
    from paper_1310_0901_amd import harness as H
    rng = np.random.default_rng(count)
    size = 1 << 20
    ctx = X.cg_create(0, 4 << 20, 16)
    try:
        X.shadow_alloc(ctx, W.DEV_BASE, size)
        cut = np.sort(rng.choice(size, 2 * count, replace=False))
        a, n = cut[::2], cut[1::2] - cut[::2]
        v = rng.integers(0, 255, count)
        X.shadow_set_batch(ctx, W.DEV_BASE + a, n, v)
        X.cg_sync(ctx)
        want = np.full(size, 0xFF, np.uint8)
        for s, k, x in zip(a, n, v):
            want[s:s + k] = x
        assert np.array_equal(H.read_device(X.shadow_ptr(ctx, W.DEV_BASE), size), want)
    finally:
        X.cg_destroy(ctx)


@pytest.mark.parametrize("nalloc", [0, 1, 2, 3, 1024, 1025, 8191, 8192, 8193, 16385, 131071, 131073, 140001])
def test_pointers_at_table_edges(X, nalloc):
    """check_pointers around the sizes where the table's middle level (8,192
    entries) stops holding every base, its stride doubles, and the fine level
    (every 16th base, from 131,073 entries on) joins in: pointers one
    below, at, inside, at the end of and one past the end of allocations, some
    of them adjacent, at 1, 300 and 300,000 pointers (both staged levels)."""
    from oracle import oracle
    rng = np.random.default_rng(nalloc)
    sizes = rng.integers(1, 700, nalloc)
    gaps = rng.integers(0, 2, nalloc) * rng.integers(1, 300, nalloc)
    base = W.DEV_BASE + np.cumsum(sizes + gaps) - sizes
    ctx = X.cg_create(0, 256 << 20, nalloc + 16)
    try:
        if nalloc:
            X.shadow_alloc_batch(ctx, base, sizes)
        ends = np.concatenate([base - 1, base, base + sizes // 2, base + sizes - 1, base + sizes, base + sizes + 1,
                               [0, 1, (1 << 63) - 1]])
        for count in (1, 300, 300_000):
            p = rng.choice(ends, count).astype(np.uint64)
            t = torch.from_numpy(p.view(np.int64)).cuda()
            out = torch.zeros((count, 3), dtype=torch.int64, device="cuda")
            X.check_pointers(ctx, t.data_ptr(), count, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(W.PTR_DTYPE).reshape(-1)
            # the oracle scans its list: give it the allocations the sample can lie in
            keep = np.arange(nalloc) if nalloc <= 1025 else np.unique(rng.choice(nalloc, 400))
            ok = np.isin(p.astype(np.int64), np.concatenate([e[keep] for e in (base - 1, base, base + sizes // 2,
                         base + sizes - 1, base + sizes, base + sizes + 1)] + [np.array([0, 1, (1 << 63) - 1])]))
            near = np.unique(np.clip(np.concatenate([keep - 1, keep, keep + 1, keep + 2]), 0, max(nalloc - 1, 0)))
            near = near[:nalloc] if nalloc else np.zeros(0, np.int64)
            want = oracle.pointers(base[near].astype(np.uint64), sizes[near].astype(np.uint64), p[ok])
            for f in ("flags", "base", "avail"):
                assert np.array_equal(got[ok][f], want[f]), (count, f)
    finally:
        X.cg_destroy(ctx)


def edge_world(rng, hl, sizes, dens=0.003):
    """A host region and allocations with faults everywhere, 4,096 bytes apart."""
    from tests import util
    hv = np.where(rng.random(hl) < dens, rng.integers(1, 256, hl), 0).astype(np.uint8)
    a = (rng.random(hl) > 0.0005).astype(np.uint8)
    a[-1] = a[0] = 1
    base = W.DEV_BASE + 4096 * np.arange(1, len(sizes) + 1) + np.concatenate([[0], np.cumsum(sizes)[:-1]]) + 5
    vs = [np.where(rng.random(int(s)) < dens, rng.integers(1, 256, int(s)), 0).astype(np.uint8) for s in sizes]
    return util.workload_from_arrays(W.HOST_BASE, hv, a, base, sizes, vs, np.zeros(0, W.RECORD_DTYPE)), base


def compare_state(H, w, base, sizes, o, call, want):
    from tests import util
    dw = H.DeviceWorld(w)
    try:
        util.assert_verdicts_equal(call(dw), want)
        for j in range(len(sizes)):
            assert np.array_equal(dw.alloc_shadow(base[j], sizes[j]), o.vs[j]), f"allocation {j}"
        assert np.array_equal(dw.host_shadow(), o.hv), "host region shadow"
    finally:
        dw.close()


@pytest.mark.parametrize("seed", range(4))
def test_windows_at_edges(X, seed):
    """Transfers at every pair of source and destination alignments and at
    lengths around a window, a wave's windows and a wave's iterations, some
    reaching past the region or their allocation on either side: checks and
    propagation, as one launch of 200 records and as a batch of 600."""
    from paper_1310_0901_amd import harness as H
    from tests import util
    rng = np.random.default_rng(9000 + seed)
    read, T = 300_001, 600
    lens = [1, 2, 15, 16, 17, 31, 33, 1007, 1023, 1024, 1025, 2047, 2049, 4095, 4096, 4097, 8191, 8193, 16_400, 33_000]
    n = rng.choice(lens, T)
    kind = rng.choice(3, T, p=[0.4, 0.3, 0.3])
    gap = rng.integers(1, 40, T)
    pos = np.cumsum(n + gap) - n
    sizes = np.array([200_003, int(pos[-1] + n[-1]) + 100])
    hl = read + int(pos[-1] + n[-1]) + 7
    w, base = edge_world(rng, hl, sizes)
    src = np.where(kind == 0, W.HOST_BASE + rng.integers(0, read - 33_000, T), base[0] + rng.integers(0, 200_003 - 33_000, T))
    dst = np.where(kind == 1, W.HOST_BASE + read + pos, base[1] + pos)
    edge = rng.random(T)
    # sources before and past the region, and past the allocation's end
    src = np.where((kind == 0) & (edge < 0.1), W.HOST_BASE - rng.integers(0, 40, T), src)
    src = np.where((kind != 0) & (edge < 0.1), base[0] + 200_003 - rng.integers(1, 40, T), src)
    rec = W.make_records(kind, src.astype(np.uint64), dst.astype(np.uint64), n.astype(np.uint64))
    for part in (rec[:200], rec):
        want = util.oracle_for(w).run(part)
        dw = H.DeviceWorld(w)
        try:
            for mode in (X.CG_CHECK, X.CG_CHECK | X.CG_KEEP_ORDER, X.CG_CHECK | X.CG_PLAIN):
                util.assert_verdicts_equal(dw.check(part, mode), want, f"mode {mode}")
        finally:
            dw.close()
        o = util.oracle_for(w)
        want = o.run(part, propagate=True)
        for mode in (X.CG_CHECK | X.CG_PROPAGATE, X.CG_CHECK | X.CG_PROPAGATE | X.CG_PLAIN):
            compare_state(H, w, base, sizes, o, lambda dw: dw.check(part, mode), want)


@pytest.mark.parametrize("width,pitch", [(1, 1), (1, 7), (15, 16), (16, 16), (17, 40), (333, 512), (1008, 1024),
                                         (1023, 1023), (1025, 1100), (4030, 4096), (65_519, 65_520), (65_520, 65_536),
                                         (65_521, 65_600), (65_537, 65_537), (100, (1 << 20) - 1), (100, 1 << 20),
                                         (2000, (1 << 20) + 5)])
def test_rows_at_edges(X, width, pitch):
    """Pitched copies around the sizes where rows change how they are worked:
    a window, a wave, 4,096 units a row, pitches of 1 MiB; tight rows on one
    side and pitched rows on the other, at odd alignments."""
    from paper_1310_0901_amd import harness as H
    from tests import util
    from tests.test_gpu_2d import check2d
    rng = np.random.default_rng(width + pitch)
    rows = 5 if pitch >= 65_000 else 77
    span, tight = (rows - 1) * pitch + width, rows * width
    sizes = np.array([span + 3, 2 * (span + 64)])
    read = max(tight, 64) + 50
    w, base = edge_world(rng, read + tight + 40, sizes, dens=0.001)
    rec = np.zeros(3, W.RECORD2D_DTYPE)
    rec["width"], rec["rows"], rec["kind"] = width, rows, [0, 1, 2]
    rec["src"] = [W.HOST_BASE + 3, base[0] + 1, base[0] + 2]
    rec["dst"] = [base[1] + 7, W.HOST_BASE + read + 5, base[1] + span + 64]
    rec["spitch"] = [width, pitch, pitch]
    rec["dpitch"] = [pitch, width, pitch]
    want = util.oracle_for(w).run2d(rec)
    dw = H.DeviceWorld(w)
    try:
        util.assert_verdicts_equal(check2d(X, dw, rec, X.CG_CHECK), want, "check")
    finally:
        dw.close()
    o = util.oracle_for(w)
    want = o.run2d(rec, propagate=True)
    compare_state(H, w, base, sizes, o, lambda dw: check2d(X, dw, rec, X.CG_CHECK | X.CG_PROPAGATE), want)


@pytest.mark.parametrize("knobs", [{}, {"XC_SHADOW_INDEX": "2"}, {"XC_SHADOW_INDEX": "2", "XC_SIDX_CAP": "40"},
                                   {"XC_REORDER_MIN": "1"}, {"XC_REORDER_MIN": "1", "XC_SHADOW_INDEX": "2"},
                                   {"XC_REORDER_MIN": "1", "XC_SHADOW_INDEX": "2", "XC_SIDX_CAP": "40"},
                                   {"XC_REORDER_MIN": "1", "XC_SHADOW_INDEX": "0"}])
def test_ranges_at_granule_edges(X, knobs, monkeypatch):
    """Checks whose ranges start and end within a byte of the index's granules
    (4 KiB) and steps (64 KiB), with faults on both sides of them: answered
    from the index, left to the scan by its cost or by full lists, worked as
    segments and in their order.  Run twice on one stream, so that the second
    batch finds the marks and states the first left."""
    from paper_1310_0901_amd import harness as H
    from tests import util
    for k, v in knobs.items():
        monkeypatch.setenv(k, v)
    rng = np.random.default_rng(77)
    hl, T = 5 * 65_536 + 4096 + 3, 700
    sizes = np.array([3 * 65_536 + 9, 4096, 200_000, 1])
    w, base = edge_world(rng, hl, sizes, dens=0.0002)
    cuts = np.array([c + d for c in list(range(0, hl, 4096)) + [hl] for d in (-1, 0, 1) if 0 <= c + d <= hl])
    kind = rng.choice(3, T, p=[0.5, 0.2, 0.3])
    pair = np.sort(rng.choice(cuts, (T, 2)), 1)
    n = np.maximum(pair[:, 1] - pair[:, 0], 1)
    host = W.HOST_BASE + np.minimum(pair[:, 0], hl - n)
    j = rng.choice([0, 0, 0, 1, 2, 3], T)
    n = np.where(kind == 0, n, np.minimum(n, sizes[j]))
    dev = base[j] + (rng.random(T) * (sizes[j] - np.minimum(n, sizes[j]) + 1)).astype(np.int64) // 4096 * 4096
    other = base[2] + rng.integers(0, 100, T)
    rec = W.make_records(kind, np.where(kind == 0, host, dev).astype(np.uint64),
                         np.where(kind == 1, host, other).astype(np.uint64), n.astype(np.uint64))
    o = util.oracle_for(w)
    dw = H.DeviceWorld(w)
    try:
        for part in (rec, rec[350:], rec[:300]):
            util.assert_verdicts_equal(dw.check(part), o.run(part), f"{knobs} {len(part)}")
    finally:
        dw.close()


def test_state_order_over_many_checks(X):
    """700 checks on four streams without a host wait, the shadow and the
    allocations they read changed between them: each check sees exactly the
    changes made before it (its completion event is shared by what waits for
    it, and comes back from the pool after 256 checks)."""
    n, K = 70_000, 700
    hv = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    ha = torch.full((64,), -1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    ctx = X.cg_create(0, 8 << 20, 64)
    try:
        X.cg_host_register(ctx, W.HOST_BASE, 4096, hv.data_ptr(), ha.data_ptr())
        a, b = W.DEV_BASE, W.DEV_BASE + (1 << 20)
        X.shadow_alloc(ctx, a, n)
        X.shadow_alloc(ctx, b, n)
        X.shadow_set(ctx, b, n, 0)
        rec = W.make_records([2], np.array([a], np.uint64), np.array([b], np.uint64), np.array([n], np.uint64))
        rt = torch.from_numpy(rec.view(np.uint8).copy()).cuda()
        out = torch.zeros((K, 4), dtype=torch.int64, device="cuda")
        streams = [torch.cuda.Stream() for _ in range(3)] + [torch.cuda.current_stream()]
        torch.cuda.synchronize()
        rng = np.random.default_rng(5)
        undef, live, want = n, True, []
        for k in range(K):
            x = rng.random()
            if x < 0.4 and live:
                m = int(rng.integers(1, n))
                X.shadow_set(ctx, a, n, 0)
                X.shadow_set(ctx, a + n - m, m, 0xFF)
                undef = m
            elif x < 0.5:
                if live:
                    X.shadow_free(ctx, a)
                else:
                    X.shadow_alloc(ctx, a, n)
                    undef = n
                live = not live
            call = X.check_transfers if rng.random() < 0.7 else X.check_transfers_noalloc
            st = streams[int(rng.integers(4))] if call is X.check_transfers else streams[3]
            call(ctx, rt.data_ptr(), 1, out[k].data_ptr(), X.CG_CHECK, st.cuda_stream)
            want.append((X.CG_SRC_UNDEF, n - undef, undef, n) if live else (X.CG_SRC_UNALLOC, 0, 0, 0))
        torch.cuda.synchronize()
        bad = np.flatnonzero((out.cpu().numpy() != np.array(want, np.int64)).any(1))
        assert bad.size == 0, (bad[:10], out.cpu().numpy()[bad[:3]], [want[i] for i in bad[:3]])
    finally:
        X.cg_destroy(ctx)


@pytest.mark.parametrize("count", [257, 511, 512, 513, 65_535, 65_537, 262_144, 262_145, 300_000])
@pytest.mark.parametrize("long", ["none", "first", "middle", "last"])
def test_tiles_of_many_records(X, count, long):
    """The tiles of a batch at the edges of a classify block and of the number
    of blocks whose sums one block holds, with one record of many tiles among
    short and empty ones, and with the records in the order given (no
    segments)."""
    from paper_1310_0901_amd import harness as H
    from tests import util
    rng = np.random.default_rng(count)
    w, base = edge_world(rng, 6_000_000, np.array([6_000_000]))
    n = rng.choice([0, 1, 16, 40, 300], count)
    if long != "none":
        n[{"first": 0, "middle": count // 2, "last": -1}[long]] = 5_000_000
    src = W.HOST_BASE + rng.integers(0, 900_000, count)
    rec = W.make_records(np.zeros(count, np.int64), src.astype(np.uint64), np.full(count, base[0], np.uint64),
                         n.astype(np.uint64))
    want = util.oracle_for(w).run(rec)
    dw = H.DeviceWorld(w)
    try:
        for mode in (X.CG_CHECK, X.CG_CHECK | X.CG_KEEP_ORDER):
            util.assert_verdicts_equal(dw.check(rec, mode), want, f"mode {mode}")
    finally:
        dw.close()

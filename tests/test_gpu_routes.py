"""Which way a call is worked: calls that differ in one argument and share
their buffers, launch shapes, and batches around the sizes where the way
changes."""
import numpy as np
import pytest

from paper_1310_0901_amd import workloads as W
from tests.test_gpu_paths import compare_state, edge_world

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def X():
    from paper_1310_0901_amd import xfercheck
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    xfercheck.lib()
    return xfercheck


@pytest.fixture(scope="module")
def H(X):
    from paper_1310_0901_amd import harness
    return harness


def uploads(rng, count, read, base, n):
    """`count` host-to-device records of n bytes (a number or one per record) from anywhere in the region."""
    n = np.broadcast_to(np.asarray(n, np.int64), count)
    src = W.HOST_BASE + (rng.random(count) * (read - n + 1)).astype(np.int64)
    return W.make_records(np.zeros(count, np.int64), src.astype(np.uint64), np.full(count, base, np.uint64),
                          n.astype(np.uint64))


@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("kept_first", [False, True])
def test_kept_order_on_the_same_buffers(X, H, timing, kept_first, monkeypatch):
    """A check and the same check with CG_KEEP_ORDER on one pair of buffers,
    both as graph replays: the first is answered from the shadow indexes, the
    second is not, whichever came first."""
    from tests import util
    monkeypatch.setenv("XC_SHADOW_INDEX", "2")
    rng = np.random.default_rng(31)
    w, base = edge_world(rng, 300_000, np.array([300_000]))
    rec = uploads(rng, 600, 300_000, base[0], rng.integers(1, 9000, 600))
    want = util.oracle_for(w).run(rec)
    dw = H.DeviceWorld(w)
    try:
        X.cg_timing(dw.ctx, timing)
        rt, out = H.records_tensor(rec), H.verdicts_tensor(len(rec))
        s = torch.cuda.current_stream().cuda_stream
        X.cg_index_ms(dw.ctx)
        modes = [X.CG_CHECK, X.CG_CHECK | X.CG_KEEP_ORDER]
        for mode in (modes[::-1] if kept_first else modes) * 2:
            out.zero_()
            X.check_transfers(dw.ctx, rt.data_ptr(), len(rec), out.data_ptr(), mode, s)
            torch.cuda.synchronize()
            util.assert_verdicts_equal(H.verdicts_np(out, len(rec)), want, f"mode {mode}")
            _, passes, read = X.cg_index_ms(dw.ctx)
            indexed = mode == X.CG_CHECK
            assert (read[0] > 0) == indexed, f"mode {mode}: index bytes {read}"
            assert passes == (1 if indexed and timing else 0)
    finally:
        dw.close()


@pytest.mark.parametrize("propagate", [False, True])
def test_one_launch_of_many_records(X, H, propagate):
    """check_transfers_noalloc of 4,096 records of 64 bytes: the verdicts are
    the oracle's, and the call, whose records are all on the device at once,
    takes less than 3 times that of 256 of them (about 1.6 times; 5 times when
    a compute unit holds one block)."""
    import time
    from tests import util
    rng = np.random.default_rng(12)
    T = 4096
    w, base = edge_world(rng, 1 << 20, np.array([80 * T]))
    rec = uploads(rng, T, 1 << 20, base[0], 64)
    rec["dst"] += np.uint64(80) * np.arange(T, dtype=np.uint64)
    mode = X.CG_CHECK | (X.CG_PROPAGATE if propagate else 0)
    want = util.oracle_for(w).run(rec, propagate=propagate)
    dw = H.DeviceWorld(w)
    try:
        rt, out = H.records_tensor(rec), H.verdicts_tensor(T)
        s = torch.cuda.current_stream().cuda_stream

        def us(count):
            best = []
            for _ in range(7):
                torch.cuda.synchronize()
                t = time.perf_counter()
                for _ in range(40):
                    X.check_transfers_noalloc(dw.ctx, rt.data_ptr(), count, out.data_ptr(), mode, s)
                torch.cuda.synchronize()
                best.append((time.perf_counter() - t) / 40 * 1e6)
            return min(best)
        few, many = us(256), us(T)
        util.assert_verdicts_equal(H.verdicts_np(out, T), want)
        assert many < 3 * few, f"256 records {few:.1f} us, {T} records {many:.1f} us"
    finally:
        dw.close()


@pytest.mark.parametrize("unroll", [1, 2, 4, 8])
@pytest.mark.parametrize("width,pitch,rows", [(333, 512, 90), (70_001, 70_400, 5)])
def test_pitched_rows_at_every_unroll(X, H, unroll, width, pitch, rows):
    """Pitched copies, checked and carried, at each unroll that cg_set_tuning takes."""
    from tests import util
    from tests.test_gpu_2d import check2d
    rng = np.random.default_rng(width)
    span, tight = (rows - 1) * pitch + width, rows * width
    sizes = np.array([span + 3, 2 * (span + 64)])
    read = tight + 50
    w, base = edge_world(rng, read + tight + 40, sizes, dens=0.001)
    rec = np.zeros(3, W.RECORD2D_DTYPE)
    rec["width"], rec["rows"], rec["kind"] = width, rows, [0, 1, 2]
    rec["src"] = [W.HOST_BASE + 3, base[0] + 1, base[0] + 2]
    rec["dst"] = [base[1] + 7, W.HOST_BASE + read + 5, base[1] + span + 64]
    rec["spitch"] = [width, pitch, pitch]
    rec["dpitch"] = [pitch, width, pitch]

    def at_unroll(mode):
        def call(dw):
            t = X.cg_get_tuning(dw.ctx)
            t.unroll = unroll
            X.cg_set_tuning(dw.ctx, t)
            return check2d(X, dw, rec, mode)
        return call
    o = util.oracle_for(w)
    compare_state(H, w, base, sizes, o, at_unroll(X.CG_CHECK), util.oracle_for(w).run2d(rec))
    o = util.oracle_for(w)
    want = o.run2d(rec, propagate=True)
    compare_state(H, w, base, sizes, o, at_unroll(X.CG_CHECK | X.CG_PROPAGATE), want)


@pytest.mark.parametrize("unroll", [1, 2, 4, 8])
def test_checks_at_every_unroll(X, H, unroll, monkeypatch):
    """Checks of all kinds at odd alignments and lengths around a wave's
    iterations, many of their sides unallocated, outside the region or past
    an end, so that a record has destination windows and no source byte, or
    the other way round: in one launch, as a batch, in the order given, one
    launch a record, and cut into segments."""
    from tests import util
    rng = np.random.default_rng(51)
    hl, T = 150_001, 900
    sizes = np.array([140_003, 5000])
    w, base = edge_world(rng, hl, sizes)
    n = rng.choice([1, 15, 16, 17, 1023, 1024, 1025, 4095, 4097, 8191, 16_400, 33_000, 70_001], T)
    kind = rng.choice(3, T)
    nowhere = W.DEV_BASE - 4096 + rng.integers(0, 64, T)

    def device(k):
        j = rng.integers(0, 2, T)
        p = base[j] + rng.integers(0, 1 << 30, T) % sizes[j]
        return np.where(rng.random(T) < 0.3, nowhere, p) if k else p
    host = W.HOST_BASE - 40 + rng.integers(0, hl + 80, T)
    rec = W.make_records(kind, np.where(kind == 0, host, device(1)).astype(np.uint64),
                         np.where(kind == 1, host, device(1)).astype(np.uint64), n.astype(np.uint64))
    want = util.oracle_for(w).run(rec)
    for knobs, part, modes in (({"XC_SHADOW_INDEX": "0"}, slice(0, 200), (0,)),
                               ({"XC_SHADOW_INDEX": "0"}, slice(0, T), (0, X.CG_KEEP_ORDER, X.CG_PLAIN)),
                               ({"XC_SHADOW_INDEX": "0", "XC_REORDER_MIN": "1"}, slice(0, T), (0,)),
                               ({"XC_SHADOW_INDEX": "0", "XC_REORDER_MIN": "1", "XC_HOST_LDS": "0"}, slice(0, T), (0,))):
        for k, v in knobs.items():
            monkeypatch.setenv(k, v)
        dw = H.DeviceWorld(w)
        try:
            t = X.cg_get_tuning(dw.ctx)
            t.unroll = unroll
            X.cg_set_tuning(dw.ctx, t)
            for mode in modes:
                util.assert_verdicts_equal(dw.check(rec[part], X.CG_CHECK | mode), want[part], f"{knobs} mode {mode}")
        finally:
            dw.close()


def test_blocks_per_cu_are_the_callers(X, H, monkeypatch):
    """A caller's blocks_per_cu is the number of blocks launched: with one
    16-byte load in flight per lane, one block of 256 threads per compute unit
    streams the shadow at a fraction of the rate that four have (four blocks
    are enough, so a launch of four times what is asked for shows no
    difference).  A new context's own choice survives cg_get_tuning and
    cg_set_tuning until the caller sets another number."""
    monkeypatch.setenv("XC_SHADOW_INDEX", "0")
    n, T = 1 << 20, 512
    hv = torch.zeros(T * n, dtype=torch.uint8, device="cuda")
    ha = torch.full((T * n // 64,), -1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    ctx = X.cg_create(0, 4 << 20, 16)
    try:
        X.cg_host_register(ctx, W.HOST_BASE, T * n, hv.data_ptr(), ha.data_ptr())
        X.shadow_alloc(ctx, W.DEV_BASE, n)
        rec = W.make_records(np.zeros(T, np.int64), (W.HOST_BASE + n * np.arange(T)).astype(np.uint64),
                             np.full(T, W.DEV_BASE, np.uint64), np.full(T, n, np.uint64))
        rt, out = H.records_tensor(rec), H.verdicts_tensor(T)
        s = torch.cuda.current_stream().cuda_stream
        X.cg_timing(ctx, True)

        def ms():
            got = []
            for _ in range(5):
                X.check_transfers(ctx, rt.data_ptr(), T, out.data_ptr(), X.CG_CHECK | X.CG_KEEP_ORDER, s)
                got.append(X.cg_kernel_ms(ctx)[0])
            return min(got)
        t = X.cg_get_tuning(ctx)
        assert (t.blocks_per_cu, list(t.reserved)) == (4, [1, 0, 0])
        own = ms()
        X.cg_set_tuning(ctx, t)
        assert list(X.cg_get_tuning(ctx).reserved) == [1, 0, 0]
        t.unroll, t.blocks_per_cu = 1, 1
        X.cg_set_tuning(ctx, t)
        assert list(X.cg_get_tuning(ctx).reserved) == [0, 0, 0]
        one = ms()
        t.blocks_per_cu = 4
        X.cg_set_tuning(ctx, t)
        four = ms()
        assert one > 1.5 * four, f"blocks per CU: 1 {one:.3f} ms, 4 {four:.3f} ms"
        assert own < 1.3 * four, f"the context's own choice {own:.3f} ms, 4 {four:.3f} ms"
    finally:
        X.cg_destroy(ctx)


def test_tuner_measures_again_on_new_kernels(X, H, tmp_path, monkeypatch):
    """cg_autotune takes its choice from a line that it wrote itself, and not
    from a line whose key names no generation of the scan kernels or another
    one."""
    monkeypatch.setenv("XC_SHADOW_INDEX", "0")
    rng = np.random.default_rng(3)
    w, base = edge_world(rng, 400_000, np.array([100_000]))
    rec = uploads(rng, 300, 400_000, base[0], 60_000)
    cache = tmp_path / "tuning.jsonl"
    dw = H.DeviceWorld(w)
    try:
        rt, out = H.records_tensor(rec), H.verdicts_tensor(len(rec))
        call = (dw.ctx, rt.data_ptr(), len(rec), out.data_ptr(), X.CG_CHECK, torch.cuda.current_stream().cuda_stream)
        own = X.cg_autotune(*call, str(cache)).as_dict()
        line = cache.read_text()
        key = line.split('"')[3]
        assert len(line.strip().split("\n")) == 1 and "/g" in key
        # a shape the tuner does not try, so that it can only come from the file
        shape = '"block": 512, "unroll": 1, "blocks_per_cu": 5, "tile_units": 131072, "nontemporal": 0'
        head = key[:key.index("/g")]
        cache.write_text("".join(f'{{"key": "{head}{g}", {shape}, "ms": 0.001}}\n' for g in ("", "/g1", "/g99")))
        assert X.cg_autotune(*call, str(cache)).as_dict()["blocks_per_cu"] != 5
        assert len(cache.read_text().strip().split("\n")) == 4
        cache.write_text(f'{{"key": "{key}", {shape}, "ms": 0.001}}\n')
        got = X.cg_autotune(*call, str(cache))
        assert (got.block, got.unroll, got.blocks_per_cu, got.tile_units, got.nontemporal) == (512, 1, 5, 131072, 0)
        assert own["blocks_per_cu"] != 5 and list(got.reserved) == [0, 0, 0]
    finally:
        dw.close()


@pytest.mark.parametrize("before", [0, 300, 3000])
def test_tuner_keys_one_launch_batches_by_their_units(X, H, tmp_path, before, monkeypatch):
    """cg_autotune on a batch worked in one launch, after `before` records in
    another batch on the stream: its key holds its own units (4,096 of a
    64 KiB upload), and only the unroll and the kind of load are chosen."""
    monkeypatch.setenv("XC_SHADOW_INDEX", "0")
    rng = np.random.default_rng(4)
    w, base = edge_world(rng, 400_000, np.array([100_000]))
    cache = tmp_path / "tuning.jsonl"
    dw = H.DeviceWorld(w)
    try:
        if before:
            dw.check(uploads(rng, before, 400_000, base[0], 60_000))
        rec = W.make_records([0], np.array([W.HOST_BASE], np.uint64), np.array([base[0]], np.uint64),
                             np.array([65_536], np.uint64))
        rt, out = H.records_tensor(rec), H.verdicts_tensor(1)
        t0 = X.cg_get_tuning(dw.ctx)
        t = X.cg_autotune(dw.ctx, rt.data_ptr(), 1, out.data_ptr(), X.CG_CHECK,
                          torch.cuda.current_stream().cuda_stream, str(cache))
        assert "/n1/u2^12/m1" in cache.read_text()
        # what one launch does not use stays as it was
        assert (t.block, t.blocks_per_cu, t.tile_units, t.reserved[0]) == \
               (t0.block, t0.blocks_per_cu, t0.tile_units, t0.reserved[0])
    finally:
        dw.close()


@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("count", [1, 2, 40, 600])
def test_one_launch_records_of_several_blocks(X, H, count, kind):
    """Records that one launch works in more than one block (above 128 KiB),
    at lengths around the units of a block and around an iteration of all the
    record's waves, at odd alignments, some reaching past an end, over holes
    and undefined bytes: checked and carried, twice on one stream (the second
    finds the accumulators as the first left them), by check_transfers and by
    check_transfers_noalloc (which alone takes 600 in one launch)."""
    from tests import util
    rng = np.random.default_rng(7 * count + kind)
    lens = np.array([65_536 * k + d for k in range(2, 7) for d in (-17, -1, 0, 1, 33)] + [500, 1_000_003])
    n = rng.choice(lens, count) if count > 2 else np.array([1_000_003, 262_145][:count])
    if count == 600:   # blocks of 512 threads, most records small
        n = np.where(rng.random(count) < 0.9, rng.integers(1, 3000, count), n)
    gap = rng.integers(1, 40, count)
    pos = np.cumsum(n + gap) - n
    far = int(pos[-1] + n[-1]) + 100
    read = 1_300_001
    sizes = np.array([read, far if kind != 1 else 64])
    w, base = edge_world(rng, read + (far if kind == 1 else 0), sizes, dens=0.0005)
    src = (W.HOST_BASE if kind == 0 else base[0]) + rng.integers(0, read - n + 1)
    # (the allocations are 4,096 bytes apart: none of these starts in the one written)
    past = rng.random(count) < 0.2
    src = np.where(past, (W.HOST_BASE if kind == 0 else base[0]) + read - n + rng.integers(1, 4000, count), src)
    dst = (W.HOST_BASE + read if kind == 1 else base[1]) + pos
    rec = W.make_records(np.full(count, kind), src.astype(np.uint64), dst.astype(np.uint64), n.astype(np.uint64))
    s = torch.cuda.current_stream().cuda_stream
    rt, out = H.records_tensor(rec), H.verdicts_tensor(count)

    def call(entry, mode):
        def go(dw):
            for _ in range(2):
                out.zero_()
                entry(dw.ctx, rt.data_ptr(), count, out.data_ptr(), mode, s)
            torch.cuda.synchronize()
            return H.verdicts_np(out, count)
        return go
    for entry in (X.check_transfers, X.check_transfers_noalloc):
        compare_state(H, w, base, sizes, util.oracle_for(w), call(entry, X.CG_CHECK), util.oracle_for(w).run(rec))
        o = util.oracle_for(w)
        want = o.run(rec, propagate=True)
        compare_state(H, w, base, sizes, o, call(entry, X.CG_CHECK | X.CG_PROPAGATE), want)


@pytest.mark.parametrize("n0,nd,ni", [(0, 0, 1), (0, 0, 21), (1, 1, 1), (63, 0, 16), (255, 2, 31), (255, 0, 32), (256, 3, 31),
                                      (257, 1, 32), (5000, 96, 0), (5000, 97, 0), (5000, 1, 133), (5000, 1000, 3),
                                      (9000, 3, 31), (9000, 40, 20), (140_001, 3, 31), (140_001, 5000, 4000)])
def test_tables_made_by_merge(X, n0, nd, ni):
    """A table version made by merging nd frees and ni allocations, nd + 3 ni
    words, into the one before (up to 96 words travel in the launch's
    arguments, up to 4,096 through a small upload, more through a large one):
    made by a merge, and every level right.  The entries and the top level are
    read; the middle level (above 8,192 entries) and the fine level (above
    131,072) answer 300,000 pointers."""
    rng = np.random.default_rng(n0 + 7 * nd + ni)
    step = 4096
    old = W.DEV_BASE + step * 3 * np.arange(1, n0 + 1, dtype=np.int64)
    ctx = X.cg_create(0, (n0 + ni + 16) * 512, n0 + ni + 16)
    try:
        if n0:
            X.shadow_alloc_batch(ctx, old, np.full(n0, 300))
        before = X.cg_table_read(ctx, n0 + 16)
        kill = rng.choice(old, nd, replace=False)
        if nd:
            X.shadow_free_batch(ctx, kill)
        # before, between, after and in place of the old entries
        free = np.concatenate([kill, W.DEV_BASE + step * np.setdiff1d(np.arange(3 * n0 + 3 * ni + 9), 3 * np.arange(1, n0 + 1))])
        new = np.unique(np.concatenate([kill[:ni // 2], rng.choice(np.setdiff1d(free, kill), ni - len(kill[:ni // 2]), replace=False)]))
        size = rng.integers(1, 500, len(new))
        if ni:
            X.shadow_alloc_batch(ctx, new, size)
        t = X.cg_table_read(ctx, n0 + ni + 16)
        assert len(new) == ni and len(kill) == nd
        assert t["merges"] == before["merges"] + 1 and t["full_uploads"] == before["full_uploads"]
        live = {int(b): 300 for b in old}
        for b in kill:
            live.pop(int(b))
        live.update({int(b): int(k) for b, k in zip(new, size)})
        base = np.array(sorted(live), np.uint64)
        end = base + np.array([live[int(b)] for b in base], np.uint64)
        assert np.array_equal(t["base"], base) and np.array_equal(t["end"], end)
        assert np.array_equal(t["top"], base[:: 1 << t["shift"]])
        some = np.arange(len(base)) if len(base) < 300 else rng.choice(len(base), 300, replace=False)
        for j in some:
            assert X.shadow_ptr(ctx, int(base[j])) == t["pool"] + int(t["off"][j])
        p = rng.choice(np.concatenate([base - 1, base, end - 1, end, end + 1, kill.astype(np.uint64)]), 300_000).astype(np.uint64)
        pt = torch.from_numpy(p.view(np.int64)).cuda()
        out = torch.zeros((len(p), 3), dtype=torch.int64, device="cuda")
        X.check_pointers(ctx, pt.data_ptr(), len(p), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(W.PTR_DTYPE).reshape(-1)
        j = np.searchsorted(base, p, side="right") - 1
        k = np.maximum(j, 0)
        ok = (j >= 0) & (p <= end[k])
        assert np.array_equal(got["flags"], np.where(ok, 0, X.CG_PTR_UNALLOC))
        assert np.array_equal(got["base"], np.where(ok, base[k], 0)) and np.array_equal(got["avail"], np.where(ok, end[k] - p, 0))
    finally:
        X.cg_destroy(ctx)


@pytest.mark.parametrize("host_lds", ["1", "0", "2"])
@pytest.mark.parametrize("cap", ["30", "3000"])
@pytest.mark.parametrize("large", [4, 40])
def test_segments_beside_the_indexes(X, H, large, cap, host_lds, monkeypatch):
    """A check of a few large records among many small ones, with the indexes
    on and full (so that nothing or one space is answered from them): with
    40 large ones the batch reads each of its granules more than 4 times and
    is cut into segments, the large records into many; with 4 it reads them
    fewer times and keeps its order.  (A batch that propagates always keeps its
    order.)"""
    from tests import util
    for k, v in (("XC_REORDER_MIN", "1"), ("XC_SEG_MIN_LOG2", "4"), ("XC_SHADOW_INDEX", "2"), ("XC_SIDX_CAP", cap),
                 ("XC_HOST_LDS", host_lds)):
        monkeypatch.setenv(k, v)
    rng = np.random.default_rng(large)
    hl, sizes = 1_500_001, np.array([1_400_003, 1_300_007])
    w, base = edge_world(rng, hl, sizes, dens=0.001)
    T = 500
    n = rng.integers(1, 3000, T)
    n[rng.choice(T, large, replace=False)] = rng.integers(600_000, 1_200_000, large)
    kind = rng.choice([0, 2], T)
    src = np.where(kind == 0, W.HOST_BASE + rng.integers(0, hl - n + 1), base[0] + rng.integers(0, 1_400_003 - n + 1))
    rec = W.make_records(kind, src.astype(np.uint64), np.full(T, base[1], np.uint64), n.astype(np.uint64))
    # the rule's two sides: bytes read, and bytes of the granules they lie in
    off = np.where(kind == 0, src - W.HOST_BASE, src - base[0])
    grans = sum(len(np.unique(np.concatenate([np.arange(o >> 12, ((o + k - 1) >> 12) + 1) for o, k in zip(off[m], n[m])])))
                for m in (kind == 0, kind == 2))
    reads = int(n.sum()) / (4096 * grans)
    assert (reads > 4.5) if large == 40 else (reads < 3.5), reads
    want = util.oracle_for(w).run(rec)
    dw = H.DeviceWorld(w)
    try:
        for mode in (X.CG_CHECK, X.CG_CHECK | X.CG_EAGER, X.CG_CHECK):
            util.assert_verdicts_equal(dw.check(rec, mode), want, f"mode {mode}")
    finally:
        dw.close()


def test_no_room_for_the_indexes(X, H, monkeypatch):
    """Checks on a stream for whose index space there is no room (lists of 2^36
    entries): scanned, with the same verdicts, again and in other shapes, and
    pitched ones as well."""
    from tests import util
    from tests.test_gpu_2d import check2d
    monkeypatch.setenv("XC_SIDX_CAP", str(1 << 36))
    rng = np.random.default_rng(77)
    w, base = edge_world(rng, 300_000, np.array([300_000]))
    rec = uploads(rng, 700, 300_000, base[0], rng.integers(1, 9000, 700))
    want = util.oracle_for(w).run(rec)
    r2 = np.zeros(300, W.RECORD2D_DTYPE)
    r2["width"], r2["rows"], r2["spitch"], r2["dpitch"] = 100, 20, 100, 128
    r2["src"], r2["dst"] = W.HOST_BASE + rng.integers(0, 290_000, 300), base[0]
    dw = H.DeviceWorld(w)
    try:
        for mode in (X.CG_CHECK, X.CG_CHECK | X.CG_EAGER, X.CG_CHECK, X.CG_CHECK | X.CG_KEEP_ORDER):
            util.assert_verdicts_equal(dw.check(rec, mode), want, f"mode {mode}")
        util.assert_verdicts_equal(check2d(X, dw, r2, X.CG_CHECK), util.oracle_for(w).run2d(r2), "pitched")
        assert X.cg_index_ms(dw.ctx)[2] == (0, 0)
    finally:
        dw.close()


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
@pytest.mark.parametrize("entry", ["check_transfers", "check_transfers_noalloc", "check_pointers"])
def test_checks_beside_a_capture(X, H, entry, mode):
    """A program captures work of its own on one stream and checks on another
    meanwhile, the shadow having been written just before: the check sees the
    write, more checks than the context keeps events for go through, and the
    capture stands and replays."""
    from tests import util
    rng = np.random.default_rng(9)
    w, base = edge_world(rng, 100_000, np.array([100_000]))
    rec = W.make_records(np.full(64, 2), (base[0] + 7 * np.arange(64)).astype(np.uint64),
                         np.full(64, base[0] + 50_000, np.uint64), np.full(64, 300, np.uint64))
    o = util.oracle_for(w)
    o.vs[0][:40] = 0xFF
    want = o.run(rec)
    dw = H.DeviceWorld(w)
    try:
        side, other = torch.cuda.Stream(), torch.cuda.Stream()
        rt, out = H.records_tensor(rec), H.verdicts_tensor(64)
        pt = torch.zeros((64, 3), dtype=torch.int64, device="cuda")
        x = torch.zeros(1000, device="cuda")

        def check():
            if entry == "check_pointers":
                X.check_pointers(dw.ctx, rt.data_ptr(), 64, pt.data_ptr(), other.cuda_stream)
            else:
                getattr(X, entry)(dw.ctx, rt.data_ptr(), 64, out.data_ptr(), X.CG_CHECK, other.cuda_stream)
        check()
        torch.cuda.synchronize()
        X.shadow_set(dw.ctx, int(base[0]), 40, 0xFF)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side, capture_error_mode=mode):
            x += 1
            for _ in range(300):
                check()
            x += 1
        torch.cuda.synchronize()
        if entry != "check_pointers":
            util.assert_verdicts_equal(H.verdicts_np(out, 64), want)
        for k in range(3):
            g.replay()
            check()
            torch.cuda.synchronize()
            assert bool((x == 2 * (k + 1)).all())
    finally:
        dw.close()


@pytest.mark.parametrize("index", ["0", "2"])
@pytest.mark.parametrize("width,spitch,dpitch,rows", [
    (1, 16, 16, 300), (15, 16, 21, 300), (16, 17, 18, 300), (17, 19, 33, 300), (33, 50, 49, 130), (17, 32, 48, 200),
    (240, 256, 240, 70), (1000, 0, 1000, 40), (333, 160, 350, 90), (4032, 4096, 4099, 9), (4000, 4041, 4000, 9),
    (65_518, 65_536, 65_520, 4), (65_520, 65_601, 65_603, 3), (65_537, 65_552, 65_537, 3), (65_537, 65_555, 65_537, 3),
    (90, 1 << 20, 100, 4), (1500, 1 << 20, (1 << 20) + 5, 3), (1500, (1 << 20) + 9, 1500, 3)])
def test_pitched_rows_in_aligned_chunks(X, H, width, spitch, dpitch, rows, index, monkeypatch):
    """Checked rows whose windows are aligned chunks of their sources, at
    pitches that keep the 16-byte phase and others, from every kind of start up
    to the ends of the region and of the allocation, with clean and with dirty
    shadow; rows of 16 bytes and pitches of a megabyte beside them."""
    from tests import util
    from tests.test_gpu_2d import check2d
    monkeypatch.setenv("XC_SHADOW_INDEX", index)
    rng = np.random.default_rng(width + rows)
    s_span, d_span = (rows - 1) * spitch + width, (rows - 1) * dpitch + width
    span = max(s_span, d_span)
    sizes = np.array([span + 40, span + 40])
    for dens in (0.0, 0.002):
        w, base = edge_world(rng, span + 40, sizes, dens=dens)
        at = []
        for o in (0, 1, 7, 15, 24, 40):
            at += [(0, W.HOST_BASE + o + span - s_span, base[0] + 40 - o, spitch, dpitch),
                   (1, base[1] + o + span - s_span, W.HOST_BASE + 40 - o + span - d_span, spitch, dpitch),
                   (2, base[0] + o, base[1] + 40 - o, spitch, spitch)]
        rec = np.zeros(len(at), W.RECORD2D_DTYPE)
        for i, (kind, src, dst, sp, dp) in enumerate(at):
            rec[i]["kind"], rec[i]["src"], rec[i]["dst"], rec[i]["spitch"], rec[i]["dpitch"] = kind, src, dst, sp, dp
        rec["width"], rec["rows"] = width, rows
        want = util.oracle_for(w).run2d(rec)
        dw = H.DeviceWorld(w)
        try:
            util.assert_verdicts_equal(check2d(X, dw, rec, X.CG_CHECK), want, f"dirty share {dens}")
        finally:
            dw.close()


def test_strided_rows_scanned_like_close_ones(X, H, monkeypatch):
    """Rows of 4,032 bytes at 4,096, scanned without an index: one call takes
    less than 1.5 times that of rows of 4,096 bytes back to back, which read
    as much (about as long; twice as long with windows that start with the
    rows)."""
    import time
    from tests import util
    monkeypatch.setenv("XC_SHADOW_INDEX", "0")
    rng = np.random.default_rng(8)
    T, rows, pitch = 800, 640, 4096
    hl, base = 64 << 20, np.array([W.DEV_BASE + 4096])
    w = util.workload_from_arrays(W.HOST_BASE, np.zeros(hl, np.uint8), np.ones(hl, np.uint8), base, base * 0 + rows * pitch,
                                  [np.zeros(rows * pitch, np.uint8)], np.zeros(0, W.RECORD_DTYPE))
    rec = np.zeros(T, W.RECORD2D_DTYPE)
    rec["src"] = W.HOST_BASE + rng.integers(0, hl - rows * pitch, T)
    rec["dst"], rec["rows"], rec["spitch"], rec["dpitch"] = base[0], rows, pitch, pitch
    dw = H.DeviceWorld(w)
    try:
        s = torch.cuda.current_stream().cuda_stream
        out = H.verdicts_tensor(T)

        def us(width):
            rec["width"] = width
            rt = torch.from_numpy(rec.view(np.uint8).copy()).to("cuda:0")
            best = []
            for _ in range(12):
                torch.cuda.synchronize()
                t = time.perf_counter()
                X.check_transfers_2d(dw.ctx, rt.data_ptr(), T, out.data_ptr(), X.CG_CHECK, s)
                torch.cuda.synchronize()
                best.append((time.perf_counter() - t) * 1e6)
            assert (H.verdicts_np(out, T)["flags"] == 0).all()
            return min(best)
        close, strided = us(4096), us(4032)
        assert strided < 1.5 * close, f"back to back {close:.1f} us, strided {strided:.1f} us"
    finally:
        dw.close()

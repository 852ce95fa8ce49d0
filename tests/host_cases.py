"""Cases of test_host_paths_cpu.py, each run in a process of its own on the
HIP runtime in host memory (host_hip.py)."""
import ctypes as C
import struct

import numpy as np


def _part_sums(launch):
    """(first byte, bytes) of every region of partial sums that k_sum_parts reads."""
    raw = bytes(launch.arg)
    n_jobs = struct.unpack_from("<i", raw, 12 * 32)[0]
    out = []
    for k in range(n_jobs):
        src, _, rows, cols, stride, _ = struct.unpack_from("<QQiiii", raw, 32 * k)
        out.append((src, 4 * ((rows - 1) * stride + cols)))
    return out


def gradient_parts(hh, gsp):
    """The partial sums of every batch fit the buffer that any larger batch
    reserved (a training set's last batch is a short one)."""
    ctx = gsp.Context(0)
    top = 8192
    host = np.zeros(1 << 20, np.float32)
    loss = C.c_float()

    def call(net, n):
        hh.clear()
        rc = gsp.lib().gsp_cnn_gradients(net.h, 4096, 4096, n, host.ctypes.data_as(C.c_void_p), C.byref(loss), None)
        assert rc == gsp.GSP_OK, (n, rc)
        (sums,) = hh.launches("k_sum_parts")
        regions = _part_sums(sums)
        base = min(p for p, _ in regions)
        return base, max(p + b for p, b in regions) - base

    big = gsp.Cnn(ctx, seed=1)
    call(big, top)
    need = np.array([0] + [call(big, n)[1] for n in range(1, top + 1)])
    big.close()
    for r in (1, 171, 204, 205, 256, 384, 512, 1000, 2592, top):
        net = gsp.Cnn(ctx, seed=1)
        base, _ = call(net, r)
        room = hh.room(base)
        assert room >= need[:r + 1].max(), f"{r} images reserve {room} bytes, {need[:r + 1].argmax()} take {need[:r + 1].max()}"
        net.close()


# rows large enough for the pattern tile, and one for the other tile
STREAM_ROWS = [(0.0, 0.05, 400, 1), (20.0, 0.1, 330, 2), (53.0, 0.2, 300, 4), (113.0, 30.0, 3, 4)]
STREAM_TSAMP = 49.152e-6


def _stream_freqs(nchan):
    return 1400.0 + (np.arange(nchan) + 0.5) * 100.0 / nchan


def _pattern_tiles(hh):
    """(tiles listed, workgroups launched) of every pattern launch of the log."""
    return [(C.c_int64.from_address(struct.unpack_from("<Q", bytes(l.arg))[0]).value, l.grid[0])
            for l in hh.launches("k_dedisp_pat_jobs")]


def stream_graph_switched_on_and_off(hh, gsp):
    """The captured step holds a workgroup for every pattern tile, also where
    the tiles grew in steps that were launched without the graph."""
    ctx = gsp.Context(0)
    nchan, block = 1024, 2064
    s = gsp.Stream(ctx, 1 << 34, block, [1, 2, 4], 50.0)
    bid, ok = s.open_beam(nchan, _stream_freqs(nchan), STREAM_TSAMP, STREAM_ROWS)
    assert ok
    data = np.zeros((block, nchan), np.uint8)
    seen = []
    for k, graph in enumerate([True, False, False, True, True]):
        s.set_graph(graph)
        s.push(bid, data)
        hh.clear()
        assert s.step() == 1
        tiles = _pattern_tiles(hh)
        print(k, graph, tiles)
        assert all(l.replayed == int(graph) for l in hh.launches("k_dedisp_pat_jobs"))
        assert all(n <= grid for n, grid in tiles), (k, tiles)
        seen.append(sorted(n for n, _ in tiles if n))
    assert seen[1] and all(n == seen[1] for n in seen[1:]), seen  # full windows: the same tiles every step
    assert seen[0] != seen[1]  # the first window is a shorter one
    s.close()


def forced_shape_after_default(hh, gsp, how):
    """A shape that is asked for is built (or refused) also where the row's
    default asked for the same one and settled for another."""
    freqs = 1000.0 + (np.arange(64) + 0.5) * 500.0 / 64
    desc = gsp.plan_shape(20000, freqs, 1e-4, [(0.0, 1.0, 40, 1), (0.0, 1.0, 40, 2)])
    wide = np.linspace(300.0, 1500.0, 64)  # a group's patterns do not fit the LDS
    far = gsp.plan_shape(1 << 20, wide, 1e-4, [(0.0, 1.0, 96, 1)])
    for plan, f, rows in ((desc, freqs, [(0, 12), (1, 8)]), (far, wide, [(0, 12)])):
        for r, tpw in rows:
            fresh = gsp.Context(0)  # what the shape gives without a default before it
            try:
                fresh.set_row_shape(f, plan, r, 4, tpw, 8, 16, 4)
                want = fresh.row_shape(f, plan, r)
            except gsp.GspError as e:
                assert e.status == gsp.GSP_EINVAL
                want = None
            ctx = gsp.Context(0)
            before = ctx.row_shape(f, plan, r)
            assert before[4] != 4, before
            got = None
            try:
                if how == "set":
                    ctx.set_row_shape(f, plan, r, 4, tpw, 8, 16, 4)
                else:
                    fresh_file = f"{how}/{r}"
                    donor = gsp.Context(0)
                    try:
                        donor.set_row_shape(f, plan, r, 4, tpw, 8, 16, 4)
                    except gsp.GspError:
                        continue
                    donor.tuning_save(fresh_file)
                    ctx.tuning_load(fresh_file)
                got = ctx.row_shape(f, plan, r)
            except gsp.GspError as e:
                assert e.status == gsp.GSP_EINVAL
            print(r, before, "->", got, "wanted", want)
            assert got == want
            if want is None:  # refused: the default stands
                assert ctx.row_shape(f, plan, r) == before


def _least_budget(gsp, ctx, nchan, block, rows):
    """Smallest budget a beam is accepted under: what the beam itself takes."""
    lo, hi = 1, 1 << 34
    while lo < hi:
        mid = (lo + hi) // 2
        s = gsp.Stream(ctx, mid, block, [1, 2, 4], 50.0)
        try:
            s.open_beam(nchan, _stream_freqs(nchan), STREAM_TSAMP, rows)
            hi = mid
        except gsp.GspError as e:
            assert e.status == gsp.GSP_ENOMEM
            lo = mid + 1
        s.close()
    return lo


# job tables and search scratch that a stream holds beside its beams
STREAM_FIXED = 8 << 20


def stream_budget(hh, gsp):
    """Linear copies and pattern tables are held in what the beams leave of
    the budget, and given up for a beam that fits without them."""
    ctx = gsp.Context(0)
    nchan, block = 1024, 2064
    one = _least_budget(gsp, ctx, nchan, block, STREAM_ROWS)
    freqs = _stream_freqs(nchan)
    data = np.zeros((block, nchan), np.uint8)

    def steps(s, ids, n=3):
        hh.clear()
        for _ in range(n):
            for b in ids:
                s.push(b, data)
            assert s.step() == len(ids)
        return sum(n for n, _ in _pattern_tiles(hh))

    for beams, spare, pattern in ((1, 0, False), (1, 64 << 20, True), (3, 64 << 20, True), (2, 0, False)):
        base = hh.used()
        s = gsp.Stream(ctx, beams * one + spare, block, [1, 2, 4], 50.0)
        ids = []
        for k in range(beams):
            bid, ok = s.open_beam(nchan, freqs, STREAM_TSAMP, STREAM_ROWS)
            assert ok, (beams, k)
            ids.append(bid)
            tiles = steps(s, ids)
            rep = s.report()
            print(f"{k + 1} of {beams} beams, {spare} bytes to spare: {tiles} pattern tiles, {rep['mem_used']} held")
            assert rep["mem_used"] <= rep["mem_budget"]
            assert hh.used() - base <= rep["mem_used"] + STREAM_FIXED
            if k + 1 < beams:
                assert tiles > 0  # the room of the beams to come
        assert (tiles > 0) == pattern
        assert not s.open_beam(nchan, freqs, STREAM_TSAMP, STREAM_ROWS)[1] or spare >= one
        for b in ids:
            s.close_beam(b)
        s.close()
        assert hh.used() - base <= STREAM_FIXED


def stream_budget_with_worker(hh, gsp):
    """The same while a worker thread steps: openings wait for its steps."""
    ctx = gsp.Context(0)
    nchan, block = 1024, 2064
    one = _least_budget(gsp, ctx, nchan, block, STREAM_ROWS)
    s = gsp.Stream(ctx, 3 * one + (1 << 20), block, [1, 2, 4], 50.0)
    data = np.zeros((block, nchan), np.uint8)
    s.start()
    live = []
    for k in range(40):
        if len(live) == 3:
            s.close_beam(live.pop(0))
        bid, ok = s.open_beam(nchan, _stream_freqs(nchan), STREAM_TSAMP, STREAM_ROWS)
        live.append(bid)
        for b in live:
            for _ in range(3):
                s.push(b, data)
        rep = s.report()
        assert rep["mem_used"] <= rep["mem_budget"], (k, rep)
    s.flush()
    s.stop()
    rep = s.report()
    print(rep)
    assert rep["beams_queued"] == 0 and rep["blocks_pending"] == 0 and rep["mem_used"] <= rep["mem_budget"]
    s.close()


def stream_without_room_for_tables(hh, gsp):
    """A beam whose pattern tables get no device memory runs on the other tile."""
    ctx = gsp.Context(0)
    nchan, block = 1024, 2064
    freqs = _stream_freqs(nchan)
    one = _least_budget(gsp, ctx, nchan, block, STREAM_ROWS)
    s = gsp.Stream(ctx, 1 << 34, block, [1, 2, 4], 50.0)
    hh.limit(hh.used() + one + (256 << 10))  # the beam, and a part of the tables
    bid, ok = s.open_beam(nchan, freqs, STREAM_TSAMP, STREAM_ROWS)
    assert ok
    hh.clear()
    for _ in range(3):
        s.push(bid, np.zeros((block, nchan), np.uint8))
        assert s.step() == 1
    assert not _pattern_tiles(hh) and hh.launches("k_dedisp_jobs")
    s.close()


def row_tables_without_room(hh, gsp):
    """A default row shape whose tables get no device memory gives way to one
    with smaller tables; a shape that was asked for is refused."""
    freqs = 1000.0 + (np.arange(1024) + 0.5) * 500.0 / 1024
    for row, room, kind in (((0.0, 0.1, 400, 1), 500000, 2), ((100.0, 0.4, 400, 2), 1800000, 0)):
        desc = gsp.plan_shape(1 << 19, freqs, 49.152e-6, [row])
        ctx = gsp.Context(0)
        assert ctx.row_shape(freqs, desc, 0)[4] == 4
        ctx = gsp.Context(0)
        hh.limit(hh.used() + room)
        shape = ctx.row_shape(freqs, desc, 0)
        print(row, "with", room, "bytes:", shape)
        assert shape[4] == kind
        other = gsp.Context(0)
        try:
            other.set_row_shape(freqs, desc, 0, 4, 8, 8, 16, 4)
            assert False
        except gsp.GspError as e:
            assert e.status == gsp.GSP_ENOMEM
        hh.limit(1 << 36)


def rfi_without_room_for_sums(hh, gsp):
    """Mitigation that gets no memory for its split channel sums runs without them."""
    nsamp, nchan, block = 8256, 4096, 129
    fb, out = hh.malloc(nsamp * nchan), hh.malloc(nsamp * nchan)
    n = C.c_int64()
    for room, split in ((1 << 24, True), (600 << 10, False)):
        ctx = gsp.Context(0)
        hh.limit(hh.used() + room)
        hh.clear()
        rc = gsp.lib().gsp_rfi_clean(ctx.h, fb, nsamp, nchan, 3.0, block, 1, out, C.byref(n), None)
        assert rc == gsp.GSP_OK, rc
        assert len(hh.launches("k_rfi_means")) == 1 and bool(hh.launches("k_rfi_sums")) == split
        hh.limit(1 << 36)


def network_after_a_batch_without_room(hh, gsp):
    """A batch whose buffers got no memory leaves the network usable."""
    ctx = gsp.Context(0)
    net = gsp.Cnn(ctx, seed=1)
    logits = np.zeros(4096, np.float32)
    x = hh.malloc(1 << 20)

    def forward(n):
        return gsp.lib().gsp_cnn_forward(net.h, x, n, logits.ctypes.data_as(C.c_void_p), None)

    assert forward(64) == gsp.GSP_OK
    held = hh.used()
    hh.limit(held + (64 << 20))
    assert forward(4096) == gsp.GSP_ENOMEM
    hh.limit(1 << 36)
    try:  # the activations of the batch before are gone with their buffers
        net.activation(0, 64)
        assert False
    except gsp.GspError as e:
        assert e.status == gsp.GSP_EINVAL
    assert forward(64) == gsp.GSP_OK
    print(held, hh.used())
    assert hh.used() >= held  # every buffer is there again
    for l in hh.launches("k_conv_pool"):
        assert hh.room(struct.unpack_from("<Q", bytes(l.arg))[0]) > 0


def stream_rows_of_one_round(hh, gsp):
    """Rows of at most a tile to a CU: the estimate that the pattern tile is
    compared with is that of the streaming kernel (8 waves a workgroup), which
    takes longer there than the batch kernel's form for so few tiles."""
    ctx = gsp.Context(0)
    nchan, block = 256, 8192
    s = gsp.Stream(ctx, 1 << 34, block, [1, 2, 4], 50.0)
    bid, ok = s.open_beam(nchan, _stream_freqs(nchan), STREAM_TSAMP, STREAM_ROWS)
    assert ok
    hh.clear()
    for _ in range(3):
        s.push(bid, np.zeros((block, nchan), np.uint8))
        s.step()
    print(_pattern_tiles(hh))
    assert sum(n for n, _ in _pattern_tiles(hh)) > 0
    s.close()

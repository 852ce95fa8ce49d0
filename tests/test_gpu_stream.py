"""Streaming engine: block-by-block results equal the oracle's window
semantics, a beam's results are the same alone and in a mix of beams,
admission by memory queues and later admits beams, snapshot/restore
continues bit-identically, graph replay equals direct launches."""
import numpy as np
import pytest

import oracle
from paper_2110_12749_amd import synth
from tests._util import match_candidates, oracle_cands_with_seg, say

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 4, 8, 16, 32]
THR = 6.0
BLOCK = 512


def beam_workload(k, nchan=64, nsamp=3000, segs=None):
    if segs is None:
        segs = [(0.0, 1.0, 40, 1), (40.0, 2.0, 13, 2)]
    w = synth.small(nchan=nchan, nsamp=nsamp, segments=segs, n_pulses=2, seed_offset=10 + k, widths=WIDTHS)
    return w


def windows_of(w):
    """Per block k and row r: (a, b) output window."""
    max_delay, _ = oracle.plan_shape(w.nsamp, w.freqs, w.tsamp, w.segments)
    nblk = (w.nsamp + BLOCK - 1) // BLOCK
    out = []
    for k in range(nblk):
        rows = []
        for r, seg in enumerate(w.segments):
            D = seg[3]
            M = int(max_delay[r])
            N0 = (k * BLOCK) // D
            N1 = N0 + min(BLOCK, w.nsamp - k * BLOCK) // D
            rows.append((max(0, N0 - M), max(0, N1 - M)))
        out.append(rows)
    return out


def oracle_window_cands(full, w, r, a, b):
    rows = []
    for i in range(full.shape[0]):
        c = oracle.search_window(full[i], a, b, WIDTHS, THR, trial=i)
        if len(c):
            rows.append(c)
    c = np.concatenate(rows) if rows else np.zeros(0, oracle.CAND_DTYPE)
    return oracle_cands_with_seg([(r, c)])


@pytest.fixture(scope="module")
def env(dev):
    import torch
    from paper_2110_12749_amd import gsp
    ctx = gsp.Context(0)
    yield gsp, ctx, torch
    torch.cuda.synchronize()
    ctx.close()


def run_beams(env, beams, interleave=True, graph=True, budget=1 << 34, check_windows=None, frag_cap=None):
    """Push every beam's blocks (round robin) and step; returns per-beam candidates."""
    gsp, ctx, torch = env
    s = gsp.Stream(ctx, budget, BLOCK, WIDTHS, THR)
    s.set_graph(graph)
    if frag_cap is not None:
        s.set_fragment_capacity(frag_cap)
    ids = []
    for w, X in beams:
        bid, ok = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
        ids.append(bid)
    nblk = max((w.nsamp + BLOCK - 1) // BLOCK for w, _ in beams)
    for k in range(nblk):
        for (w, X), bid in zip(beams, ids):
            if k * BLOCK < w.nsamp:
                s.push(bid, X[k * BLOCK: (k + 1) * BLOCK])
        while s.step():
            if check_windows:
                check_windows(s, ids, k)
            break
    s.flush()
    cands = s.poll()
    rep = s.report()
    s.close()
    return ids, cands, rep


# 64 channels: one channel tile staged 16 channels per thread; 40: not a
# multiple of 16, staged one channel per thread; 160: two channel tiles, the
# second partly empty, and a D = 4 row
SINGLE = [dict(nchan=64), dict(nchan=40), dict(nchan=160, segs=[(0.0, 1.0, 40, 1), (40.0, 2.0, 13, 2),
                                                                   (66.0, 4.0, 8, 4)])]


@pytest.mark.parametrize("cfg", SINGLE, ids=lambda c: f"nchan{c['nchan']}")
def test_single_beam_windows_and_candidates_match_oracle(env, cfg):
    gsp, ctx, torch = env
    w = beam_workload(0, nsamp=3000, **cfg)
    X = w.generate()
    full = oracle.dedisperse(X, w.freqs, w.tsamp, w.segments)
    wins = windows_of(w)
    say(f"[case] single beam, {cfg}, windows {wins}")
    seen = []

    def check(s, ids, k):
        if k == len(wins) - 1:
            return  # the beam ended with this block and is gone (its candidates are checked below)
        for r, seg in enumerate(w.segments):
            t0, arr = s.window(ids[0], r, seg[2])
            a, b = wins[k][r]
            assert (t0, arr.shape[1]) == (a, b - a), (k, r)
            assert (arr == full[r][:, a:b]).all(), (k, r)
            seen.append((k, r, b - a))

    ids, cands, rep = run_beams(env, [(w, X)], check_windows=check)
    assert any(n == 0 for _, _, n in seen) and any(n > 0 for _, _, n in seen)
    # candidates window by window
    for k, rows in enumerate(wins):
        for r, (a, b) in enumerate(rows):
            co = oracle_window_cands(full[r], w, r, a, b)
            cg = cands[(cands["block"] == k) & (cands["seg"] == r)]
            match_candidates(cg, co, THR)
    assert rep["blocks"] == len(wins)


@pytest.mark.parametrize("graph", [True, False])
def test_fragment_overflow_searches_again_and_loses_nothing(env, graph):
    """A step whose search finds more run fragments than the stream's buffer
    holds grows the buffer and searches the same windows again: with a
    capacity of 3 fragments, the candidates still equal the oracle's window
    by window, and the report counts the repeated search."""
    gsp, ctx, torch = env
    w = beam_workload(0, nsamp=3000)
    X = w.generate()
    full = oracle.dedisperse(X, w.freqs, w.tsamp, w.segments)
    wins = windows_of(w)
    say(f"[case] fragment capacity 3, graph {graph}")
    ids, cands, rep = run_beams(env, [(w, X)], graph=graph, frag_cap=3)
    say(f"  {len(cands)} candidates, {rep['search_repeats']} repeated searches of {rep['steps']} steps")
    assert rep["blocks"] == len(wins)
    for k, rows in enumerate(wins):
        for r, (a, b) in enumerate(rows):
            co = oracle_window_cands(full[r], w, r, a, b)
            cg = cands[(cands["block"] == k) & (cands["seg"] == r)]
            match_candidates(cg, co, THR)
    assert rep["search_repeats"] >= 1  # the grown buffer then holds every later step's fragments


def test_mix_equals_alone_and_oracle(env):
    gsp, ctx, torch = env
    cfgs = [dict(nchan=64, nsamp=2900), dict(nchan=96, nsamp=1800, segs=[(0.0, 0.5, 37, 1)]),
            dict(nchan=48, nsamp=3700, segs=[(10.0, 1.5, 21, 2), (41.5, 3.0, 9, 4)]), dict(nchan=64, nsamp=700)]
    beams = []
    for k, c in enumerate(cfgs):
        w = beam_workload(k + 1, **c)
        beams.append((w, w.generate()))
    _, mix, rep = run_beams(env, beams)
    say(f"  mix: {len(mix)} candidates, report {rep}")
    for j, (w, X) in enumerate(beams):
        _, alone, _ = run_beams(env, [(w, X)])
        m = mix[mix["beam"] == j]
        key = ["block", "seg", "dm_index", "t_first", "t_last", "t_peak", "width"]
        a_sorted = np.sort(alone[key])
        m_sorted = np.sort(m[key])
        assert len(a_sorted) == len(m_sorted) and (a_sorted == m_sorted).all(), j
        assert np.allclose(np.sort(alone["snr"]), np.sort(m["snr"]), rtol=0, atol=0)
        # and against the oracle, window by window (a row shorter than its
        # maximum delay has only empty windows)
        _, n_out = oracle.plan_shape(w.nsamp, w.freqs, w.tsamp, w.segments)
        full = [oracle.dedisperse_segment(X, w.freqs, w.tsamp, seg) if n_out[r] > 0 else None
                for r, seg in enumerate(w.segments)]
        for k, rows in enumerate(windows_of(w)):
            for r, (a, b) in enumerate(rows):
                if n_out[r] <= 0:
                    assert b == a == 0
                    assert not ((m["block"] == k) & (m["seg"] == r)).any()
                    continue
                co = oracle_window_cands(full[r], w, r, a, b)
                match_candidates(m[(m["block"] == k) & (m["seg"] == r)], co, THR)


def test_graph_replay_equals_direct_launch(env):
    w = beam_workload(7, nsamp=2600)
    X = w.generate()
    _, c1, _ = run_beams(env, [(w, X)], graph=True)
    _, c2, _ = run_beams(env, [(w, X)], graph=False)
    key = ["block", "seg", "dm_index", "t_first", "t_last", "t_peak", "width", "snr"]
    assert len(c1) == len(c2) and (np.sort(c1[key]) == np.sort(c2[key])).all()


def test_admission_queues_and_admits_later(env):
    gsp, ctx, torch = env
    w0 = beam_workload(11, nsamp=1100)
    w1 = beam_workload(12, nsamp=1600)
    w2 = beam_workload(13, nsamp=1500)
    s0 = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    # measure one beam's footprint, then budget for two
    bid, _ = s0.open_beam(w0.nchan, w0.freqs, w0.tsamp, w0.segments)
    one = s0.report()["mem_used"]
    s0.close()
    s = gsp.Stream(ctx, 2 * one + one // 2, BLOCK, WIDTHS, THR)
    ids = [s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments) for w in (w0, w1, w2)]
    assert [ok for _, ok in ids] == [True, True, False]
    X = [w.generate() for w in (w0, w1, w2)]
    for k in range(4):
        for j, w in enumerate((w0, w1, w2)):
            if k * BLOCK < w.nsamp:
                s.push(ids[j][0], X[j][k * BLOCK:(k + 1) * BLOCK])
        s.step()
    assert s.report()["beams_queued"] == 0  # beam 0 ended -> beam 2 admitted
    s.flush()
    mix = s.poll()
    s.close()
    _, alone, _ = run_beams(env, [(w2, X[2])])
    m = mix[mix["beam"] == ids[2][0]]
    assert len(m) == len(alone)
    assert (np.sort(m[["block", "seg", "dm_index", "t_peak", "width"]]) ==
            np.sort(alone[["block", "seg", "dm_index", "t_peak", "width"]])).all()


def test_snapshot_restore_continues_identically(env):
    gsp, ctx, torch = env
    w = beam_workload(21, nsamp=3300)
    X = w.generate()
    _, ref, _ = run_beams(env, [(w, X)])
    s = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    bid, _ = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    for k in range(3):
        s.push(bid, X[k * BLOCK:(k + 1) * BLOCK])
        s.step()
    first = s.poll()
    snap = s.snapshot(bid)
    s.close()
    s2 = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    bid2, _ = s2.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    s2.restore(bid2, snap)
    for k in range(3, (w.nsamp + BLOCK - 1) // BLOCK):
        s2.push(bid2, X[k * BLOCK:(k + 1) * BLOCK])
        s2.step()
    rest = s2.poll()
    s2.close()
    got = np.concatenate([first, rest])
    key = ["block", "seg", "dm_index", "t_first", "t_last", "t_peak", "width"]
    assert len(got) == len(ref) and (np.sort(got[key]) == np.sort(ref[key])).all()


def test_worker_thread_and_latency_report(env):
    gsp, ctx, torch = env
    w = beam_workload(31, nsamp=2500)
    X = w.generate()
    _, ref, _ = run_beams(env, [(w, X)])
    s = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    bid, _ = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    s.start()
    for k in range((w.nsamp + BLOCK - 1) // BLOCK):
        s.push(bid, X[k * BLOCK:(k + 1) * BLOCK])
    s.flush()
    s.stop()
    got = s.poll()
    rep = s.report()
    s.close()
    assert rep["blocks"] == (w.nsamp + BLOCK - 1) // BLOCK
    assert 0 < rep["lat_p50_s"] <= rep["lat_p99_s"] <= rep["lat_max_s"]
    key = ["block", "seg", "dm_index", "t_first", "t_last", "t_peak", "width"]
    assert (np.sort(got[key]) == np.sort(ref[key])).all()


def test_triage_scores_are_the_network_on_oracle_cutouts(env):
    """With a network attached, every streamed candidate carries the logit of
    the network on its cutout, and that cutout is the oracle's (DM-time series
    from the window, padding at the window's mean; frequency-time from the
    downsampled input): scoring the oracle's cutouts with the same network
    gives the same logits."""
    from oracle import cnn as ocnn
    gsp, ctx, torch = env
    w = beam_workload(41, nsamp=2600)
    X = w.generate()
    net = gsp.Cnn(ctx, seed=9)
    s = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    s.set_triage(net, -1e30)  # score everything, reject nothing
    bid, _ = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    for k in range((w.nsamp + BLOCK - 1) // BLOCK):
        s.push(bid, X[k * BLOCK:(k + 1) * BLOCK])
        s.step()
    got = s.poll()
    rep = s.report()
    s.close()
    assert len(got) > 0 and np.isfinite(got["score"]).all()
    assert rep["triage_scored"] == len(got) and rep["triage_rejected"] == 0
    full = oracle.dedisperse(X, w.freqs, w.tsamp, w.segments)
    wins = windows_of(w)
    imgs = []
    for c in got:
        r = int(c["seg"])
        seg = w.segments[r]
        a, b = wins[int(c["block"])][r]
        mu = np.array([oracle.stats(full[r][i, a:b])[0] for i in range(seg[2])])
        Y = oracle.downsample(X, seg[3])
        delays = oracle.delay_table(w.freqs, w.tsamp, seg)
        imgs.append(ocnn.bf16_bits(ocnn.cutout(full[r], mu, Y, delays, (c["dm_index"], c["t_peak"], c["width"]))))
    x = torch.from_numpy(np.stack(imgs).view(np.int16)).cuda()
    z = net.forward(x).cpu().numpy()
    say(f"  {len(got)} streamed candidates scored; max |logit difference| {np.abs(z - got['score']).max():.2e}")
    assert np.allclose(z, got["score"], rtol=1e-3, atol=1e-3)
    net.close()


def test_triage_threshold_filters_and_detaches(env):
    gsp, ctx, torch = env
    w = beam_workload(42, nsamp=1600)
    X = w.generate()
    _, plain, _ = run_beams(env, [(w, X)])
    assert np.isnan(plain["score"]).all()
    net = gsp.Cnn(ctx, seed=10)
    s = gsp.Stream(ctx, 1 << 34, BLOCK, WIDTHS, THR)
    s.set_triage(net, 1e30)  # reject everything
    bid, _ = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    for k in range((w.nsamp + BLOCK - 1) // BLOCK):
        s.push(bid, X[k * BLOCK:(k + 1) * BLOCK])
        s.step()
    got = s.poll()
    rep = s.report()
    s.close()
    assert len(got) == 0 and rep["triage_rejected"] == rep["triage_scored"] == len(plain)
    net.close()


def test_full_shape_windows_equal_batch_and_oracle(env):
    """One beam of the streaming workload's shape (4096 channels over
    1000-1500 MHz, tsamp 49.152 us, blocks of 20480 samples; the ladder's
    four rows D = 1, 2, 4, 8 cut to 100-200 trials each), every block pushed
    before the first step so that each step's next block is copied during the
    step: after every step each row's window equals the batch dedispersion of
    the whole beam over the same outputs, bit for bit, and 40 sampled outputs
    per window equal the oracle's."""
    gsp, ctx, torch = env
    B = 20480
    segs = [(0.0, 0.1, 200, 1), (150.0, 0.3, 100, 2), (450.0, 1.0, 100, 4), (1200.0, 3.0, 100, 8)]
    # trials whose streamed candidates are compared with the oracle's window
    # search over the oracle's own dedispersed series: the first, the last
    # and two inside each row
    cand_trials = [[0, 57, 131, 199], [0, 37, 74, 99], [0, 37, 74, 99], [0, 37, 74, 99]]
    w = synth.Workload("stream-shape", 4096, 1000.0, 1500.0, 49.152e-6, 8 * B, segs, synth.WIDTHS_512, 6.0,
                       synth.BASE_SEED + 7)
    say("[case] full-shape stream beam: generate")
    X = w.generate()
    desc = gsp.plan_shape(w.nsamp, w.freqs, w.tsamp, w.segments)
    dmt = ctx.dedisperse(torch.from_numpy(X).to("cuda"), w.freqs, desc)
    views = gsp.segment_views(desc, dmt)
    max_delay, n_out = oracle.plan_shape(w.nsamp, w.freqs, w.tsamp, w.segments)
    s = gsp.Stream(ctx, 1 << 34, B, synth.WIDTHS_512, 6.0)
    bid, ok = s.open_beam(w.nchan, w.freqs, w.tsamp, w.segments)
    assert ok
    for k in range(w.nsamp // B):
        s.push(bid, X[k * B:(k + 1) * B])
    rng = np.random.default_rng(3)
    checked = 0
    streamed = []
    for k in range(w.nsamp // B):
        assert s.step() == 1
        streamed.append(s.poll())
        for r, seg in enumerate(segs):
            D, M = seg[3], int(max_delay[r])
            a, b = max(0, k * B // D - M), max(0, (k + 1) * B // D - M)
            t0, arr = s.window(bid, r, seg[2])
            assert (t0, arr.shape[1]) == (a, b - a), (k, r)
            if b == a:
                continue
            ref = views[r][:, a:b].cpu().numpy()
            assert (arr == ref).all(), (k, r)
            tr = rng.integers(0, seg[2], 40)
            tt = rng.integers(a, b, 40)
            pts = oracle.dedisperse_points(X, w.freqs, w.tsamp, seg, tr, tt)
            assert (arr[tr, tt - a].astype(np.int64) == pts).all(), (k, r)
            checked += b - a
        say(f"  step {k}: windows checked")
    assert checked == int(sum(n_out))  # every output of every row, once
    s.close()
    cands = np.concatenate(streamed)
    n_cmp = 0
    for r, seg in enumerate(segs):
        D, M = seg[3], int(max_delay[r])
        trials = cand_trials[r]
        for i in trials:
            series = oracle.dedisperse_segment(X, w.freqs, w.tsamp, seg, trials=(i, i + 1))[0]
            for k in range(w.nsamp // B):
                a, b = max(0, k * B // D - M), max(0, (k + 1) * B // D - M)
                if b == a:
                    continue
                co = oracle.search_window(series, a, b, synth.WIDTHS_512, 6.0, trial=i)
                co = oracle_cands_with_seg([(r, co)])
                sel = (cands["block"] == k) & (cands["seg"] == r) & (cands["dm_index"] == i)
                match_candidates(cands[sel], co, 6.0)
                n_cmp += len(co)
    say(f"  streamed candidates of {sum(map(len, cand_trials))} trials match the oracle ({n_cmp} oracle runs)")
    del dmt
    torch.cuda.empty_cache()


@pytest.mark.parametrize("nchan,block,graph", [(256, 8192, True), (203, 4112, False), (1024, 2064, True)])
def test_pattern_rows_equal_batch(env, nchan, block, graph):
    """Rows large enough for the pattern tile (copied out of their rings, which
    these lengths wrap at many offsets), two beams in a mix, and rows of the
    other tile beside them: every window equals the batch dedispersion on the
    16-bit tile; the first windows are short, and the last block is."""
    gsp, ctx, torch = env
    segs = [(0.0, 0.05, 400, 1), (20.0, 0.1, 330, 2), (53.0, 0.2, 300, 4), (113.0, 30.0, 3, 4)]
    freqs = 1400.0 + (np.arange(nchan) + 0.5) * 100.0 / nchan
    ts = 49.152e-6
    n_blk, last = 7, block // 2
    nsamp = (n_blk - 1) * block + last
    rng = np.random.default_rng(nchan)
    X = [rng.integers(0, 256, (nsamp, nchan), dtype=np.uint8) for _ in range(2)]
    X[1][:] = 255
    desc = gsp.plan_shape(nsamp, freqs, ts, segs)
    ref = []
    for x in X:
        c = gsp.Context(0)
        for r in range(len(segs)):
            c.set_row_shape(freqs, desc, r, 4, 4, 8, 32, 0)
        v = gsp.segment_views(desc, c.dedisperse(torch.from_numpy(x).cuda(), freqs, desc))
        ref.append([t.cpu().numpy() for t in v])
        c.close()
    s = gsp.Stream(ctx, 1 << 34, block, WIDTHS, 50.0)
    s.set_graph(graph)
    ids = [s.open_beam(nchan, freqs, ts, segs)[0] for _ in X]
    say(f"[case] stream pattern rows, {nchan} channels, blocks of {block}")
    checked = 0
    for k in range(n_blk - 1):
        for bid, x in zip(ids, X):
            s.push(bid, x[k * block:(k + 1) * block])
        assert s.step() == 2
        for bid, full in zip(ids, ref):
            for r, seg in enumerate(segs):
                M = nsamp // seg[3] - int(desc.n_out[r])
                a, b = max(0, k * block // seg[3] - M), max(0, (k + 1) * block // seg[3] - M)
                t0, arr = s.window(bid, r, seg[2])
                assert (t0, arr.shape[1]) == (a, b - a), (k, r)
                assert np.array_equal(arr, full[r][:, a:b]), (k, r)
                checked += b - a
    assert checked > 0
    s.push(ids[0], X[0][(n_blk - 1) * block:])  # a short last block: the beam ends
    assert s.step() == 1
    s.close()


def test_pattern_rows_with_the_graph_switched_on_and_off(env):
    """Windows grow while the step graph is off: switched on again, its replays
    compute every tile (each window against the batch dedispersion)."""
    gsp, ctx, torch = env
    nchan, block = 1024, 2064
    segs = [(0.0, 0.05, 400, 1), (20.0, 0.1, 330, 2), (53.0, 0.2, 300, 4)]
    freqs = 1400.0 + (np.arange(nchan) + 0.5) * 100.0 / nchan
    ts = 49.152e-6
    graphs = [True, False, False, True, True, False, True]
    nsamp = len(graphs) * block
    X = np.random.default_rng(5).integers(0, 256, (nsamp, nchan), dtype=np.uint8)
    desc = gsp.plan_shape(nsamp, freqs, ts, segs)
    c = gsp.Context(0)
    for r in range(len(segs)):
        c.set_row_shape(freqs, desc, r, 4, 4, 8, 32, 0)
    ref = [v.cpu().numpy() for v in gsp.segment_views(desc, c.dedisperse(torch.from_numpy(X).cuda(), freqs, desc))]
    c.close()
    s = gsp.Stream(ctx, 1 << 34, block, WIDTHS, 50.0)
    bid, ok = s.open_beam(nchan, freqs, ts, segs)
    assert ok
    say("[case] stream graph switched on and off")
    checked = 0
    for k, graph in enumerate(graphs):
        s.set_graph(graph)
        s.push(bid, X[k * block:(k + 1) * block])
        assert s.step() == 1
        for r, seg in enumerate(segs):
            M = nsamp // seg[3] - int(desc.n_out[r])
            a, b = max(0, k * block // seg[3] - M), max(0, (k + 1) * block // seg[3] - M)
            t0, arr = s.window(bid, r, seg[2])
            assert (t0, arr.shape[1]) == (a, b - a), (k, r)
            assert np.array_equal(arr, ref[r][:, a:b]), (k, r)
            checked += b - a
    assert checked == int(sum(desc.n_out[r] for r in range(len(segs))))
    s.close()

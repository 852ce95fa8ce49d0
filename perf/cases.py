"""Performance cases of the library: what a user's program calls, over the
range of sizes it calls it at.

A case is a dict of plain values with an "op":

  dedisperse     brute-force dedispersion of one beam over a DDplan-style plan
  subband        the two-stage dedispersion over the same kind of plan
  search         boxcar search of a dedispersed plan
  rfi            clip and zero-DM filter of a filterbank
  pipeline       one whole step of a beam: dedispersion, search, grouping,
                 cutouts of every event, network scores
  stream         one step of a streaming engine: a block per beam pushed,
                 processed and its candidates drained
  cnn_forward    network scores of a batch of cutouts
  cnn_gradients  loss and gradients of a training batch

Bands, sampling times, DM ladders, width sets and batch sizes are those of
this repository's synthetic workloads, tests and benchmark.
"""
import math

import numpy as np
import torch

from paper_2110_12749_amd import gsp

K_DM = 4148.808
LADDER = "0:0.1:1500:1;150:0.3:1000:2;450:1:750:4;1200:3:600:8"
LADDER_1500 = "0:0.1:1500:1;150:0.3:1000:2;450:1:750:4;1200:3:100:8"
WIDTHS_512 = "1,2,4,8,16,32,64,128,256,512"
WIDTHS_32 = "1,2,4,8,16,32"
BAND = {"f_lo": 1000.0, "f_hi": 1500.0, "tsamp": 49.152e-6}


def listed():
    return [
        # the smallest call: a quick look at 3 s of a coarse filterbank, where launches and latency count
        {"name": "dedisperse_tiny", "op": "dedisperse", "nchan": 128, "nsamp": 16384, "f_lo": 1000.0,
         "f_hi": 1500.0, "tsamp": 196.608e-6, "plan": "0:1:200:1", "pulses": 1},
        # a survey beam: 51.5 s of 4096 channels, the full DM ladder with every downsampling
        {"name": "dedisperse_survey", "op": "dedisperse", "nchan": 4096, "nsamp": 1 << 20, **BAND, "plan": LADDER,
         "pulses": 20},
        # a very wide low-frequency band, where delays spread most
        {"name": "dedisperse_wideband", "op": "dedisperse", "nchan": 4096, "nsamp": 1 << 19, "f_lo": 270.0,
         "f_hi": 1620.0, "tsamp": 196.608e-6, "plan": LADDER_1500, "pulses": 20},
        # sizes that are a multiple of nothing: odd channel and sample counts, a downsampling of 3
        {"name": "dedisperse_ragged", "op": "dedisperse", "nchan": 1023, "nsamp": 200003, "f_lo": 1200.0,
         "f_hi": 1600.0, "tsamp": 64e-6, "plan": "0:0.37:301:1;111.37:1.1:203:3", "pulses": 4},
        # the survey beam with the approximate two-stage algorithm
        {"name": "subband_survey", "op": "subband", "nchan": 4096, "nsamp": 1 << 19, **BAND, "plan": LADDER,
         "n_sub": "32,32,64,128", "group": "24,32,24,19", "pulses": 10},
        # search of a quick look
        {"name": "search_tiny", "op": "search", "nchan": 128, "nsamp": 16384, "f_lo": 1000.0, "f_hi": 1500.0,
         "tsamp": 196.608e-6, "plan": "0:1:200:1", "widths": WIDTHS_32, "threshold": 6.0, "pulses": 2, "room": 256},
        # search of a survey beam's whole DM-time array
        {"name": "search_survey", "op": "search", "nchan": 4096, "nsamp": 1 << 19, **BAND, "plan": LADDER,
         "widths": WIDTHS_512, "threshold": 6.0, "pulses": 200, "room": 16384},
        # mitigation of a survey beam before its dedispersion
        {"name": "rfi_survey", "op": "rfi", "nchan": 4096, "nsamp": 1 << 18, **BAND, "clip": 6.0, "block": 2048,
         "zero_dm": True, "spikes": 30},
        # what the program around the library does with each recorded beam, triage included
        {"name": "pipeline_beam", "op": "pipeline", "nchan": 4096, "nsamp": 1 << 18, **BAND, "plan": LADDER,
         "widths": WIDTHS_512, "threshold": 6.0, "pulses": 10, "room": 16384},
        # real-time use: one-second blocks of several beams, candidates back on the host
        {"name": "stream_step", "op": "stream", "nchan": 4096, "block": 20480, "beams": 4, **BAND,
         "plan": "0:0.1:700:1;70:0.3:350:2;175:1:125:4", "widths": WIDTHS_512, "threshold": 6.0, "pulses": 2,
         "room": 8192},
        # triage of a survey beam's events
        {"name": "cnn_forward_events", "op": "cnn_forward", "n": 6754},
        # one batch of the network's training
        {"name": "cnn_gradients_batch", "op": "cnn_gradients", "n": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_plan(rng, c, max_trials):
    """A DDplan-style ladder for the band of `c`: contiguous rows, the step
    growing with the downsampling, the largest delay at most half the data."""
    sweep = K_DM * (1 / c["f_lo"] ** 2 - 1 / c["f_hi"] ** 2)
    dm_top = min(1500.0, 0.5 * c["nsamp"] * c["tsamp"] / sweep)
    step = rng.uniform(2.5, 9.0) * c["tsamp"] / sweep  # samples per trial at the bottom of the band
    lo, rows = 0.0, []
    for d in rng.choice([[1], [1], [1, 2], [1, 2, 4], [1, 2, 4, 8], [1, 3], [2, 4]]):
        s = float("%.3g" % (step * d * rng.uniform(0.8, 1.6)))
        n = min(_log_int(rng, 16, max_trials), int((dm_top - lo) / s))
        if n < 3:
            break
        rows.append("%.10g:%.10g:%d:%d" % (lo, s, n, d))
        lo += n * s
    return ";".join(rows)


def draw(rng):
    op = rng.choice(["dedisperse"] * 4 + ["pipeline", "subband", "search", "search", "rfi", "stream",
                                          "cnn_forward", "cnn_gradients"])
    if op == "cnn_forward":
        return {"op": op, "n": _log_int(rng, 1, 7000)}
    if op == "cnn_gradients":
        return {"op": op, "n": _log_int(rng, 16, 512)}
    f_lo, f_hi = rng.choice([(1000.0, 1500.0), (1000.0, 1500.0), (1200.0, 1600.0), (270.0, 1620.0)])
    c = {"op": op, "f_lo": f_lo, "f_hi": f_hi, "tsamp": rng.choice([49.152e-6, 64e-6, 196.608e-6])}
    unit = rng.choice([1, 4, 16, 64, 1024])
    c["nchan"] = max(unit, _log_int(rng, 64, 4096) // unit * unit)
    if op == "rfi":
        c.update(nsamp=_log_int(rng, 1 << 12, 1 << 18), clip=rng.choice([0.0, 4.0, 6.0]),
                 block=rng.choice([1000, 2048, 4096]), zero_dm=rng.random() < 0.7, spikes=rng.randint(0, 30))
        c["zero_dm"] = c["zero_dm"] or c["clip"] == 0.0
        return c
    if op == "stream":
        c.update(f_lo=1000.0, f_hi=1500.0, tsamp=49.152e-6, nchan=rng.choice([256, 1024, 2048, 4096]),
                 block=rng.choice([8192, 10240, 20480]), beams=rng.randint(1, 4), widths=WIDTHS_512, threshold=6.0,
                 pulses=2, room=8192)
        c["nsamp"] = 2 * c["block"]
        c["plan"] = _draw_plan(rng, c, 500)
        del c["nsamp"]
        return c
    c["nsamp"] = _log_int(rng, 1 << 14, 1 << 19 if op != "pipeline" else 1 << 18)
    c["plan"] = _draw_plan(rng, c, 1500 if op != "pipeline" else 700)
    c["pulses"] = rng.randint(1, 8)
    if op in ("search", "pipeline"):
        c.update(widths=rng.choice([WIDTHS_32, WIDTHS_512]), threshold=6.0, room=4096)
    if op == "subband":
        rows = _rows(c)
        sub = [max(8, -(-c["nchan"] // max(1, 65535 // (255 * r[3])))) for r in rows]
        sub = [min(c["nchan"], max(s, rng.choice([16, 32, 50]))) for s in sub]
        c["n_sub"] = ",".join(map(str, sub))
        c["group"] = ",".join(str(rng.choice([8, 16, 24, 32])) for _ in rows)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rows(c):
    return [(float(a), float(b), int(n), int(d)) for a, b, n, d in (r.split(":") for r in c["plan"].split(";"))]


def _ints(text):
    return [int(v) for v in text.split(",")]


def _freqs(c):
    return c["f_lo"] + (np.arange(c["nchan"]) + 0.5) * (c["f_hi"] - c["f_lo"]) / c["nchan"]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _filterbank(c, nsamp, seed):
    """uint8 [nsamp][nchan] noise (mean 128, sigma 16) with `pulses`
    dispersed Gaussian pulses (matched-filter SNR 8-30) or `spikes` zero-DM
    spikes."""
    g, rng = _generator(seed), np.random.default_rng(seed)
    nchan = c["nchan"]
    fb = torch.empty((nsamp, nchan), dtype=torch.uint8, device="cuda")
    flat = fb.view(-1)
    for a in range(0, flat.numel(), 1 << 28):
        part = flat[a:a + (1 << 28)]
        x = torch.randn(part.numel(), generator=g, device="cuda").mul_(16.0).add_(128.0)
        part.copy_(x.round_().clamp_(0, 255))
    f = _freqs(c)
    ch = torch.arange(nchan, device="cuda")
    dm_top = max((r[0] + r[1] * r[2] for r in _rows(c)), default=0.0) if "plan" in c else 0.0
    for _ in range(c.get("pulses", 0)):
        dm = math.exp(rng.uniform(math.log(min(10.0, 0.1 * dm_top + 1e-3)), math.log(0.9 * dm_top + 1e-2)))
        fwhm = math.exp(rng.uniform(math.log(0.5e-3), math.log(20e-3)))
        sig = max(fwhm / 2.3548 / c["tsamp"], 0.3)
        amp = rng.uniform(8.0, 30.0) * 16.0 / math.sqrt(nchan * sig * math.sqrt(math.pi))
        delay = K_DM * dm * (1 / f ** 2 - 1 / f.max() ** 2) / c["tsamp"]
        t0 = rng.uniform(0.02, 0.95) * max(1.0, nsamp - delay.max())
        centre = torch.from_numpy(t0 + delay).cuda()
        half = int(3 * sig) + 1
        for k0 in range(-half, half + 1, 64):
            off = torch.arange(k0, min(k0 + 64, half + 1), device="cuda")
            t = centre.floor().long()[None] + off[:, None]
            v = amp * torch.exp(-0.5 * ((t - centre[None]) / sig) ** 2)
            ok = (t >= 0) & (t < nsamp)
            tt, cc = t[ok], ch[None].expand_as(t)[ok]
            fb[tt, cc] = (fb[tt, cc] + v[ok]).round().clamp(0, 255).to(torch.uint8)
    for _ in range(c.get("spikes", 0)):
        t = int(rng.integers(0, nsamp - 4))
        n = int(rng.integers(1, 4))
        fb[t:t + n] = (fb[t:t + n].float() + 40.0).clamp(0, 255).to(torch.uint8)
    return fb


def _row_lengths(c):
    """Valid outputs of every plan row: floor(nsamp / D) less its largest delay."""
    f, out = _freqs(c), []
    for lo, step, n, d in _rows(c):
        r = ((K_DM * (lo + (n - 1) * step)) * (1 / f ** 2 - 1 / f.max() ** 2)) / (c["tsamp"] * d)
        out.append(c["nsamp"] // d - int(np.floor(r + 0.5).max()))
    return out


def _dm_time(c, seed):
    """int32 DM-time array of a plan as dedispersion leaves it: sums of nchan
    channels and D samples, with single pulses over neighbouring trials."""
    g, rng = _generator(seed), np.random.default_rng(seed)
    parts = []
    lens = _row_lengths(c)
    total = sum(r[2] * m for r, m in zip(_rows(c), lens))
    flat = torch.empty(total, dtype=torch.int32, device="cuda")
    at = 0
    for (lo, step, n, d), m in zip(_rows(c), lens):
        mean, sig = 128.0 * c["nchan"] * d, 16.0 * math.sqrt(c["nchan"] * d)
        row = flat[at:at + n * m].view(n, m)
        at += n * m
        step_rows = max(1, (1 << 27) // m)
        for i in range(0, n, step_rows):
            x = torch.randn((min(step_rows, n - i), m), generator=g, device="cuda").mul_(sig).add_(mean)
            row[i:i + step_rows] = x.round_()
        for _ in range(max(1, c["pulses"] // len(lens))):
            i, w, snr = int(rng.integers(n)), 2 ** int(rng.integers(0, 9)), rng.uniform(6.0, 30.0)
            w = min(w, m)
            t = int(rng.integers(0, m - w + 1))
            for j in range(max(0, i - 8), min(n, i + 9)):
                row[j, t:t + w] += int(snr * sig / math.sqrt(w) * math.exp(-((j - i) / 4.0) ** 2))
    return flat


_CONV = [(2, 16), (16, 32), (32, 64), (64, 128)]


def _network(seed):
    """He-uniform weights and small biases in the library's order: conv
    w[cout][3][3][cin], b; fc1 w[192][2048], b; fc2 w[192], b[1]."""
    rng = np.random.default_rng([seed, 7])
    p = []
    for cin, cout in _CONV:
        p += [rng.uniform(-1, 1, cout * 9 * cin) * math.sqrt(6 / (9 * cin)), rng.uniform(-0.1, 0.1, cout)]
    p += [rng.uniform(-1, 1, 192 * 2048) * math.sqrt(6 / 2048), rng.uniform(-0.1, 0.1, 192)]
    p += [rng.uniform(-1, 1, 192) * math.sqrt(6 / 192), rng.uniform(-0.1, 0.1, 1)]
    return np.concatenate(p).astype(np.float32)


def _images(n, seed):
    """bf16 cutouts: z-scored noise, half of them with a pulse in the last bins."""
    g = _generator(seed)
    x = torch.randn((n, 2, 64, 64), generator=g, device="cuda")
    x[::2, :, :, 60:] += torch.rand((x[::2].shape[0], 1, 1, 1), generator=g, device="cuda") * 3.0
    x -= x.mean((2, 3), keepdim=True)
    x /= x.std((2, 3), keepdim=True, unbiased=False)
    return x.to(torch.bfloat16)


def _labels(n, seed):
    y = torch.zeros(n, dtype=torch.float32, device="cuda")
    y[::2] = 1.0
    return y


def _push_blocks(st):
    for b, blk in zip(st["beams"], st["blocks"]):
        st["stream"].push(b, blk)
    st["stream"].step()
    return st["stream"].poll()


def prepare(case, seed):
    c, op = dict(case), case["op"]
    ctx = gsp.context(0)
    st = {"case": c, "ctx": ctx, "op": op}
    if op in ("cnn_forward", "cnn_gradients"):
        st["x"], st["y"] = _images(c["n"], seed), _labels(c["n"], seed)
        st["net"] = gsp.Cnn(ctx, seed=1)
        st["net"].set_params(_network(seed))
        return st
    st["freqs"] = _freqs(c)
    if op == "rfi":
        st["fb"] = _filterbank(c, c["nsamp"], seed)
        st["out"] = torch.empty_like(st["fb"])
        return st
    rows = _rows(c)
    if op == "stream":
        st["blocks"] = [_filterbank({**c, "nsamp": c["block"]}, c["block"], seed * 64 + b).cpu().numpy()
                        for b in range(c["beams"])]
        s = gsp.Stream(ctx, 60 << 30, c["block"], _ints(c["widths"]), c["threshold"])
        st["stream"] = s
        st["beams"] = [s.open_beam(c["nchan"], st["freqs"], c["tsamp"], rows)[0] for _ in range(c["beams"])]
        # a stream that has been running: every row of its plan has output
        f = st["freqs"]
        top = max(lo + (n - 1) * step for lo, step, n, _ in rows)
        delay = K_DM * top * (1 / f.min() ** 2 - 1 / f.max() ** 2) / c["tsamp"]
        for _ in range(int(delay / c["block"]) + 2):
            _push_blocks(st)
        return st
    st["widths"] = _ints(c["widths"]) if "widths" in c else None
    if op == "subband":
        st["n_sub"], st["group"] = _ints(c["n_sub"]), _ints(c["group"])
        st["desc"] = gsp.subband_plan_shape(c["nsamp"], st["freqs"], c["tsamp"], rows, st["n_sub"], st["group"])
    else:
        st["desc"] = gsp.plan_shape(c["nsamp"], st["freqs"], c["tsamp"], rows)
    if op == "search":
        st["dmt"] = _dm_time(c, seed)
        return st
    st["fb"] = _filterbank(c, c["nsamp"], seed)
    st["dmt"] = torch.empty(st["desc"].total, dtype=torch.int32, device="cuda")
    if op == "pipeline":
        st["net"] = gsp.Cnn(ctx, seed=1)
        st["net"].set_params(_network(1))
    return st


def _fields(cands, room):
    """The candidates field by field, in a table with room for `room` of them."""
    table = np.zeros(max(room, len(cands)), cands.dtype)
    table[:len(cands)] = cands
    return {k: table[k] for k in ("seg", "dm_index", "dm", "t_peak", "t_first", "t_last", "width", "snr", "time_s")}


def run(st):
    op, ctx, c = st["op"], st["ctx"], st["case"]
    if op == "dedisperse":
        return ctx.dedisperse(st["fb"], st["freqs"], st["desc"], out=st["dmt"])
    if op == "subband":
        return ctx.dedisperse_subband(st["fb"], st["freqs"], st["desc"], st["n_sub"], st["group"], out=st["dmt"])
    if op == "search":
        return _fields(ctx.single_pulse_search(st["dmt"], st["desc"], st["widths"], c["threshold"]), c["room"])
    if op == "rfi":
        out, n = ctx.rfi_clean(st["fb"], c["clip"], c["block"], zero_dm=c["zero_dm"], out=st["out"])
        return {"out": out, "replaced": n}
    if op == "pipeline":
        ctx.dedisperse(st["fb"], st["freqs"], st["desc"], out=st["dmt"])
        cands = ctx.single_pulse_search(st["dmt"], st["desc"], st["widths"], c["threshold"])
        rep, n = gsp.group_candidates(cands)
        events = cands[np.unique(rep)]
        x = gsp.cutouts(ctx, st["fb"], st["freqs"], st["dmt"], st["desc"], events)
        logits = st["net"].forward(x) if n else 0.0
        scores = torch.zeros(max(c["room"], n), device="cuda")
        scores[:n] = logits
        return {"candidates": _fields(cands, c["room"]), "n_events": n, "logits": scores}
    if op == "stream":
        got = _push_blocks(st)
        return _fields(got, c["room"])
    if op == "cnn_forward":
        return st["net"].forward(st["x"])
    grads, loss = st["net"].gradients(st["x"], st["y"])
    return {"grads": grads, "loss": loss}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: every input read once, every output written once.  Operations:
    the network's products; sums over channels are shared between trials (no
    count of additions per output is a bound), a search's box sums come from
    one prefix sum per series."""
    c, op = case, case["op"]
    if op in ("cnn_forward", "cnn_gradients"):
        side, flops = 64, 0
        for cin, cout in _CONV:
            flops += 2 * side * side * 9 * cin * cout
            side //= 2
        flops += 2 * (2048 * 192 + 192)
        n_par = len(_network(1))
        if op == "cnn_forward":
            return {"bytes": c["n"] * (2 * 4096 * 2 + 4) + 2 * n_par, "flops": c["n"] * flops}
        first = 2 * 64 * 64 * 9 * 2 * 16  # no gradient of the input is needed
        return {"bytes": c["n"] * (2 * 4096 * 2 + 4) + 6 * n_par, "flops": c["n"] * (3 * flops - first)}
    if op == "rfi":
        return {"bytes": 2 * c["nsamp"] * c["nchan"], "flops": 0}
    rows = _rows(c)
    if op == "stream":
        outs = sum(r[2] * (c["block"] // r[3]) for r in rows)
        return {"bytes": c["beams"] * c["block"] * c["nchan"], "flops": c["beams"] * outs * len(_ints(c["widths"]))}
    outs = sum(r[2] * m for r, m in zip(rows, _row_lengths(c)))
    if op == "search":
        return {"bytes": 4 * outs, "flops": outs * len(_ints(c["widths"]))}
    return {"bytes": c["nsamp"] * c["nchan"] + 4 * outs, "flops": 0}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _exact_search(c, seed):
    flat = _dm_time(c, seed)
    widths, thr = sorted(set(_ints(c["widths"]))), float(np.float32(c["threshold"]))
    got = {k: [] for k in ("seg", "dm_index", "dm", "t_peak", "t_first", "t_last", "width", "snr", "time_s")}
    at = 0
    for s, ((lo, step, n, d), m) in enumerate(zip(_rows(c), _row_lengths(c))):
        row = flat[at:at + n * m].view(n, m)
        at += n * m
        take = max(1, (1 << 25) // m)
        for i0 in range(0, n, take):
            x = row[i0:i0 + take].long()
            x0 = x[:, :1]
            y = x - x0
            s1, s2 = y.sum(1).double() / m, (y * y).sum(1).double() / m
            mu, sd = (x0[:, 0].double() + s1)[:, None], (s2 - s1 * s1).clamp_min(0).sqrt()[:, None]
            cs = torch.nn.functional.pad(x.cumsum(1), (1, 0))
            best = torch.full(x.shape, -math.inf, dtype=torch.float64, device=x.device)
            arg = torch.zeros(x.shape, dtype=torch.int32, device=x.device)
            for w in widths:
                if w > m:
                    continue
                v = ((cs[:, w:] - cs[:, :-w]).double() - w * mu) / (sd * math.sqrt(w))
                b, a = best[:, w - 1:], arg[:, w - 1:]
                better = v > b
                b[better] = v[better]
                a[better] = w
            at2 = torch.nonzero((best >= thr) & (sd > 0))
            if not len(at2):
                continue
            snr, wid = best[at2[:, 0], at2[:, 1]].cpu().numpy(), arg[at2[:, 0], at2[:, 1]].cpu().numpy()
            tr, e = at2[:, 0].cpu().numpy(), at2[:, 1].cpu().numpy()
            cut = np.flatnonzero((np.diff(tr) != 0) | (np.diff(e) != 1)) + 1
            first, last = np.concatenate([[0], cut]), np.concatenate([cut, [len(e)]]) - 1
            run_of = np.repeat(np.arange(len(first)), last - first + 1)
            order = np.lexsort((e, -snr, run_of))
            peak = order[np.unique(run_of[order], return_index=True)[1]]
            t = e[peak] - wid[peak] + 1
            order = np.lexsort((e[first], t, tr[peak]))
            peak, first, last, t = peak[order], first[order], last[order], t[order]
            w = wid[peak]
            got["seg"].append(np.full(len(peak), s))
            got["dm_index"].append(tr[peak] + i0)
            got["dm"].append(lo + (tr[peak] + i0) * step)
            got["t_peak"].append(t)
            got["t_first"].append(e[first])
            got["t_last"].append(e[last])
            got["width"].append(w)
            got["snr"].append(snr[peak])
            got["time_s"].append((t + 0.5 * w) * d * c["tsamp"])
    out = {k: np.concatenate(v) if v else np.zeros(0) for k, v in got.items()}
    out = {k: np.pad(v, (0, max(0, c["room"] - len(v)))) for k, v in out.items()}
    return {k: v.astype(np.float64) if k in ("dm", "snr", "time_s") else v.astype(np.int64) for k, v in out.items()}


def _exact_network(c, seed, grad):
    par = torch.from_numpy(_network(seed)).cuda()
    at, lay = 0, []

    def take(n, rounded):
        nonlocal at
        v = par[at:at + n]
        at += n
        return (v.to(torch.bfloat16) if rounded else v).double().requires_grad_(grad)

    for cin, cout in _CONV:
        lay.append((take(cout * 9 * cin, True), take(cout, False)))
    lay.append((take(192 * 2048, True), take(192, False)))
    lay.append((take(192, True), take(1, False)))

    def logits(x):
        h = x.double()
        for (w, b), (cin, cout) in zip(lay, _CONV):
            k = w.view(cout, 3, 3, cin).permute(3, 1, 2, 0).reshape(cin * 9, cout)
            u = torch.nn.functional.unfold(h, 3, padding=1).transpose(1, 2)
            side = h.shape[-1]
            h = (u.reshape(-1, cin * 9) @ k + b).relu().view(-1, side, side, cout).permute(0, 3, 1, 2)
            h = torch.nn.functional.max_pool2d(h, 2)
        h = h.permute(0, 2, 3, 1).reshape(len(x), 2048)
        h = (h @ lay[4][0].view(192, 2048).t() + lay[4][1]).relu()
        return h @ lay[5][0] + lay[5][1]

    x = _images(c["n"], seed)
    if not grad:
        return torch.cat([logits(x[k:k + 256]) for k in range(0, len(x), 256)])
    y = _labels(c["n"], seed).double()
    loss = torch.nn.functional.binary_cross_entropy_with_logits(logits(x), y)
    g = torch.autograd.grad(loss, [t for l in lay for t in l])
    return {"grads": torch.cat([t.reshape(-1) for t in g]), "loss": float(loss)}


def exact(case, seed):
    """Computed numbers in 64 bits; dedispersion and mitigation give whole
    numbers, which have to be equal."""
    op = case["op"]
    if op == "search":
        return _exact_search(case, seed)
    if op in ("cnn_forward", "cnn_gradients"):
        return _exact_network(case, seed, op == "cnn_gradients")
    return None

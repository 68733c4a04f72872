"""Performance cases of the multibeam transient path.

Each case is work that a program built on this package gives it through the
public entry points (`paper_1307_5700_amd.api`), on synthetic data shaped like
the 20 MHz beams (398-418 MHz) the package is written for:

* `step`     RFI pass, dedispersion with normalisation, detection of one chunk
             that is already on the GPU (eager calls);
* `graph`    the same step captured as a HIP graph and replayed;
* `execute`  dedispersion with normalisation alone, for chunks that need no
             cleaning;
* `stream`   a beam's stream: consecutive chunks through its overlap ring;
* `batch`    several uneven beams per launch, two consecutive chunks each;
* `median`, `codec`, `voltages`  the stages around the path: the windowed
             median of a plane, the data writer's 8-bit codec there and back,
             and the front end's power step with the 4+4-bit voltage codec;
* `cluster`, `fdbscan`  clustering of a detection list.

`listed()` names the cases, `draw(rng)` makes one more of the same ranges,
`prepare` builds what a program holds before the call, `run` is one pass,
`work` what a pass cannot do without and `exact` the outputs in 64 bits.
"""
import math

import numpy as np
import torch

from paper_1307_5700_amd import api, synth

BAND_LO, BAND_MHZ = 398.0, 20.0
TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "u8": torch.uint8}
SIZE = {"f32": 4, "f16": 2, "u8": 1}
NSIGMA = 6.0
CAPACITY = 1 << 15


def listed():
    return [
        # the smallest beam of the benchmarks, one captured step per chunk:
        # launches and single-workgroup kernels count
        dict(name="graph_f32_256ch", kind="graph", nchans=256, nsamps=8192, ndms=64, dm_step=1.0, tsamp=100e-6,
             dtype="f32", rfi=True),
        # odd channel, DM and sample counts, a coarse DM step, a ragged row
        dict(name="execute_f32_ragged", kind="execute", nchans=300, nsamps=9001, ndms=37, dm_step=0.7,
             tsamp=51.2e-6, dtype="f32", rfi=False),
        # the paper-shaped beam, the benchmark's default workload
        dict(name="step_f32_1024ch", kind="step", nchans=1024, nsamps=65536, ndms=640, dm_step=0.2, tsamp=51.2e-6,
             dtype="f32", rfi=True),
        # the same beam stored in 8 bits, no cleaning
        dict(name="execute_u8_1024ch", kind="execute", nchans=1024, nsamps=65536, ndms=640, dm_step=0.2,
             tsamp=51.2e-6, dtype="u8", rfi=False),
        # many channels and DMs in half precision: the precision sweep's beam
        dict(name="execute_f16_4096ch", kind="execute", nchans=4096, nsamps=65536, ndms=2048, dm_step=0.2,
             tsamp=51.2e-6, dtype="f16", rfi=False),
        # one served beam: 8-bit chunks of uneven length with the RFI pass
        dict(name="stream_u8_1024ch", kind="stream", nchans=1024, chunks="16384,8192,24576", ndms=640, dm_step=0.2,
             tsamp=51.2e-6, dtype="u8", rfi=True),
        # uneven beams batched into one launch, two chunks each
        dict(name="batch_u8_4beams", kind="batch", beams="512x320x16384,768x480x32768,1024x640x65536,2048x320x16384",
             dm_step=0.2, tsamp=51.2e-6, dtype="u8", rfi=True),
        # median of a dedispersed plane, 5-sample window
        dict(name="median_640x59434", kind="median", rows=640, cols=59434, half=2),
        # 8-bit codes of a power buffer and back (data writer)
        dict(name="codec_1024x65536", kind="codec", rows=1024, cols=65536, mu=255.0),
        # beamformed 16-bit complex voltages: power, and 4+4-bit codes and back
        dict(name="voltages_1024x65536", kind="voltages", rows=1024, cols=65536, mu=255.0),
        # detections of a low-threshold pass: exact DBSCAN
        dict(name="cluster_640x59434", kind="cluster", ndms=640, cols=59434, density=1.35e-3, npulses=5),
        # the paper's FDBSCAN on such a list
        dict(name="fdbscan_640x59434", kind="fdbscan", ndms=640, cols=59434, density=1.35e-3, npulses=5),
    ]


# ---- drawn cases --------------------------------------------------------

MAX_ADDS = 4096.0 * 2048 * (65536 - 19562)      # the largest listed dedispersion


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _max_delay(ndms, dm_step, tsamp):
    return 4150.0 * (ndms - 1) * dm_step * (1 / 398.0 ** 2 - 1 / 418.0 ** 2) / tsamp


def _draw_beam(rng, max_adds, nsamps_hi=131072):
    while True:
        nchans, ndms = _log_int(rng, 64, 4096), _log_int(rng, 16, 2048)
        nsamps = _log_int(rng, 4096, nsamps_hi)
        tsamp = rng.choice([51.2e-6, 51.2e-6, 100e-6])
        dm_step = rng.choice([0.2, 0.2, 0.3, 0.5, 1.0])
        smax = _max_delay(ndms, dm_step, tsamp)
        if smax < 0.6 * nsamps and nchans * ndms * (nsamps - smax) <= max_adds:
            return nchans, ndms, nsamps, dm_step, tsamp


def draw(rng):
    kind = rng.choice(["graph", "step", "step", "execute", "execute", "execute", "execute", "stream", "stream",
                       "batch", "median", "codec", "voltages", "cluster", "fdbscan"])
    if kind in ("graph", "step", "execute"):
        nchans, ndms, nsamps, dm_step, tsamp = _draw_beam(rng, MAX_ADDS if kind == "execute" else MAX_ADDS / 4)
        return dict(kind=kind, nchans=nchans, nsamps=nsamps, ndms=ndms, dm_step=dm_step, tsamp=tsamp,
                    dtype=rng.choice(["f32", "f16", "u8"]), rfi=kind != "execute")
    if kind == "stream":
        nchans, ndms, _, dm_step, tsamp = _draw_beam(rng, MAX_ADDS / 16)
        lo = int(_max_delay(ndms, dm_step, tsamp)) + 512
        chunks = ",".join(str(4 * (_log_int(rng, max(lo, 4096), max(2 * lo, 32768)) // 4)) for _ in range(3))
        return dict(kind=kind, nchans=nchans, chunks=chunks, ndms=ndms, dm_step=dm_step, tsamp=tsamp,
                    dtype=rng.choice(["f32", "f16", "u8", "u8"]), rfi=rng.random() < 0.7)
    if kind == "batch":
        dm_step, beams = 0.2, []
        for _ in range(rng.randint(2, 5)):
            while True:
                C, nd, L = _log_int(rng, 128, 2048), _log_int(rng, 64, 1280), 4 * _log_int(rng, 2048, 16384)
                if _max_delay(nd, dm_step, 51.2e-6) < 0.6 * L and C * nd * L <= MAX_ADDS / 8:
                    break
            beams.append(f"{C}x{nd}x{L}")
        return dict(kind=kind, beams=",".join(beams), dm_step=dm_step, tsamp=51.2e-6,
                    dtype=rng.choice(["f32", "u8", "u8"]), rfi=rng.random() < 0.8)
    if kind == "median":
        return dict(kind=kind, rows=_log_int(rng, 16, 1280), cols=_log_int(rng, 1024, 65536),
                    half=rng.choice([1, 2, 2, 3, 4, 8]))
    if kind in ("codec", "voltages"):
        return dict(kind=kind, rows=_log_int(rng, 16, 1024), cols=_log_int(rng, 1024, 65536),
                    mu=rng.choice([255.0, 100.0]))
    return dict(kind=kind, ndms=_log_int(rng, 64, 640), cols=_log_int(rng, 4096, 59434),
                density=rng.choice([3e-4, 1.35e-3]), npulses=rng.randint(1, 5))


# ---- shared helpers -----------------------------------------------------

def _delays(nchans, ndms, dm_step, tsamp):
    """Integer delays of Eq. (1), [ndms][nchans]."""
    df = BAND_MHZ / nchans
    f = BAND_LO + df / 2 + np.arange(nchans) * df
    inv = 1.0 / (f * f) - 1.0 / (f[-1] * f[-1])
    dm = np.arange(ndms) * dm_step
    return np.floor((4150.0 * dm)[:, None] * inv[None, :] / tsamp + 0.5).astype(np.int64)


def _filterbank(C, T, dtype, seed, delays, rfi):
    """Noise of unit variance with three dispersed pulses and, for beams that
    are cleaned, a narrowband burst, two broadband spikes and a zeroed gap;
    rows padded to a multiple of 8 samples."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    ld = (T + 7) // 8 * 8
    v = torch.randn((C, ld), generator=g, device="cuda")
    v[:, T:] = 0
    ch = torch.arange(C, device="cuda")
    for _ in range(3):
        row = torch.from_numpy(delays[int(rng.integers(len(delays) // 8, len(delays)))]).cuda()
        t0, amp = int(rng.integers(0, max(T - int(row.max()) - 16, 1))), float(rng.uniform(0.3, 1.0))
        for k in range(int(rng.integers(1, 17))):
            v[ch, (row + t0 + k).clamp(max=T - 1)] += amp
    gap = None
    if rfi:
        c0, t0 = int(rng.integers(0, max(C - 5, 1))), int(rng.integers(0, T // 2))
        v[c0:c0 + 5, t0:t0 + int(rng.integers(1024, 4097))] += 20.0
        for _ in range(2):
            t0 = int(rng.integers(0, T - 3))
            v[:, t0:t0 + int(rng.integers(1, 4))] += 20.0
        gap = (int(rng.integers(0, C)), int(rng.integers(0, T - 64)))
    v[:, T:] = 0
    if dtype == "u8":
        x = torch.clamp(torch.round(128 + 16 * v), 0, 255).to(torch.uint8)
        if gap:
            x[gap[0]:gap[0] + 64, gap[1]:gap[1] + 64] = 0
    else:
        x = v.to(TORCH_DTYPE[dtype])
    return x[:, :T]


def _plan(nchans, ndms, dm_step, tsamp, dtype):
    f0, df = synth.band(nchans, BAND_LO, BAND_MHZ)
    return api.Plan(nchans, f0, df, tsamp, ndms, 0.0, dm_step, dtype=dtype)


def _det_buffers(plan):
    """Candidate records, their count and the detection workspace (no peaks)."""
    return (torch.zeros(CAPACITY * 24, dtype=torch.uint8, device="cuda"),
            torch.zeros(1, dtype=torch.int64, device="cuda"), None,
            torch.empty(plan.detect_work_bytes, dtype=torch.uint8, device="cuda"))


def _records(det):
    """Candidate records as (integers, floats): dm index, 64-bit sample; SNR, DM."""
    cands, count = det[0], det[1]
    i = cands.view(torch.int32).view(-1, 6)
    return {"dm_index": i[:, 0], "sample": cands.view(torch.int64).view(-1, 3)[:, 1],
            "snr": cands.view(torch.float32).view(-1, 6)[:, 4], "dm": cands.view(torch.float32).view(-1, 6)[:, 5],
            "count": count}


def _beams_of(case):
    if case["kind"] == "batch":
        return [tuple(int(v) for v in b.split("x")) for b in case["beams"].split(",")]
    return []


def _chunks_of(case):
    return [int(v) for v in case["chunks"].split(",")]


class _Lane:
    """One beam's plan, ring, chunks and output buffers."""

    def __init__(self, C, nd, lengths, case, seed):
        s = _delays(C, nd, case["dm_step"], case["tsamp"])
        self.plan = _plan(C, nd, case["dm_step"], case["tsamp"], case["dtype"])
        self.beam = api.Beam(self.plan)
        self.xs = [_filterbank(C, L, case["dtype"], seed + 101 * k, s, case["rfi"]) for k, L in enumerate(lengths)]
        self.states = [self.plan.alloc_rfi_state(L) if case["rfi"] else None for L in lengths]
        self.outs, seen = [], 0
        for L in lengths:
            nout = max(min(seen, self.plan.max_delay) + L - self.plan.max_delay, 0)
            self.outs.append(self.plan.alloc_output(nout))
            seen += L
        self.norms = [self.plan.alloc_norm() for _ in lengths]
        self.dets = [_det_buffers(self.plan) for _ in lengths]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "execute", "graph"):
        s = _delays(case["nchans"], case["ndms"], case["dm_step"], case["tsamp"])
        x = _filterbank(case["nchans"], case["nsamps"], case["dtype"], seed, s, case["rfi"])
        plan = _plan(case["nchans"], case["ndms"], case["dm_step"], case["tsamp"], case["dtype"])
        st = {"case": case, "plan": plan, "x": x}
        if kind == "graph":
            st["graph"] = api.ChunkGraph(plan, x, rfi=case["rfi"], nsigma=NSIGMA, capacity=CAPACITY)
            st["graph"].det[0].zero_()
            return st
        st["out"] = plan.alloc_output(case["nsamps"] - plan.max_delay)
        st["norm"] = plan.alloc_norm()
        if kind == "step":
            st["state"] = plan.alloc_rfi_state(case["nsamps"])
            st["det"] = _det_buffers(plan)
        return st
    if kind == "stream":
        return {"case": case, "lanes": [_Lane(case["nchans"], case["ndms"], _chunks_of(case), case, seed)]}
    if kind == "batch":
        lanes = [_Lane(C, nd, [L, L], case, seed + 13 * i) for i, (C, nd, L) in enumerate(_beams_of(case))]
        return {"case": case, "lanes": lanes, "work": api.alloc_batch_work(len(lanes))}
    g = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "median":
        ld = (case["cols"] + 3) // 4 * 4
        plane = 32.0 * torch.randn((case["rows"], ld), generator=g, device="cuda")
        return {"case": case, "plane": plane, "out": torch.zeros_like(plane)}
    if kind == "codec":
        ld = (case["cols"] + 3) // 4 * 4
        x = torch.randn((case["rows"], ld), generator=g, device="cuda") ** 2 \
            + torch.randn((case["rows"], ld), generator=g, device="cuda") ** 2
        return {"case": case, "x": x, "codes": torch.zeros((case["rows"], ld), dtype=torch.uint8, device="cuda"),
                "xmax": torch.zeros(case["rows"], device="cuda"), "out": torch.zeros_like(x)}
    if kind == "voltages":
        n = torch.randn((case["rows"], case["cols"], 2), generator=g, device="cuda")
        v = torch.clamp(torch.round(2000.0 * n), -32768, 32767).to(torch.int16)
        rows, ld = case["rows"], (case["cols"] + 3) // 4 * 4
        return {"case": case, "v": v, "power": torch.zeros((rows, ld), device="cuda"),
                "codes": torch.zeros((rows, ld), dtype=torch.uint8, device="cuda"),
                "xmax": torch.zeros(rows, dtype=torch.int32, device="cuda"),
                "back": torch.zeros((rows, ld, 2), device="cuda")}
    s, d, q = synth.detections(case["ndms"], case["cols"], seed, density=case["density"], npulses=case["npulses"])
    rec = np.zeros(len(s), dtype=api.CANDIDATE_DTYPE)
    rec["dm_index"], rec["sample"], rec["snr"], rec["dm"] = d, s, q, 0.2 * d
    buf = torch.from_numpy(rec.view(np.uint8).copy()).cuda()
    # labels of at most this many detections (lists differ in length by seed)
    room = int(1.2 * case["density"] * case["ndms"] * case["cols"]) + 4096 * case["npulses"]
    st = {"case": case, "cands": buf, "n": len(s), "labels": torch.full((room,), -2, dtype=torch.int32, device="cuda")}
    if kind == "cluster":
        st["work"] = api.alloc_cluster_work(len(s), case["ndms"], buf.device)
        st["nclusters"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return st


def _run_chunk(lane, k, case):
    x, state, out, norm, det = lane.xs[k], lane.states[k], lane.outs[k], lane.norms[k], lane.dets[k]
    if state is not None:
        lane.plan.rfi_threshold(x, state)
    _, _, nout, _ = lane.plan.execute(x, rfi_state=state, out=out, norm=norm, beam=lane.beam)
    lane.plan.detect(out, nout, norm, NSIGMA, buffers=det, beam=lane.beam)
    return {"plane": out[:, :nout], "norm": norm, **_records(det)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("step", "execute"):
        plan, x, out, norm = state["plan"], state["x"], state["out"], state["norm"]
        if kind == "execute":
            _, _, nout, _ = plan.execute(x, out=out, norm=norm)
            return {"plane": out[:, :nout], "norm": norm}
        plan.rfi_threshold(x, state["state"])
        _, _, nout, s0 = plan.execute(x, rfi_state=state["state"], out=out, norm=norm)
        plan.detect(out, nout, norm, NSIGMA, sample0=s0, buffers=state["det"])
        return {"plane": out[:, :nout], "norm": norm, **_records(state["det"])}
    if kind == "graph":
        g = state["graph"]
        g.replay()
        return {"plane": g.out[:, :g.nout], "norm": g.norm, **_records(g.det)}
    if kind == "stream":
        lane = state["lanes"][0]
        lane.beam.seek(0)
        return [_run_chunk(lane, k, case) for k in range(len(lane.xs))]
    if kind == "batch":
        lanes, res = state["lanes"], []
        for ln in lanes:
            ln.beam.seek(0)
        for k in range(2):
            for ln in lanes:
                if case["rfi"]:
                    ln.plan.rfi_threshold(ln.xs[k], ln.states[k])
            outs = api.execute_batch([dict(plan=ln.plan, x=ln.xs[k], rfi_state=ln.states[k], out=ln.outs[k],
                                           norm=ln.norms[k], beam=ln.beam) for ln in lanes], work=state["work"])
            for ln, (out, norm, nout, _) in zip(lanes, outs):
                ln.plan.detect(out, nout, norm, NSIGMA, buffers=ln.dets[k], beam=ln.beam)
                res.append({"plane": out[:, :nout], "norm": norm, **_records(ln.dets[k])})
        return res
    if kind == "median":
        api.median_filter(state["plane"], case["cols"], case["half"], out=state["out"])
        return state["out"][:, :case["cols"]]
    if kind == "codec":
        codes, xmax = api.mulaw_encode(state["x"], case["cols"], mu=case["mu"], codes=state["codes"], xmax=state["xmax"])
        out = api.mulaw_decode(codes, xmax, case["cols"], mu=case["mu"], out=state["out"])
        return {"codes": codes[:, :case["cols"]], "xmax": xmax, "out": out[:, :case["cols"]]}
    if kind == "voltages":
        power = api.power_from_voltages(state["v"], out=state["power"])
        codes, xmax = api.mulaw_encode_complex(state["v"], mu=case["mu"], codes=state["codes"], xmax=state["xmax"])
        back = api.mulaw_decode_complex(codes, xmax, case["cols"], mu=case["mu"], out=state["back"])
        return {"power": power[:, :case["cols"]], "codes": codes[:, :case["cols"]], "xmax": xmax,
                "back": back[:, :case["cols"]]}
    args = (state["cands"], state["n"], case["ndms"], 16, 4, 2.0, 5)
    if kind == "cluster":
        labels, nc = api.cluster_candidates(*args, labels=state["labels"], nclusters=state["nclusters"],
                                            work=state["work"])
        return {"labels": state["labels"], "nclusters": nc}
    labels, nc, nq = api.fdbscan_candidates(*args, labels=state["labels"])
    return {"labels": state["labels"], "nclusters": nc, "nqueries": nq}


# ---- what a pass cannot do without ---------------------------------------

def _beam_work(C, nd, T, nout, case):
    """Samples in, plane and lines out; one add per channel and output."""
    return (C * T * SIZE[case["dtype"]] + nd * nout * 4 + nd * 32, float(C) * nd * nout + 2.0 * C * T * case["rfi"])


def work(case):
    kind = case["kind"]
    if kind in ("step", "execute", "graph", "stream", "batch"):
        jobs = []
        if kind == "batch":
            for C, nd, L in _beams_of(case):
                smax = int(_max_delay(nd, case["dm_step"], case["tsamp"]))
                jobs += [(C, nd, L, L - smax), (C, nd, L, L)]
        else:
            C, nd = case["nchans"], case["ndms"]
            smax, seen = int(_max_delay(nd, case["dm_step"], case["tsamp"])), 0
            for L in (_chunks_of(case) if kind == "stream" else [case["nsamps"]]):
                jobs.append((C, nd, L, max(min(seen, smax) + L - smax, 0)))
                seen += L
        w = [_beam_work(*j, case) for j in jobs]
        return {"bytes": float(sum(b for b, _ in w)), "flops": sum(f for _, f in w)}
    if kind == "median":
        n = case["rows"] * case["cols"]
        return {"bytes": 8.0 * n, "flops": float(n * (2 * case["half"] + 1))}
    if kind == "codec":
        n = case["rows"] * case["cols"]
        return {"bytes": 10.0 * n, "flops": 4.0 * n}
    if kind == "voltages":
        n = case["rows"] * case["cols"]
        return {"bytes": 18.0 * n, "flops": 6.0 * n}
    n = case["density"] * case["ndms"] * case["cols"] + 500.0 * case["npulses"]
    return {"bytes": 28.0 * n, "flops": 3.0 * n * n * min(1.0, 33.0 * 9 / (case["ndms"] * case["cols"]))}


# ---- outputs in 64 bits ----------------------------------------------------

def _clean64(x):
    """The RFI pass in 64 bits with the default parameters: degree-3 bandpass
    with repeated masking, 256-sample channel chunks, spectra, 5 sigma each."""
    y = x.double()
    C, T = y.shape
    W, k, p = 256, 5.0, 3
    B = (y.sum(1) / T).cpu().numpy()
    u = (2.0 * np.arange(C) - (C - 1)) / (C - 1)
    q, r = np.linalg.qr(np.vander(u, p + 1, increasing=True))
    masked, Bi = np.zeros(C, bool), B
    for _ in range(8):
        fit = q @ (q.T @ Bi)
        grown = masked | (np.abs(B - fit) > k * np.sqrt(np.mean((Bi - fit) ** 2)))
        settled, masked = bool((grown == masked).all()), grown
        keep, Bi = np.flatnonzero(~masked), B.copy()
        for c in np.flatnonzero(masked):
            i = int(np.searchsorted(keep, c))
            near = [B[keep[j]] for j in (i - 1, i) if 0 <= j < len(keep)]
            Bi[c] = sum(near) / len(near)
        if settled:
            break
    fit = q @ (q.T @ Bi)
    sigma = float(np.sqrt(np.mean((Bi - fit) ** 2)) * math.sqrt(T * C / (C - p - 1)))
    y -= torch.from_numpy(fit).cuda()[:, None]
    J = (T + W - 1) // W
    pad = torch.zeros((C, J * W), dtype=torch.float64, device="cuda")
    pad[:, :T] = y
    lens = torch.full((J,), float(W), dtype=torch.float64, device="cuda")
    lens[-1] = T - (J - 1) * W
    F = (pad.view(C, J, W).sum(2) / lens).abs() > k * sigma / lens.sqrt()
    Fx = F.clone()
    Fx[:, 1:] |= F[:, :-1]
    Fx[:, :-1] |= F[:, 1:]
    y[Fx.repeat_interleave(W, 1)[:, :T]] = 0.0
    y[:, (y.sum(0) / C).abs() > k * sigma / math.sqrt(C)] = 0.0
    return y


def _dedisperse64(y, delays, nout):
    out = torch.zeros((len(delays), nout), dtype=torch.float64, device="cuda")
    s = torch.from_numpy(delays).cuda()
    for c in range(y.shape[0]):
        out += y[c].double().unfold(0, nout, 1)[s[:, c]]
    return out


def _outputs64(D, sample0, dm_step, detect):
    """Plane, normalisation lines (a, b, sigma, flags) and, if asked for, the
    detections above NSIGMA in (DM, sample) order."""
    nd, N = D.shape
    t = torch.arange(N, dtype=torch.float64, device="cuda")
    tc = t - (N - 1) / 2.0
    mean = D.mean(1)
    b = ((D - mean[:, None]) @ tc) / (tc @ tc)
    a = mean - b * (N - 1) / 2.0
    r = D - a[:, None] - b[:, None] * t
    sigma = (r * r).mean(1).sqrt()
    norm = torch.stack([a, b, sigma, torch.zeros_like(a)], 1)
    if not detect:
        return {"plane": D, "norm": norm}
    z = r / sigma[:, None]
    hit = (z > NSIGMA).nonzero()
    n = min(len(hit), CAPACITY)
    res = {"plane": D, "norm": norm, "dm_index": torch.zeros(CAPACITY, dtype=torch.int32, device="cuda"),
           "sample": torch.zeros(CAPACITY, dtype=torch.int64, device="cuda"),
           "snr": torch.zeros(CAPACITY, dtype=torch.float64, device="cuda"),
           "dm": torch.zeros(CAPACITY, dtype=torch.float64, device="cuda"),
           "count": torch.tensor([len(hit)], device="cuda")}
    d, s = hit[:n, 0], hit[:n, 1]
    res["dm_index"][:n], res["sample"][:n] = d.int(), s + sample0
    res["snr"][:n], res["dm"][:n] = z[d, s], d.double() * dm_step
    return res


def _stream64(C, nd, lengths, case, seed):
    delays = _delays(C, nd, case["dm_step"], case["tsamp"])
    smax, seen, res = int(delays.max()), 0, []
    tail = torch.zeros((C, 0), dtype=torch.float64, device="cuda")
    for k, L in enumerate(lengths):
        x = _filterbank(C, L, case["dtype"], seed + 101 * k, delays, case["rfi"])
        y = torch.cat([tail, _clean64(x) if case["rfi"] else x.double()], 1)
        D = _dedisperse64(y, delays, y.shape[1] - smax)
        res.append(_outputs64(D, seen - tail.shape[1], case["dm_step"], True))
        tail, seen = y[:, y.shape[1] - smax:].clone(), seen + L
    return res


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "execute", "graph"):
        delays = _delays(case["nchans"], case["ndms"], case["dm_step"], case["tsamp"])
        x = _filterbank(case["nchans"], case["nsamps"], case["dtype"], seed, delays, case["rfi"])
        y = _clean64(x) if case["rfi"] else x
        D = _dedisperse64(y, delays, case["nsamps"] - int(delays.max()))
        return _outputs64(D, 0, case["dm_step"], kind != "execute")
    if kind == "stream":
        return _stream64(case["nchans"], case["ndms"], _chunks_of(case), case, seed)
    if kind == "batch":
        per = [_stream64(C, nd, [L, L], case, seed + 13 * i) for i, (C, nd, L) in enumerate(_beams_of(case))]
        return [p[k] for k in range(2) for p in per]
    if kind == "median":
        x = prepare(case, seed)["plane"][:, :case["cols"]].double()
        h = case["half"]
        p = torch.cat([x[:, :1].expand(-1, h), x, x[:, -1:].expand(-1, h)], 1)
        return torch.cat([r.unfold(1, 2 * h + 1, 1).median(2).values for r in p.split(64)])
    if kind == "codec":
        st = prepare(case, seed)
        x = st["x"][:, :case["cols"]].double()
        X = x.max(1).values
        mu = float(np.float32(case["mu"]))
        q = torch.floor(255 * torch.log1p(mu * x / X[:, None]) / math.log1p(mu) + 0.5)
        return {"codes": None, "xmax": X, "out": X[:, None] / mu * torch.expm1(q / 255 * math.log1p(mu))}
    if kind == "voltages":
        v = prepare(case, seed)["v"].double()
        X = v.abs().amax((1, 2))
        mu = float(np.float32(case["mu"]))
        # (whole-number samples meet half levels exactly, e.g. X/17 for mu = 255)
        m = torch.floor(7 * torch.log1p(mu * v.abs() / X[:, None, None]) / math.log1p(mu) + 0.5 + 1e-12)
        back = torch.sign(v) * X[:, None, None] / mu * torch.expm1(m / 7 * math.log1p(mu))
        return {"power": (v * v).sum(2), "codes": None, "xmax": None, "back": back}
    return None

"""The work that users of this library have it do, as cases that can be timed.

Each case is one pass through the public entry points of ``paper_1601_01165_amd``
with its default (untuned) kernel choice.  The set-ups are the two surveys of
the library's own workloads and tests: an Apertif-like band (1270-1570 MHz,
50 us, DM step 0.25), the small test band (1400-1500 MHz, 50 us, DM step 1)
and a LOFAR-like band (134.875-141.125 MHz, 5 us, DM step 0.01).

Kinds of case
  forward   dedisperse one or several beams: float32 (optional per-channel
            weights) or uint8 input
  batch     many uneven float32 beams in one persistent launch
  train     differentiable step: forward, adjoint and weight gradient
  detect    dedispersion with the single-pulse search, float32 or uint8
  rows      the single-pulse search over series that are already stored
"""
import math

import numpy as np
import torch

import paper_1601_01165_amd as dd

#: band name: (low MHz, high MHz, sample time s, DM step)
BANDS = {
    "apertif": (1270.0, 1570.0, 50e-6, 0.25),
    "test": (1400.0, 1500.0, 50e-6, 1.0),
    "lofar": (134.875, 141.125, 5e-6, 0.01),
}


def listed():
    return [
        # a first look at a short stretch of data, or one call of an interactive session: the smallest
        # call, where launch and latency count (the library's own tiny workload)
        {"name": "forward_tiny", "kind": "forward", "dtype": "f32", "band": "test", "nbeam": 1, "nchan": 64, "ndm": 32,
         "nsamp": 4096, "weighted": False},
        # a low-latency pipeline that hands over a tenth of a second at a time with a coarse DM list,
        # sizes that divide nothing
        {"name": "forward_chunk", "kind": "forward", "dtype": "f32", "band": "apertif", "nbeam": 1, "nchan": 1024,
         "ndm": 301, "nsamp": 2003, "weighted": False},
        # one second of one Apertif-like beam with the full DM list: the ordinary call
        {"name": "forward_apertif", "kind": "forward", "dtype": "f32", "band": "apertif", "nbeam": 1, "nchan": 1024,
         "ndm": 2048, "nsamp": 20000, "weighted": False},
        # a few beams sharing one plan, with a per-channel gain (bandpass or RFI mask), ragged sizes
        {"name": "forward_weighted", "kind": "forward", "dtype": "f32", "band": "apertif", "nbeam": 3, "nchan": 768,
         "ndm": 1001, "nsamp": 9973, "weighted": True},
        # one second of one LOFAR-like beam as recorded, 8 bits: the largest output
        {"name": "forward_lofar_u8", "kind": "forward", "dtype": "u8", "band": "lofar", "nbeam": 1, "nchan": 32,
         "ndm": 2048, "nsamp": 200000, "weighted": False},
        # one second of one Apertif-like beam as recorded, 8 bits: many channels
        {"name": "forward_apertif_u8", "kind": "forward", "dtype": "u8", "band": "apertif", "nbeam": 1, "nchan": 1024,
         "ndm": 2048, "nsamp": 20000, "weighted": False},
        # a multi-beam second with uneven set-ups in one launch: the largest amount of work
        {"name": "batch_uneven", "kind": "batch", "nbeam": 24, "mix": 1604},
        # a training step of per-channel weights on a few beams
        {"name": "train_apertif", "kind": "train", "band": "apertif", "nbeam": 2, "nchan": 1024, "ndm": 1024,
         "nsamp": 20000},
        # a training step at the size of a unit test or a notebook
        {"name": "train_tiny", "kind": "train", "band": "test", "nbeam": 1, "nchan": 64, "ndm": 32, "nsamp": 4096},
        # real-time search of one second of one beam, in each data type
        {"name": "detect_lofar_u8", "kind": "detect", "dtype": "u8", "band": "lofar", "nbeam": 1, "nchan": 32,
         "ndm": 2048, "nsamp": 200000},
        {"name": "detect_apertif", "kind": "detect", "dtype": "f32", "band": "apertif", "nbeam": 1, "nchan": 1024,
         "ndm": 2000, "nsamp": 20000},
        # searching series that another step stored
        {"name": "rows_f32", "kind": "rows", "dtype": "f32", "nrows": 2000, "nsamp": 20000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds: sizes spread over their logarithm, most of them odd."""
    kind = rng.choice(["forward", "forward", "forward_u8", "forward_u8", "batch", "train", "detect", "detect_u8", "rows"])
    if kind == "batch":
        return {"kind": "batch", "nbeam": _log_int(rng, 3, 20), "mix": rng.randrange(1 << 20)}
    if kind == "rows":
        return {"kind": "rows", "dtype": rng.choice(["f32", "i32"]), "nrows": _log_int(rng, 32, 4000),
                "nsamp": _log_int(rng, 1000, 20000)}
    if kind in ("forward_u8", "detect_u8"):
        lofar = rng.random() < 0.6
        return {"kind": kind.split("_")[0], "dtype": "u8", "band": "lofar" if lofar else "apertif",
                "nbeam": rng.choice([1, 1, 1, 2]), "nchan": _log_int(rng, 16, 48) if lofar else _log_int(rng, 128, 1024),
                "ndm": _log_int(rng, 32, 1024), "nsamp": _log_int(rng, 4000, 200000) if lofar else _log_int(rng, 1000, 20000),
                **({"weighted": False} if kind == "forward_u8" else {})}
    small = rng.random() < 0.25
    case = {"kind": kind, "band": "test" if small else "apertif", "nbeam": rng.choice([1, 1, 2, 3]),
            "nchan": _log_int(rng, 48, 256) if small else _log_int(rng, 256, 1536),
            "ndm": _log_int(rng, 24, 256) if small else _log_int(rng, 64, 2048), "nsamp": _log_int(rng, 1000, 20000)}
    if kind == "train":
        case["ndm"] = min(case["ndm"], 1024)
    else:
        case["dtype"] = "f32"
    if kind == "forward":
        case["weighted"] = rng.random() < 0.4
    return case


# ---------------------------------------------------------------------------
# What a user's program has in hand.
# ---------------------------------------------------------------------------
def _setup(band, nchan, ndm):
    lo, hi, tsamp, step = BANDS[band]
    freqs = lo + (np.arange(nchan, dtype=np.float64) + 0.5) * (hi - lo) / nchan
    return freqs, tsamp, np.arange(ndm, dtype=np.float64) * step


def _beams_of(case):
    """The uneven beams of a batch: channels, DM trials and samples of each."""
    rng = np.random.default_rng(case["mix"])
    return [(int(rng.choice([256, 512, 1024, 1536])), int(rng.integers(512, 4096, endpoint=True)),
             int(rng.integers(8000, 20000, endpoint=True))) for _ in range(case["nbeam"])]


def _delays(freqs, tsamp, dms):
    """Delays in samples, [ndm][nchan]: 4150 DM (1/f^2 - 1/fmax^2) s, rounded half up."""
    k = 4150.0 * dms[:, None] * (1.0 / freqs ** 2 - 1.0 / freqs.max() ** 2)[None, :]
    return np.floor(k / tsamp + 0.5).astype(np.int64)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1601 + int(seed))
    return g


def _noise(shape, dtype, g):
    """Rows as a receiver delivers them: unit noise, or 8-bit samples around 128 with a spread of 16."""
    t = dd.empty_rows(*shape, {"f32": torch.float32, "u8": torch.uint8, "i32": torch.int32}[dtype], "cuda")
    n = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    if dtype == "u8":
        n = n.mul_(16.0).add_(128.0).round_().clamp_(0, 255)
    elif dtype == "i32":  # sums of 32 such samples
        n = n.mul_(16.0 * math.sqrt(32.0)).add_(128.0 * 32.0).round_()
    t.copy_(n)
    return t


def _weights(nchan, g):
    """A smooth bandpass with a twentieth of the channels masked."""
    w = 1.0 + 0.1 * torch.randn(nchan, generator=g, device="cuda", dtype=torch.float32)
    w[torch.randperm(nchan, generator=g, device="cuda")[:nchan // 20]] = 0.0
    return w


def _pulse(x, delta, nsamp, g):
    """One dispersed boxcar pulse per beam (width 4, amplitude of a strong burst)."""
    nbeam, nchan, _ = x.shape
    at = torch.rand((nbeam, 2), generator=g, device="cuda").cpu().tolist()
    c = torch.arange(nchan, device="cuda")
    for b, (u, v) in enumerate(at):
        d = torch.from_numpy(delta[int(u * delta.shape[0])]).cuda()
        for k in range(4):
            s = int(v * max(1, nsamp - 4)) + k
            if x.dtype == torch.uint8:
                x[b, c, s + d] = (x[b, c, s + d].int() + 24).clamp_(max=255).to(torch.uint8)
            else:
                x[b, c, s + d] += 1.0


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "rows":
        return {"kind": kind, "rows": _noise((1, case["nrows"], case["nsamp"]), case["dtype"], g)[0]}
    if kind == "batch":
        plans, xs, outs = [], [], []
        for nchan, ndm, nsamp in _beams_of(case):
            freqs, tsamp, dms = _setup("apertif", nchan, ndm)
            plans.append(dd.Plan(freqs, tsamp, dms))
            xs.append(_noise((1, nchan, nsamp + plans[-1].max_delay), "f32", g))
            _pulse(xs[-1], plans[-1].delays().astype(np.int64), nsamp, g)
            outs.append(dd.empty_rows(1, ndm, nsamp, torch.float32, "cuda"))
        return {"kind": kind, "batch": dd.Batch(plans, xs, outs), "xs": xs, "outs": outs}
    freqs, tsamp, dms = _setup(case["band"], case["nchan"], case["ndm"])
    plan = dd.Plan(freqs, tsamp, dms)
    dtype = case.get("dtype", "f32")
    plan.prepare(dtype)
    x = _noise((case["nbeam"], case["nchan"], case["nsamp"] + plan.max_delay), dtype, g)
    _pulse(x, plan.delays().astype(np.int64), case["nsamp"], g)
    state = {"kind": kind, "plan": plan, "x": x, "nsamp": case["nsamp"], "w": None}
    if kind == "train":
        plan.prepare("f32", adjoint=True)
        state["x"] = x.requires_grad_(True)
        state["w"] = _weights(case["nchan"], g).requires_grad_(True)
        state["g"] = _noise((case["nbeam"], case["ndm"], case["nsamp"]), "f32", g).mul_(1e-3)
    elif case.get("weighted"):
        state["w"] = _weights(case["nchan"], g)
    return state


def run(state):
    kind = state["kind"]
    if kind == "rows":
        return dd.detect_rows(state["rows"])
    if kind == "batch":
        state["batch"].execute()
        return state["outs"]
    if kind == "detect":
        return dd.detect(state["x"], state["plan"], nsamp=state["nsamp"])
    if kind == "train":
        out = dd.dedisperse_autograd(state["x"], state["plan"], state["w"], state["nsamp"])
        grad_x, grad_w = torch.autograd.grad(out, (state["x"], state["w"]), state["g"])
        return {"out": out.detach(), "grad_x": grad_x, "grad_w": grad_w}
    return dd.dedisperse(state["x"], state["plan"], state["w"], nsamp=state["nsamp"])


def work(case):
    """Each input read once, each output written once; one addition per (channel, DM trial, sample)."""
    kind = case["kind"]
    if kind == "rows":
        n, s = case["nrows"], case["nsamp"]
        return {"bytes": 4 * n * s + 32 * n, "flops": 2 * n * s}
    if kind == "batch":
        beams = [("apertif", 1, *b) for b in _beams_of(case)]
    else:
        beams = [(case["band"], case["nbeam"], case["nchan"], case["ndm"], case["nsamp"])]
    size = 1 if case.get("dtype") == "u8" else 4
    nbytes = flops = 0
    for band, nbeam, nchan, ndm, nsamp in beams:
        nin = nsamp + int(_delays(*_setup(band, nchan, ndm))[-1].max())
        series = nbeam * ndm * nsamp
        nbytes += nbeam * nchan * nin * size + 4 * nchan * ndm
        nbytes += 32 * nbeam * ndm if kind == "detect" else 4 * series
        flops += series * nchan
        if kind == "train":  # the output gradient is read, the input gradient written
            nbytes += 4 * series + 4 * nbeam * nchan * nin + 8 * nchan
            flops += series * nchan
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits, from the definitions alone.
# ---------------------------------------------------------------------------
def _series(x, delta, nsamp, w):
    """sum over channels of w[c] x[c][t + delta[dm][c]] for one beam, [ndm][nsamp]."""
    wide = torch.int64 if x.dtype == torch.uint8 else torch.float64
    out = torch.zeros((delta.shape[0], nsamp), dtype=wide, device=x.device)
    for c in range(x.shape[0]):
        row = x[c].to(wide) if w is None else x[c].to(wide) * w[c].to(wide)
        out += row.unfold(0, nsamp, 1)[delta[:, c]]
    return out


def _transpose(g, delta, nin, nchan):
    """sum over DM trials of g[dm][t - delta[dm][c]] for one beam, [nchan][nin]."""
    ndm, nsamp = g.shape
    top = nin - nsamp
    wide = torch.zeros((ndm, nsamp + 2 * top), dtype=torch.float64, device=g.device)
    wide[:, top:top + nsamp] = g.double()
    t = torch.arange(nin, device=g.device)
    out = torch.empty((nchan, nin), dtype=torch.float64, device=g.device)
    for c in range(nchan):
        out[c] = wide.gather(1, t[None, :] + (top - delta[:, c])[:, None]).sum(0)
    return out


def _search(y):
    """Boxcar search of series [n][nsamp]: S/N, mean and standard deviation in 64 bits."""
    y = y.double()
    nsamp = y.shape[1]
    mean, std = y.mean(1), y.std(1, correction=0)
    best = torch.full_like(mean, -math.inf)
    total = torch.nn.functional.pad(y.cumsum(1), (1, 0))
    for k in range(6):
        width = 1 << k
        if width <= nsamp:
            top = (total[:, width:] - total[:, :-width]).amax(1) if k else y.amax(1)
            best = torch.maximum(best, (top - width * mean) / (std * math.sqrt(width)))
    return {"snr": torch.where(std > 0, best, torch.zeros_like(best)), "width": None, "start": None, "mean": mean,
            "std": std}


def exact(case, seed):
    state = prepare(case, seed)
    kind = case["kind"]
    if kind == "rows":
        parts = [_search(p) for p in state["rows"].split(256)]
        return {k: None if parts[0][k] is None else torch.cat([p[k] for p in parts]) for k in parts[0]}
    if kind == "batch":
        outs = []
        for x, (nchan, ndm, nsamp) in zip(state["xs"], _beams_of(case)):
            delta = torch.from_numpy(_delays(*_setup("apertif", nchan, ndm))).cuda()
            outs.append(_series(x[0], delta, nsamp, None)[None])
        return outs
    delta = torch.from_numpy(_delays(*_setup(case["band"], case["nchan"], case["ndm"]))).cuda()
    x, nsamp = state["x"].detach(), case["nsamp"]
    w = None if state["w"] is None else state["w"].detach()
    if kind == "detect":
        beams = []
        for b in range(case["nbeam"]):
            step = max(1, (1 << 28) // nsamp)
            parts = [_search(_series(x[b], d, nsamp, None)) for d in delta.split(step)]
            beams.append({k: None if parts[0][k] is None else torch.cat([p[k] for p in parts]) for k in parts[0]})
        return {k: None if beams[0][k] is None else torch.stack([q[k] for q in beams]) for k in beams[0]}
    out = torch.stack([_series(x[b], delta, nsamp, w) for b in range(case["nbeam"])])
    if kind != "train":
        return out
    nin = x.shape[-1]
    back = torch.stack([_transpose(state["g"][b], delta, nin, case["nchan"]) for b in range(case["nbeam"])])
    grad_w = torch.zeros(case["nchan"], dtype=torch.float64, device="cuda")
    for b in range(case["nbeam"]):
        grad_w += (x[b].double() * back[b]).sum(1)
    return {"out": out, "grad_x": back * w.double()[None, :, None], "grad_w": grad_w}

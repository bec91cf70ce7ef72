"""Performance cases of the PVFinder path, through the library's public calls.

One pass is one call on one batch of events: track network and histogram,
UNet, peak finder.  The library has no entry point for a single layer, so
every case is a whole call; what varies is what a caller chooses: the number
of events (one event, where latency and launches count, up to the largest
batches), the track-count mix, the compute type, the network's width, the
UNet's layout, and the way of calling (eager, as a captured graph, or with
the library's own scratch).

Inputs are synthetic, as no detector data or trained weights are public:
events with Poisson(5.6) vertices and Poisson(180) or log-normal track counts,
He-normal weights and uniform biases.

A pass returns the probability rows and the status words, and in the 16- and
8-bit types the vertex lists too.  In FP32 the lists are left out: whether a
bin is a vertex is a comparison of neighbouring probabilities, and where two
of them agree to FP32 rounding the rounding decides it (in these untrained
networks, with some 1400 vertices an event, that happens in most batches).
The rows from which the vertices follow come back whole.
"""

import functools
import math
import struct

import numpy as np
import torch
import torch.nn.functional as F

import paper_2602_19959_amd as pv

N_BINS, BINS, N_INTERVALS = 4000, 100, 40
Z_MIN, INTERVAL_MM = -100.0, 10.0
HIDDEN, N_HIDDEN, TAPS = 20, 6, 5
MAX_TRACKS = 1500
SLOPE = float(np.float32(0.01))
S_IN = 1.0 / 32.0
SHIFT = np.float32([0, 0, 0, 0.0564, 0.0564, 0.0564, 0, 0, 0])
SCALE = np.float32([1, 1 / 0.064, 1 / 0.064, 1 / 0.030, 1 / 0.030, 1 / 0.030, 1 / 0.2, 1 / 0.2, 1 / 0.2])
# events whose working buffers fit the library's scratch (pvf_execute_scratch), 32 channels
SCRATCH_EVENTS = {"fp32": 8, "bf16": 17, "fp16": 17, "fp8_e4m3": 35}


def _case(name, dtype, events, mix="poisson", width=32, layout="event", boundary_mm=0.0, call="execute"):
    c = {"dtype": dtype, "events": events, "mix": mix, "width": width, "layout": layout,
         "boundary_mm": boundary_mm, "call": call}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the deployed precision, one event at a time: a caller with a latency budget per event
        _case("fp32_1", "fp32", 1),
        # a handful of events from code that may not allocate: the scratch's largest FP32 batch
        _case("fp32_8_scratch", "fp32", 8, call="scratch"),
        # a slice as a server packs it, of any size, with heavy-tailed track counts
        _case("fp32_333_tail", "fp32", 333, mix="lognormal"),
        # the trigger's production slice
        _case("fp32_1000", "fp32", 1000),
        # the wide network that the paper deploys, a small slice
        _case("fp32_w64_123", "fp32", 123, width=64),
        # one event in a serving loop, as one graph launch
        _case("bf16_1_graph", "bf16", 1, call="graph"),
        # the production slice in the mixed-precision path
        _case("bf16_1000", "bf16", 1000),
        # throughput batching: the largest batch, heavy-tailed, one graph launch a step
        _case("bf16_4096_tail_graph", "bf16", 4096, mix="lognormal", call="graph"),
        # the interval-batched layout with boundary tracks in two intervals
        _case("bf16_interval_250", "bf16", 250, layout="interval", boundary_mm=1.0),
        # FP16, a small odd batch
        _case("fp16_97", "fp16", 97),
        # FP8 with calibrated scales: the scratch's largest batch, and the production slice
        _case("fp8_35_scratch", "fp8_e4m3", 35, call="scratch"),
        _case("fp8_1000", "fp8_e4m3", 1000),
    ]


def draw(rng):
    dtype = rng.choice(["fp32", "fp32", "bf16", "bf16", "fp16", "fp8_e4m3"])
    width = rng.choice([32, 32, 32, 64])
    layout = rng.choice(["event", "event", "event", "interval"])
    boundary_mm = rng.choice([0.0, 0.0, 0.0, 0.5, 2.5])
    most = 1000 if dtype == "fp32" else 4096
    events = int(round(math.exp(rng.uniform(0.0, math.log(most // 4 if width == 64 else most)))))
    call = rng.choice(["execute", "execute", "execute", "graph", "scratch"])
    if call == "scratch" and (width == 64 or layout == "interval" or events > SCRATCH_EVENTS[dtype]):
        call = "execute"
    return _case(None, dtype, events, rng.choice(["poisson", "lognormal"]), width, layout, boundary_mm, call)


# ---------------------------------------------------------------- inputs


def _levels(case):
    return 3 if case["layout"] == "interval" else 4     # 100-bin sequences halve twice


def _tensors(case):
    """(name, shape, fan in) of every tensor, in the weight blob's order."""
    out = []
    dims = [9] + [HIDDEN] * N_HIDDEN + [BINS]
    for l in range(N_HIDDEN + 1):
        out += [(f"mlp{l}.w", (dims[l + 1], dims[l]), dims[l]), (f"mlp{l}.b", (dims[l + 1],), dims[l])]

    def conv(name, c, cin):
        return [(name + ".w", (c, cin, TAPS), cin * TAPS), (name + ".b", (c,), cin * TAPS)]

    n, cin = _levels(case), 1
    for l in range(n):
        c = case["width"] << l
        out += conv(f"enc{l}.c1", c, cin) + conv(f"enc{l}.c2", c, c)
        cin = c
    for l in range(n - 2, -1, -1):
        c = case["width"] << l
        out += [(f"up{l}.w", (2 * c, c, 2), 2 * c), (f"up{l}.b", (c,), 2 * c)]
        out += conv(f"dec{l}.c1", c, 2 * c) + conv(f"dec{l}.c2", c, c)
    c = case["width"]
    return out + [("head.w", (1, c), c), ("head.b", (1,), c)]


def _weights(case, seed):
    g = np.random.default_rng([seed, 1])
    w = {}
    for name, shape, fan_in in _tensors(case):
        if name.endswith(".w"):
            v = g.standard_normal(shape, dtype=np.float32) * np.float32(math.sqrt(2.0 / fan_in))
        else:
            v = (2 * g.random(shape, dtype=np.float32) - 1) / np.float32(math.sqrt(fan_in))
        w[name] = np.ascontiguousarray(v, dtype=np.float32)
    return w


def _blob(case, w):
    names = [n for n, _, _ in _tensors(case)]
    head = b"PVFW" + struct.pack("<I7i2f", 1, 9, HIDDEN, N_HIDDEN, BINS, _levels(case), case["width"], TAPS, SLOPE, S_IN)
    head += SHIFT.tobytes() + SCALE.tobytes()
    head += struct.pack("<%di" % (len(names) + 1), len(names), *(w[n].size for n in names))
    return head + b"".join(w[n].tobytes() for n in names)


def _events(events, mix, seed):
    """float32 [9][T] track features and int32 [E+1] offsets, on the host."""
    g = np.random.default_rng([seed, 2])
    if mix == "poisson":
        counts = g.poisson(180.0, events)
    else:
        counts = np.clip(np.rint(g.lognormal(math.log(180.0), 1.0, events)), 5, MAX_TRACKS).astype(np.int64)
    n_pv = np.maximum(1, g.poisson(5.6, events))
    first = np.cumsum(n_pv) - n_pv                       # each event's first vertex
    total = int(n_pv.sum())
    vz = np.clip(g.normal(0.0, 45.0, total), -100.0, 300.0)
    vx, vy = g.normal(0.0, 0.04, total), g.normal(0.0, 0.04, total)
    offsets = np.concatenate([[0], np.cumsum(counts)])
    T = int(offsets[-1])
    event = np.repeat(np.arange(events), counts)
    v = first[event] + (g.random(T) * n_pv[event]).astype(np.int64)
    f = np.empty((9, T), np.float32)
    f[0] = vz[v] + g.normal(0.0, 0.1, T)
    f[1] = vx[v] + g.normal(0.0, 0.05, T)
    f[2] = vy[v] + g.normal(0.0, 0.05, T)
    f[3:6] = np.exp(g.normal(-3.0, 0.5, (3, T)))
    f[6:9] = g.normal(0.0, 0.2, (3, T))
    return f, offsets.astype(np.int32)


def _spec(case, dtype, events):
    return pv.default_spec(max_events=events, max_tracks_total=events * MAX_TRACKS, compute_dtype=dtype,
                           n_levels=_levels(case), base_channels=case["width"], unet_layout=case["layout"],
                           boundary_mm=case["boundary_mm"])


def prepare(case, seed):
    blob = _blob(case, _weights(case, seed))
    amax = None
    if case["dtype"] == "fp8_e4m3":                      # channel scales from other events, in BF16
        f, o = _events(32, "lognormal", seed + (1 << 32))
        eng = pv.Engine(blob, _spec(case, "bf16", 32))
        amax = eng.calibrate(torch.from_numpy(f).cuda(), torch.from_numpy(o).cuda())
        eng.close()
    f, o = _events(case["events"], case["mix"], seed)
    feat, offsets = torch.from_numpy(f).cuda(), torch.from_numpy(o).cuda()
    eng = pv.Engine(blob, _spec(case, case["dtype"], case["events"]), fp8_amax=amax)
    out = eng.alloc_outputs(case["events"])
    torch.cuda.synchronize()
    if case["call"] == "graph":
        eng.graph_capture(feat, offsets, out)
    call = {"execute": functools.partial(eng.execute, feat, offsets, out),
            "scratch": functools.partial(eng.execute_scratch, feat, offsets, out),
            "graph": eng.graph_launch}[case["call"]]
    keys = ["prob", "status"]
    if case["dtype"] != "fp32":
        keys += ["n_vertices", "bin", "z", "peak_prob", "integral"]
    return {"engine": eng, "call": call, "out": {k: getattr(out, k) for k in keys}}


def run(state):
    state["call"]()
    return state["out"]


# ---------------------------------------------------------------- work, exact values


def work(case):
    """Track features in, weights in, probability rows and vertex counts out;
    the operations of the track network and of every convolution."""
    E = case["events"]
    tracks = E * (180.0 if case["mix"] == "poisson" else 280.0)
    n, units = _levels(case), N_INTERVALS if case["layout"] == "interval" else 1
    L0 = N_BINS // units
    macs = float(L0 * case["width"])
    cin = 1
    for l in range(n):
        L, C = L0 >> l, case["width"] << l
        macs += L * C * (cin + C) * TAPS
        if l < n - 1:
            macs += L * C * 2 * C + L * C * 3 * C * TAPS
        cin = C
    mlp = 9 * HIDDEN + (N_HIDDEN - 1) * HIDDEN * HIDDEN + HIDDEN * BINS
    eb = {"fp32": 4, "fp8_e4m3": 1}.get(case["dtype"], 2)
    params = sum(math.prod(s) for _, s, _ in _tensors(case))
    return {"bytes": 36.0 * tracks + 4.0 * E * (N_BINS + 3) + eb * params,
            "flops": 2.0 * (E * units * macs + tracks * mlp)}


def _histogram(w, f, o, boundary_mm):
    E = len(o) - 1
    hist = torch.zeros(E * N_BINS, dtype=torch.float64, device="cuda")
    f, o = torch.from_numpy(f).cuda().double(), torch.from_numpy(o).cuda().long()
    event = torch.repeat_interleave(torch.arange(E, device="cuda"), o.diff())
    z = f[0]
    i = torch.floor((z - Z_MIN) / INTERVAL_MM).long()
    inside = (i >= 0) & (i < N_INTERVALS)
    feeds = [(i, inside)]
    if boundary_mm > 0:
        lo = Z_MIN + INTERVAL_MM * i
        feeds += [(i - 1, inside & (z - lo < boundary_mm) & (i > 0)),
                  (i + 1, inside & (lo + INTERVAL_MM - z < boundary_mm) & (i < N_INTERVALS - 1))]
    g = (f - torch.from_numpy(SHIFT).cuda().double()[:, None]) * torch.from_numpy(SCALE).cuda().double()[:, None]
    for at, use in feeds:
        k = at[use]
        x = g[:, use].T.contiguous()
        x[:, 0] = (z[use] - (Z_MIN + INTERVAL_MM * k)) / (INTERVAL_MM / 2) - 1
        for l in range(N_HIDDEN):
            x = F.leaky_relu(F.linear(x, w[f"mlp{l}.w"], w[f"mlp{l}.b"]), SLOPE)
        y = F.softplus(F.linear(x, w[f"mlp{N_HIDDEN}.w"], w[f"mlp{N_HIDDEN}.b"]))
        cell = (event[use] * N_BINS + k * BINS)[:, None] + torch.arange(BINS, device="cuda")
        hist.index_add_(0, cell.reshape(-1), y.reshape(-1))
    return hist.reshape(E, N_BINS)


def _conv(w, name, x):
    """x [sequences][L][Cin] -> [sequences][L][Cout], zero padding, LeakyReLU."""
    n, L, cin = x.shape
    k = w[name + ".w"]
    p = F.pad(x, (0, 0, TAPS // 2, TAPS // 2))
    y = w[name + ".b"].expand(n * L, -1).clone()
    for j in range(TAPS):
        y.addmm_(p[:, j:j + L].reshape(n * L, cin), k[:, :, j].T.contiguous())
    return F.leaky_relu(y, SLOPE).reshape(n, L, -1)


def _unet(case, w, x):
    n, skips = _levels(case), []
    for l in range(n):
        x = _conv(w, f"enc{l}.c2", _conv(w, f"enc{l}.c1", x))
        if l < n - 1:
            skips.append(x)
            x = torch.maximum(x[:, 0::2], x[:, 1::2])
    for l in range(n - 2, -1, -1):
        s, L, cin = x.shape
        k = w[f"up{l}.w"]                                # [Cin][Cout][2]
        u = torch.stack([x.reshape(s * L, cin) @ k[:, :, j].contiguous() for j in (0, 1)], 1) + w[f"up{l}.b"]
        x = torch.cat([skips[l], u.reshape(s, 2 * L, -1)], 2)
        x = _conv(w, f"dec{l}.c2", _conv(w, f"dec{l}.c1", x))
    return torch.sigmoid(x @ w["head.w"][0] + w["head.b"])


def exact(case, seed):
    """The probability rows in 64 bits; the lists that follow from them have no value apart from their type's rounding."""
    w = {k: torch.from_numpy(v).cuda().double() for k, v in _weights(case, seed).items()}
    f, o = _events(case["events"], case["mix"], seed)
    h = _histogram(w, f, o, case["boundary_mm"]) * S_IN
    x = h.reshape(-1, BINS if case["layout"] == "interval" else N_BINS, 1)
    step = 64 * N_BINS // x.shape[1]
    rows = [_unet(case, w, x[k:k + step]) for k in range(0, x.shape[0], step)]
    keys = ["status"] if case["dtype"] == "fp32" else ["status", "n_vertices", "bin", "z", "peak_prob", "integral"]
    return {"prob": torch.cat(rows).reshape(case["events"], N_BINS), **dict.fromkeys(keys)}

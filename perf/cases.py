"""Performance cases of the trigger-station selection.

Each case is one call (or one short chain of calls) that a program using this
library makes: the triplet selection over batches from a thousand to a million
events in its execution forms, the station filter, event building, the three
in a row, and the serving runtime on host data.  Inputs follow the recipe of
``paper_1810_11966_amd/synth.py`` (uniform noise in the station's annulus,
Poisson multiplicities, injected muon pairs, staggered modules, free-streaming
times), drawn on the GPU so that they are quick to make.

    listed()             the cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs and buffers, on the GPU (serving: on the host)
    run(state)           one pass, returns every output
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the outputs from float64 arithmetic in plain torch
"""
from __future__ import annotations

import math

import torch

from paper_1810_11966_amd import events, filter as stations, serve, trig

R_MIN, R_MAX = 20.0, 200.0          # the station's annulus, cm
Z = (400.0, 410.0, 420.0)           # layer positions, cm
N_STATIONS = 16
LAYERS = (13, 14, 15)               # station numbers of the trigger layers
MSD_MAX = (0.03, 0.025)
NDF = 2
WINDOW = 0.005
STAGGER = 0.75                      # module offset of the per-hit-z sets, cm


# ------------------------------------------------------------------ cases ---

def _select(name, n_events, hits_mean, form, test="msd", mixture=False, compact=True, two=False, decision=False,
            hit_z=False, p_inject=0.01, pairs_max=1, binding="call"):
    return {"name": name, "kind": "select", "n_events": n_events, "hits_mean": float(hits_mean), "mixture": mixture,
            "form": form, "test": test, "compact": compact, "two": two, "decision": decision, "hit_z": hit_z,
            "p_inject": p_inject, "pairs_max": pairs_max, "binding": binding}


def listed():
    return [
        # The smallest batch of the paper's Table 1: 1000 events of about 15
        # hits per layer.  A trigger node with little data per call: latency
        # and the number of launches.
        _select("select_small_1k", 1_000, 15, "pruned", p_inject=0.05),
        # The binding's default call: every triplet tested, outputs allocated
        # by the call.
        _select("select_plain_100k", 100_000, 30, "plain", compact=False, binding="default"),
        # The headline batch: a million events of 30 hits per layer, the
        # autotuned form with the list of accepted events.
        _select("select_medium_1m", 1_000_000, 30, "auto"),
        # Minimum-bias-like, very uneven events, autotuned.
        _select("select_mixture_1m", 1_000_000, 120, "auto", mixture=True),
        # High multiplicity: 200 hits per layer, slope-cell binning.
        _select("select_dense_100k", 100_000, 200, "binned", p_inject=0.10, pairs_max=3),
        # The slope-window test with the two-particle acceptance.
        _select("select_window_two_300k", 300_000, 30, "pruned", test="window", two=True),
        # Staggered modules: every hit carries its own z.
        _select("select_hit_z_1m", 1_000_000, 30, "pruned", compact=False, hit_z=True, binding="default"),
        # All of an event's hits (about 5000 on 16 stations, detector order)
        # down to the trigger layers.
        {"name": "filter_100k", "kind": "filter", "n_events": 100_000, "other_mean": 378.0, "shuffle": False},
        # The same with the stations in random order within each event.
        {"name": "filter_shuffled_5k", "kind": "filter", "n_events": 5_003, "other_mean": 378.0, "shuffle": True},
        # A free-streaming timeslice of 100 million hits cut into events.
        {"name": "build_100m", "kind": "build", "n_events": 20_000, "other_mean": 378.0},
        # A small timeslice through the whole device path: event building,
        # station filter, selection; the program reads the number of events
        # and of accepted ones, as it must to go on.
        {"name": "chain_2k", "kind": "chain", "n_events": 2_000, "other_mean": 378.0},
        # Serving: six host timeslices of different sizes handed over
        # together, all results collected on the host.
        {"name": "serve_6", "kind": "serve", "n_slices": 6, "min_events": 10_000, "max_events": 150_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("select", "filter", "build", "chain", "serve"), (12, 3, 3, 1, 1))[0]
    if kind == "select":
        hit_z = rng.random() < 0.15
        form = rng.choice(("plain", "pruned", "pruned", "binned", "persistent", "persistent_pruned",
                           "persistent_binned", "auto"))
        test = rng.choice(("msd", "msd", "window", "msd_basis"))
        if hit_z and test == "msd_basis":
            test = "msd"  # not provided with per-hit z
        if hit_z and form == "auto":
            form = "pruned"
        mixture = rng.random() < 0.25
        mean = math.exp(rng.uniform(math.log(2.0), math.log(240.0)))
        most = min(1_000_000, int(90e6 / (3 * mean)))
        if form in ("plain", "persistent"):  # every triplet: no more of them than the listed case has
            most = min(most, int(2.7e9 / mean ** 3))
            if hit_z:
                most = max(1, most // 4)
        n = min(_log_int(rng, 100, 1_000_000), max(most, 1))
        two = rng.random() < 0.2
        return _select("", n, mean, form, test=test, mixture=mixture, compact=rng.random() < 0.7, two=two,
                       decision=rng.random() < 0.15, hit_z=hit_z, p_inject=rng.choice((0.01, 0.05, 0.1)),
                       pairs_max=rng.choice((1, 3)))
    if kind == "filter":
        shuffle = rng.random() < 0.4
        mean = math.exp(rng.uniform(math.log(4.0), math.log(500.0)))
        most = int((26e6 if shuffle else 500e6) / (13 * mean + 90))
        return {"kind": "filter", "n_events": min(_log_int(rng, 20, 100_000), most), "other_mean": mean,
                "shuffle": shuffle}
    if kind == "build":
        mean = math.exp(rng.uniform(math.log(20.0), math.log(500.0)))
        most = int(100e6 / (13 * mean + 90))
        return {"kind": "build", "n_events": min(_log_int(rng, 10, 100_000), most), "other_mean": mean}
    if kind == "chain":
        return {"kind": "chain", "n_events": _log_int(rng, 100, 5_000), "other_mean": rng.uniform(100.0, 400.0)}
    lo = _log_int(rng, 500, 10_000)
    return {"kind": "serve", "n_slices": rng.randint(1, 6), "min_events": lo,
            "max_events": lo + _log_int(rng, 1_000, 100_000)}


# ----------------------------------------------------------------- inputs ---

def _generator(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _rand(n, g, dtype=torch.float32):
    return torch.rand(n, generator=g, device="cuda", dtype=dtype)


def _annulus(n, g):
    r = torch.sqrt_(_rand(n, g).mul_(R_MAX ** 2 - R_MIN ** 2).add_(R_MIN ** 2))
    phi = _rand(n, g).mul_(2 * math.pi)
    x = torch.cos(phi).mul_(r)
    y = torch.sin_(phi).mul_(r)
    return x, y


def _trigger_events(n, hits_mean, mixture, p_inject, pairs_max, g):
    """int64 offsets[3n+1], fp32 x, y: noise and muon pairs (sigma 0.3 cm)."""
    lam = torch.full((n, 1), hits_mean, device="cuda")
    if mixture:
        b = _rand(n, g)[:, None]
        lam = hits_mean * (1.0 - b * b)
    cnt = torch.poisson(lam.expand(n, 3).contiguous(), generator=g).to(torch.int64)
    pairs = torch.randint(1, pairs_max + 1, (n,), generator=g, device="cuda")
    ntr = torch.where(_rand(n, g) < p_inject, 2 * pairs, torch.zeros_like(pairs))
    cnt += ntr[:, None]
    off = torch.zeros(3 * n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(cnt.reshape(-1), 0, out=off[1:])
    x, y = _annulus(int(off[-1]), g)
    ev = torch.repeat_interleave(torch.arange(n, device="cuda"), ntr)
    m = ev.numel()
    rank = torch.arange(m, device="cuda") - (torch.cumsum(ntr, 0) - ntr)[ev]
    tmin, tmax = R_MIN / min(Z), R_MAX / max(Z)
    cmax, cmin = 1 / math.sqrt(1 + tmin * tmin), 1 / math.sqrt(1 + tmax * tmax)
    cos_t = _rand(m, g, torch.float64) * (cmax - cmin) + cmin
    tan_t = torch.sqrt(1 - cos_t * cos_t) / cos_t
    phi = _rand(m, g, torch.float64) * (2 * math.pi)
    shift = _rand(n, g, torch.float64)
    for layer in range(3):
        # the event's tracks take consecutive slots of the layer from a random one on
        nl = cnt[ev, layer]
        slot = ((shift[ev] * nl).to(torch.int64) + rank) % nl
        pos = off[3 * ev + layer] + slot
        smear = torch.randn(2, m, generator=g, device="cuda", dtype=torch.float64) * 0.3
        x[pos] = (tan_t * torch.cos(phi) * Z[layer] + smear[0]).float()
        y[pos] = (tan_t * torch.sin(phi) * Z[layer] + smear[1]).float()
    return off, x, y


def _layer_of_hit(off):
    per = off[1:] - off[:-1]
    layer = torch.arange(3, device="cuda", dtype=torch.uint8).repeat(per.numel() // 3)
    return torch.repeat_interleave(layer, per, output_size=int(off[-1] - off[0]))


def _stagger(off, x, y):
    """Hits moved along their line of sight to their module's z."""
    zl = torch.tensor(Z, device="cuda")[_layer_of_hit(off).long()]
    sector = torch.floor((torch.atan2(y, x) + math.pi) * (16 / (2 * math.pi))).long() % 16
    z = zl + torch.where(sector % 2 == 0, -STAGGER, STAGGER)
    f = z / zl
    return x * f, y * f, z


def _select_inputs(case, seed):
    g = _generator(seed, 1)
    off, x, y = _trigger_events(case["n_events"], case["hits_mean"], case["mixture"], case["p_inject"],
                                case["pairs_max"], g)
    z = None
    if case["hit_z"]:
        x, y, z = _stagger(off, x, y)
    return off.to(torch.int32), x, y, z


def _raw_events(n, other_mean, shuffle, g):
    """All-station events: int64 offsets[n+1], uint8 station, fp32 x, y."""
    lam = torch.full((n, N_STATIONS), other_mean, device="cuda")
    for s in LAYERS:
        lam[:, s] = 30.0
    cnt = torch.poisson(lam, generator=g).to(torch.int64)
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(cnt.sum(1), 0, out=off[1:])
    total = int(off[-1])
    number = torch.arange(N_STATIONS, device="cuda", dtype=torch.uint8).repeat(n)
    station = torch.repeat_interleave(number, cnt.reshape(-1), output_size=total)
    if shuffle:
        ev = torch.repeat_interleave(torch.arange(n, device="cuda"), off[1:] - off[:-1], output_size=total)
        station = station[torch.argsort(ev.double() + _rand(total, g, torch.float64))]
    x, y = (_rand(total, g).mul_(2 * R_MAX).sub_(R_MAX) for _ in range(2))
    return off, station, x, y


def _capacity(n):
    """Length of a program's trigger-hit buffers for n events: Poisson(90)
    hits per event and ten standard deviations."""
    return int(90 * n + 10 * math.sqrt(90 * n)) + 64


def _times(off, g, apart=0):
    """int64 time of each hit, ns: interactions at 10 MHz (each at least
    `apart` after the one before), hits up to 10 ns later; not yet in time
    order."""
    n = off.numel() - 1
    dt = torch.empty(n, dtype=torch.float64, device="cuda").exponential_(1.0 / 100.0, generator=g).round_()
    start = torch.cumsum(dt.long() + apart, 0)
    total = int(off[-1])
    t = torch.repeat_interleave(start, off[1:] - off[:-1], output_size=total)
    return t + torch.randint(0, 11, (total,), generator=g, device="cuda")


GAP_NS = 5


def _stream(case, seed):
    g = _generator(seed, 3)
    off, station, x, y = _raw_events(case["n_events"], case["other_mean"], False, g)
    t, order = torch.sort(_times(off, g, apart=10 + GAP_NS + 1), stable=True)  # no pile up
    return t, station[order], x[order], y[order]


def _build_times(case, seed):
    g = _generator(seed, 4)
    lam = torch.full((case["n_events"],), 13 * case["other_mean"] + 90.0, device="cuda")
    off = torch.zeros(case["n_events"] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.poisson(lam, generator=g).long(), 0, out=off[1:])
    return torch.sort(_times(off, g))[0]


def _slices(case, seed):
    """Host timeslices: sizes spread evenly over the case's range."""
    out = []
    for k in range(case["n_slices"]):
        f = (k + 0.5) / case["n_slices"]
        n = int(case["min_events"] + f * (case["max_events"] - case["min_events"]))
        off, x, y = _trigger_events(n, 30.0, False, 0.01, 1, _generator(seed, 10 + k))
        out.append((off.to(torch.int32).cpu().numpy(), x.cpu().numpy(), y.cpu().numpy()))
    return out


# ---------------------------------------------------------------- prepare ---

def _flags(case):
    extra = trig.TRIG_ACCEPT_TWO_PARTICLES if case["two"] else 0
    return extra | (trig.TRIG_DECISION_ONLY if case["decision"] else 0)


def _prepare_select(case, seed):
    off, x, y, z = _select_inputs(case, seed)
    st = {"case": case, "off": off, "x": x, "y": y, "z": z}
    if case["binding"] == "default":
        return st
    # The C call with its arguments marshalled once, on the program's own
    # buffers (the accepted ids past the accepted ones stay 0).
    n = case["n_events"]
    flags = trig.FORMS[case["form"]] | _flags(case) | (trig.TRIG_OUT_COMPACT if case["compact"] else 0)
    p = trig.make_params(test=case["test"], flags=flags)
    st["counts"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    st["accept"] = torch.zeros(n, dtype=torch.uint8, device="cuda")
    st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    p.out_status = st["status"].data_ptr()
    if case["compact"]:
        st["ids"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        st["n_accepted"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        p.out_accepted_ids = st["ids"].data_ptr()
        p.out_n_accepted = st["n_accepted"].data_ptr()
    need = trig.trig_workspace_bytes(n, p)
    st["workspace"] = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    p.workspace = (st["workspace"].data_ptr() + 255) & ~255
    p.workspace_bytes = need
    st["ev"] = trig.TrigEventsCsr(n, off.data_ptr())
    st["hits"] = trig.TrigHits(x.numel(), x.data_ptr(), y.data_ptr(), z.data_ptr() if z is not None else None)
    st["params"] = p
    if case["form"] == "auto":
        # the program tunes once per kind of batch
        rc, _ = trig.trig_autotune(st["ev"], st["hits"], p, st["counts"].data_ptr(), st["accept"].data_ptr(), 3,
                                   torch.cuda.current_stream().cuda_stream)
        if rc:
            raise trig.TrigError(rc, trig.trig_last_error_detail())
    return st


class _Server:
    """A serving runtime that is closed with its state."""

    def __init__(self, in_bytes):
        # staging for every slice's input and results at once
        self.server = serve.Server(hbm_budget_bytes=2 * in_bytes + (64 << 20),
                                   pinned_budget_bytes=2 * in_bytes + (16 << 20), n_streams=4)

    def __del__(self):
        self.server.close()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "select":
        return _prepare_select(case, seed)
    if kind == "filter":
        n = case["n_events"]
        off, station, x, y = _raw_events(n, case["other_mean"], case["shuffle"], _generator(seed, 2))
        # the program's own output buffers, of fixed capacity (0 past the hits)
        out = stations.FilterResult(torch.zeros(3 * n + 1, dtype=torch.int32, device="cuda"),
                                    torch.zeros(_capacity(n), device="cuda"),
                                    torch.zeros(_capacity(n), device="cuda"),
                                    torch.zeros(1, dtype=torch.int32, device="cuda"), None)
        ws = torch.empty(stations.workspace_bytes(n) + 256, dtype=torch.uint8, device="cuda")
        return {"case": case, "off": off, "station": station, "x": x, "y": y, "out": out, "workspace": ws}
    if kind == "build":
        t = _build_times(case, seed)
        cap = 4 * case["n_events"] + 16
        out = events.BuildResult(torch.zeros(cap, dtype=torch.int64, device="cuda"),
                                 torch.zeros(1, dtype=torch.int64, device="cuda"),
                                 torch.zeros(1, dtype=torch.int32, device="cuda"), None)
        ws = torch.empty(events.workspace_bytes(t.numel()) + 512, dtype=torch.uint8, device="cuda")
        return {"case": case, "t": t, "out": out, "workspace": ws}
    if kind == "chain":
        n = case["n_events"]
        t, station, x, y = _stream(case, seed)
        hits = stations.FilterResult(torch.zeros(3 * n + 1, dtype=torch.int32, device="cuda"),
                                     torch.zeros(_capacity(n), device="cuda"),
                                     torch.zeros(_capacity(n), device="cuda"),
                                     torch.zeros(1, dtype=torch.int32, device="cuda"), None)
        ws = torch.empty(stations.workspace_bytes(n) + 256, dtype=torch.uint8, device="cuda")
        return {"case": case, "t": t, "station": station, "x": x, "y": y, "hits": hits, "workspace": ws,
                "ids": torch.zeros(n, dtype=torch.int32)}
    slices = _slices(case, seed)
    return {"case": case, "slices": slices, "ids": [torch.zeros(len(a) // 3, dtype=torch.int32) for a, _, _ in slices],
            "server": _Server(sum(a.nbytes + b.nbytes + c.nbytes for a, b, c in slices))}


# -------------------------------------------------------------------- run ---

def _run_select(st):
    case = st["case"]
    if case["binding"] == "default":
        r = trig.select(st["off"], st["x"], st["y"], hit_z=st["z"], form=case["form"], test=case["test"])
        return r.counts, r.accept
    rc = trig.trig_select(st["ev"], st["hits"], st["params"], st["counts"].data_ptr(), st["accept"].data_ptr(),
                          torch.cuda.current_stream().cuda_stream)
    if rc:
        raise trig.TrigError(rc, trig.trig_last_error_detail())
    out = (st["counts"], st["accept"], st["status"])
    return out + (st["ids"], st["n_accepted"]) if case["compact"] else out


def _run_chain(st):
    n = st["case"]["n_events"]
    b = events.build_events(st["t"], GAP_NS, capacity=4 * n + 16)
    off = b.offsets[: int(b.n_events) + 1]
    f = stations.filter_stations(off, st["station"], st["x"], st["y"], LAYERS, _capacity(n), out=st["hits"],
                                 workspace=st["workspace"])
    r = trig.select(f.layer_offsets, f.x, f.y, form="pruned", compact=True)
    n_accepted = int(r.n_accepted)
    st["ids"][:n_accepted] = r.ids[:n_accepted].cpu()  # the list of accepted events, on the host
    return off, f.layer_offsets, f.x, f.y, r.counts, r.accept, n_accepted, st["ids"]


def _run_serve(st):
    server = st["server"].server
    place, done = {}, {}
    for k, (off, x, y) in enumerate(st["slices"]):
        t = server.submit(off, x, y)
        while t is None:  # busy: take a result, then try again
            f = server.poll(1)
            if f is not None:
                done[f.ticket] = f
            t = server.submit(off, x, y)
        place[t] = k
    while len(done) < len(st["slices"]):
        f = server.poll(1000)
        if f is not None:
            done[f.ticket] = f
    out = [None] * len(st["slices"])
    for t, f in done.items():
        k = place[t]
        st["ids"][k][: len(f.ids)] = torch.from_numpy(f.ids)
        out[k] = (f.status, f.counts, f.accept, len(f.ids), st["ids"][k])
    return out


def run(state):
    kind = state["case"]["kind"]
    if kind == "select":
        return _run_select(state)
    if kind == "filter":
        f = stations.filter_stations(state["off"], state["station"], state["x"], state["y"], LAYERS,
                                     _capacity(state["case"]["n_events"]), out=state["out"],
                                     workspace=state["workspace"])
        return f.layer_offsets, f.x, f.y, f.status
    if kind == "build":
        b = events.build_events(state["t"], GAP_NS, out=state["out"], workspace=state["workspace"])
        return b.offsets, b.n_events, b.status
    if kind == "chain":
        return _run_chain(state)
    return _run_serve(state)


# ------------------------------------------------------------------- work ---

def _select_work(n, hits, compact, hit_z):
    """Offsets and hits in; counts and flags out; the slope of each hit in
    both planes."""
    return {"bytes": 17.0 * n + (12.0 if hit_z else 8.0) * hits + (4.0 if compact else 0.0), "flops": 2.0 * hits}


def _raw_hits(case):
    return case["n_events"] * (13 * case["other_mean"] + 90.0)


def work(case):
    kind = case["kind"]
    n = case.get("n_events", 0)
    if kind == "select":
        mean = case["hits_mean"] * (2.0 / 3.0 if case["mixture"] else 1.0)
        mean += case["p_inject"] * (1 + case["pairs_max"])
        w = _select_work(n, 3 * mean * n, case["compact"], case["hit_z"])
        if case["form"] in ("plain", "persistent"):
            # every triplet tested: at least a sum and a comparison for each
            w["flops"] = 2.0 * n * case["hits_mean"] ** 3 * (0.457 if case["mixture"] else 1.0)
        return w
    if kind == "filter":
        return {"bytes": 20.0 * n + _raw_hits(case) + 16.0 * 90.0 * n, "flops": 0.0}
    if kind == "build":
        return {"bytes": 8.0 * _raw_hits(case) + 8.0 * n, "flops": 0.0}
    if kind == "chain":
        sel = _select_work(n, 90.0 * n, True, False)
        return {"bytes": 8.0 * _raw_hits(case) + 8.0 * n + 20.0 * n + _raw_hits(case) + 16.0 * 90.0 * n +
                sel["bytes"], "flops": sel["flops"]}
    total = case["n_slices"] * 0.5 * (case["min_events"] + case["max_events"])
    return _select_work(total, 90.0 * total, True, False)


# ------------------------------------------------------------------ exact ---

_EXACT_PAIRS = 6e9  # padded layer-0 x layer-1 pairs beyond which exact() takes too long


def _pad(v, off, layer, e0, e1, width):
    """Layer hits of events [e0, e1) as [e1 - e0, width] float64, NaN-padded."""
    s, t = off[3 * e0 + layer:3 * e1 + layer:3], off[3 * e0 + layer + 1:3 * e1 + layer + 1:3]
    i = s[:, None] + torch.arange(width, device=v.device)[None, :]
    ok = i < t[:, None]
    return torch.where(ok, v[torch.where(ok, i, 0)].double(), math.nan)


def _exact_counts(off, x, y, z, test):
    """Passing triplets per event in float64: pairs that can pass (the part
    of the residual sum that depends on the pair, or the layer-1 window),
    then every layer-2 hit of the event for each of them."""
    off = off.long()
    n = (off.numel() - 1) // 3
    per = (off[1:] - off[:-1]).reshape(n, 3)
    widths = [max(int(per[:, layer].max()), 1) for layer in range(3)]
    if float(n) * widths[0] * widths[1] > _EXACT_PAIRS:
        return None
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # the library's parameters are binary32
    counts = torch.zeros(n, dtype=torch.int64, device=x.device)
    step = max(1, int(6e7 / (widths[0] * widths[1])))
    for e0 in range(0, n, step):
        e1 = min(n, e0 + step)
        c = [[_pad(v, off, layer, e0, e1, widths[layer]) for layer in range(3)] for v in (x, y)]
        if z is None:
            zs = [torch.full_like(c[0][layer], Z[layer]) for layer in range(3)]
        else:
            zs = [_pad(z, off, layer, e0, e1, widths[layer]) for layer in range(3)]
        ok = None
        for v, cut in zip(c, MSD_MAX):
            si, sj = v[0] / zs[0], v[1] / zs[1]
            d = (sj[:, None, :] - si[:, :, None]).abs_()
            if test == "window":
                m = d < f32(WINDOW)
            else:
                # |c_i/z_i - c_j/z_j| = |r_i/z_i - r_j/z_j| <= |r| sqrt(1/z_i^2 + 1/z_j^2)
                m = d <= math.sqrt(f32(cut) * NDF) * math.sqrt(2.0) / (min(Z) - STAGGER) * (1 + 1e-9)
            ok = m if ok is None else ok & m
        e, i, j = torch.nonzero(ok, as_tuple=True)
        for a in range(0, e.numel(), 1 << 20):
            ee, ii, jj = e[a:a + (1 << 20)], i[a:a + (1 << 20)], j[a:a + (1 << 20)]
            good = None
            z0, z1, z2 = zs[0][ee, ii][:, None], zs[1][ee, jj][:, None], zs[2][ee]
            for v, cut in zip(c, MSD_MAX):
                c0, c1, c2 = v[0][ee, ii][:, None], v[1][ee, jj][:, None], v[2][ee]
                if test == "window":
                    m = (c2 / z2 - c0 / z0).abs() < f32(WINDOW)
                else:
                    slope = (c0 * z0 + c1 * z1 + c2 * z2) / (z0 * z0 + z1 * z1 + z2 * z2)
                    q = (c0 - slope * z0) ** 2 + (c1 - slope * z1) ** 2 + (c2 - slope * z2) ** 2
                    m = q / NDF <= f32(cut)
                good = m if good is None else good & m
            counts.index_add_(0, ee + e0, good.sum(1))
    return counts.int()


def _accepted(counts, two):
    return None if counts is None or two else (counts >= 2).to(torch.uint8)


def _padded_ids(accept):
    found = torch.nonzero(accept)[:, 0].int()
    return torch.nn.functional.pad(found, (0, accept.numel() - found.numel()))


def _exact_filter(off, station, x, y):
    n = off.numel() - 1
    layer = torch.full((256,), 3, dtype=torch.uint8, device=off.device)
    for k, s in enumerate(LAYERS):
        layer[s] = k
    h = torch.nonzero(torch.isin(station, torch.tensor(LAYERS, dtype=torch.uint8, device=off.device)))[:, 0]
    seg = 3 * (torch.searchsorted(off, h, right=True) - 1) + layer[station[h].long()].long()
    order = torch.argsort(seg, stable=True)
    out = torch.zeros(3 * n + 1, dtype=torch.int64, device=off.device)
    torch.cumsum(torch.bincount(seg, minlength=3 * n), 0, out=out[1:])
    xy = [torch.nn.functional.pad(v[h[order]], (0, _capacity(n) - h.numel())) for v in (x, y)]
    return out.int(), xy[0], xy[1]


def _exact_build(t):
    new = torch.nonzero(t[1:] - t[:-1] > GAP_NS)[:, 0] + 1
    ends = torch.tensor([0, t.numel()], device=t.device)
    return torch.cat([ends[:1], new, ends[1:]]) if t.numel() else ends[:1]


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        off, x, y, z = _select_inputs(case, seed)
        counts = _exact_counts(off, x, y, z, case["test"])
        if counts is None:
            return None
        accept = _accepted(counts, case["two"])
        if case["decision"]:
            counts = counts.clamp(max=2)
        if case["binding"] == "default":
            return counts, accept
        out = (counts, accept, torch.zeros(1, dtype=torch.int32, device="cuda"))
        if not case["compact"]:
            return out
        if accept is None:
            return out + (None, None)
        return out + (_padded_ids(accept), accept.sum(dtype=torch.int32).reshape(1))
    if kind == "filter":
        off, station, x, y = _raw_events(case["n_events"], case["other_mean"], case["shuffle"], _generator(seed, 2))
        return _exact_filter(off, station, x, y) + (torch.zeros(1, dtype=torch.int32, device="cuda"),)
    if kind == "build":
        off = _exact_build(_build_times(case, seed))
        out = torch.zeros(4 * case["n_events"] + 16, dtype=torch.int64, device="cuda")
        out[: off.numel()] = off
        return out, torch.tensor([off.numel() - 1], device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    if kind == "chain":
        t, station, x, y = _stream(case, seed)
        off = _exact_build(t)
        lo, fx, fy = _exact_filter(off, station, x, y)
        counts = _exact_counts(lo, fx, fy, None, "msd")
        if counts is None:
            return None
        accept = _accepted(counts, False)
        ids = _padded_ids(accept)
        return off, lo, fx, fy, counts, accept, int(accept.sum()), ids.cpu()
    out = []
    for off, x, y in _slices(case, seed):
        off, x, y = (torch.from_numpy(a).cuda() for a in (off, x, y))
        counts = _exact_counts(off, x, y, None, "msd")
        if counts is None:
            out.append((0, None, None, None, None))
            continue
        accept = _accepted(counts, False)
        out.append((0, counts.cpu().numpy(), accept.cpu().numpy(), int(accept.sum()), _padded_ids(accept).cpu()))
    return out

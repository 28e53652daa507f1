"""GPU parity at the edges of single kernels' tiles, groups and dispatch
rules, bit-exact against the CPU oracle.  Every case prints its name before it
touches the GPU."""
import numpy as np
import pytest

from oracle import reference as R
from paper_1810_11966_amd import synth
from tests import helpers
from tests.test_gpu_parity import assert_parity, gpu  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("test", ("msd", "msd_basis", "window", "msd_z", "window_z"))
def test_every_triplet_loop_groups(gpu, test):  # noqa: F811
    """The every-triplet loops (plain, persistent): 1 to 9 tiles of 64 pairs
    (groups of four, two and one tiles and their remainders), layer-2 sizes
    around the groups of four and the 512-hit chunks, and thresholds with the
    larger bound in either plane."""
    pairs = [(1, 1), (8, 8), (13, 5), (16, 8), (64, 3), (3, 65), (16, 16), (15, 22), (20, 20), (7, 64), (24, 24)]
    sizes = [(a, b, n2) for a, b in pairs for n2 in (1, 2, 3, 4, 5, 8)]
    sizes += [(a, b, n2) for a, b in ((3, 5), (16, 20)) for n2 in (511, 512, 513, 1029)]
    s = synth.concat([helpers.ragged_sizes_set(sizes, seed=31),
                      helpers.near_threshold_events(60, 9, seed=32, rel=1e-5)])
    if test.endswith("_z"):
        s = synth.staggered(s)
    for form in ("plain", "persistent"):
        c = assert_parity(gpu, s, test.replace("_z", ""), form, f"loop groups {test}")
        assert c.sum() > 0
        for cut in ((0.01, 0.2), (0.2, 0.01)):
            assert_parity(gpu, s, test.replace("_z", ""), form, f"loop groups {test} {cut}", msd_max=cut,
                          slope_window=cut)


def duplicated_track_events(copies, noise, seed):
    """One event per (a, b, c): a, b and c copies of one straight track's hits
    in layers 0, 1 and 2 among `noise` other hits per layer (a b surviving
    pairs or more, a b c passing triplets or more)."""
    rng = np.random.default_rng(seed)
    events = []
    for a, b, n2 in copies:
        m = rng.uniform(-0.3, 0.3, 2)
        layers = []
        for z, n in zip((400.0, 410.0, 420.0), (a, b, n2)):
            pts = [(m[0] * z, m[1] * z)] * n + [tuple(p) for p in rng.uniform(-200, 200, (noise, 2))]
            layers.append([pts[k] for k in rng.permutation(len(pts))])
        events.append(layers)
    return synth.from_layers(events)


@pytest.mark.parametrize("test", ("msd", "msd_basis", "window"))
def test_binned_pair_list_limit(gpu, test):  # noqa: F811
    """The binned form's list of surviving pairs: events with 63, 64 and 65
    pairs of one track (both sides of its 64 entries) and with far more, layer
    2 of one to four rounds of 64 hits, also decision only (the cap inside
    the list and inside the cells)."""
    from paper_1810_11966_amd import trig
    s = synth.concat([
        duplicated_track_events([(a, b, n2) for a, b in ((7, 9), (8, 8), (5, 13), (13, 5), (1, 64), (30, 30))
                                 for n2 in (0, 1, 3, 64, 65, 200)], noise, seed=41 + noise) for noise in (1, 40)])
    for form in ("binned", "persistent_binned"):
        c = assert_parity(gpu, s, test, form, "pair list")
        assert c.max() > 30000
    for cap in (0, 1, 700):
        from tests.test_gpu_parity import oracle_result, run_gpu
        from oracle import reference as R
        print(f"[decision only] {test} min_triplets={cap}", flush=True)
        got = run_gpu(gpu, s, test, "binned", min_triplets=cap, extra_flags=trig.TRIG_DECISION_ONLY)
        want, accept, _, _ = oracle_result(s, R.OracleConfig(test=test, min_triplets=cap))
        assert np.array_equal(got["counts"], np.minimum(want, cap))
        assert np.array_equal(got["accept"], accept)


# ------------------------------------------------------- station filter ---

def filter_parity(torch, label, lens, station, layers=(13, 14, 15), workspace_bytes=None, capacity=None):
    """The station filter on events of `lens` hits against the oracle, x and
    y the hits' numbers (so that a wrong hit shows)."""
    from oracle import reference as R
    from paper_1810_11966_amd import filter as F
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    station = np.asarray(station, np.uint8)
    assert off[-1] == len(station)
    x = np.arange(len(station), dtype=np.float32)
    y = -x
    print(f"[filter edges] {label} events={len(lens)} hits={len(station)} workspace={workspace_bytes}", flush=True)
    cap = int(np.isin(station, layers).sum()) if capacity is None else capacity
    d = [torch.from_numpy(a).cuda() for a in (off, station, x, y)]
    ws = None if workspace_bytes is None else torch.empty(workspace_bytes, dtype=torch.uint8, device="cuda")
    r = F.filter_stations(*d, layers, cap, workspace=ws)
    torch.cuda.synchronize()
    lo, fx, fy, status = R.filter_stations(off, station, x, y, layers)
    assert np.array_equal(r.layer_offsets.cpu().numpy(), np.minimum(lo, cap)), label
    assert np.array_equal(r.x.cpu().numpy()[:cap], fx[:cap]) and np.array_equal(r.y.cpu().numpy()[:cap], fy[:cap]), label
    assert int(r.status.cpu()[0]) == status | (4 if lo[-1] > cap else 0), label


def scattered(n_hits, n_trigger, rng):
    """Station numbers of one event: trigger hits of all three layers at
    random places."""
    st = rng.integers(0, 13, n_hits)
    st[rng.permutation(n_hits)[:n_trigger]] = rng.integers(13, 16, n_trigger)
    return st


def together(n_hits, windows, per_window):
    """per_window trigger hits in each of `windows` runs of 64 hits."""
    st = np.zeros(n_hits, np.int64)
    for k in range(windows):
        at = 64 * k + 3 * (k % 9)
        st[at:at + per_window] = 13 + np.arange(per_window) % 3
    return st


def filter_workspace(n_events, per):
    """Workspace bytes of a layout with `per` events per wave (four waves per
    workgroup): layer counts, totals, record counts, 512 bytes of records per
    event slot."""
    a = lambda v: (v + 255) & ~255
    nb = max(1, -(-n_events // (4 * per)))
    return a(12 * n_events) + a(8 * (nb + 1)) + a(4 * n_events) + a(nb * 4 * per * 512)


@pytest.mark.parametrize("per", (1, 4))
def test_filter_record_lists(gpu, per):  # noqa: F811
    """Both kinds of the waves' lists on both sides of their ends, and waves
    whose events differ in kind, with one event per wave (small batches) and
    with four (what a workspace of that layout alone gets)."""
    rng = np.random.default_rng(51)
    kinds = {
        "entries": [scattered(3000, n, rng) for n in (127, 128, 129, 0, 300, 512, 513, 1, 128, 128, 128, 128, 128, 128,
                                                      129, 128)],
        "windows": [together(9000, w, p) for w, p in ((31, 9), (32, 9), (33, 9), (5, 30), (128, 5), (129, 5), (32, 4),
                                                      (32, 12), (33, 4), (0, 0), (96, 8), (1, 40))],
    }
    kinds["mixed"] = [e for pair in zip(kinds["entries"], kinds["windows"]) for e in pair] + \
        [scattered(4000, 90, rng) for _ in range(9)] + [together(4000, 4, 25) for _ in range(9)]
    for name, evs in kinds.items():
        for order in (0, 1, 5):
            # 512 events: there a layout of one event per wave needs more
            # than the layout of four that the smaller workspace has
            e = ((evs[order:] + evs[:order]) * (512 // len(evs) + 1))[:512]
            assert filter_workspace(512, 1) > filter_workspace(512, 4)
            ws = filter_workspace(len(e), per)
            filter_parity(gpu, f"{name} order {order}", [len(v) for v in e], np.concatenate(e), workspace_bytes=ws)
    from paper_1810_11966_amd.trig import TrigError
    with pytest.raises(TrigError):  # less than the smallest layout: refused
        filter_parity(gpu, "short workspace", [len(v) for v in evs], np.concatenate(evs),
                      workspace_bytes=filter_workspace(len(evs), 4) - 256)


@pytest.mark.parametrize("n_events", (1, 3, 16383, 16384, 32767, 32768))
def test_filter_event_split(gpu, n_events):  # noqa: F811
    """Batches on both sides of the sizes where the events per wave change,
    scattered and grouped, also with an output shorter than the hits."""
    rng = np.random.default_rng(n_events)
    lens = rng.integers(0, 40, n_events)
    st = rng.integers(8, 16, int(lens.sum()))
    filter_parity(gpu, "split scattered", lens, st)
    ev = np.repeat(np.arange(n_events), lens)
    filter_parity(gpu, "split grouped", lens, st[np.lexsort((st, ev))])
    filter_parity(gpu, "split short output", lens, st, capacity=int(np.isin(st, (13, 14, 15)).sum()) // 2)


@pytest.mark.parametrize("n_events", (6144, 6145, 12288, 12289, 32768, 32769, 49152, 49153))
@pytest.mark.parametrize("large", (False, True))
def test_filter_totals(gpu, n_events, large):  # noqa: F811
    """Both ways to the workgroups' first positions, on both sides of the sizes
    where the events per wave and the way change; batches of large events on
    average, in a few events of them."""
    rng = np.random.default_rng(n_events)
    lens = rng.integers(0, 12, n_events)
    if large:
        lens[rng.integers(0, n_events, 16)] = -(-1000 * n_events // 16)
    filter_parity(gpu, f"totals large={large}", lens, rng.integers(0, 256, int(lens.sum())))


# -------------------------------------------------- every-triplet forms ---

@pytest.mark.parametrize("test", ("msd", "msd_basis"))
@pytest.mark.parametrize("form", ("plain", "persistent"))
def test_one_tile_events(gpu, form, test):  # noqa: F811
    """Events on both sides of one tile of pairs and of sixteen layer-2 hits,
    at cuts that pass few, many and all triplets; with a NaN or infinite hit,
    and with hits at the top of binary32 in every other event."""
    sizes = [(a, b, c) for a, b in ((1, 1), (1, 64), (64, 1), (1, 65), (65, 1), (8, 8), (9, 7), (5, 13), (7, 9), (2, 32),
                                    (3, 21), (63, 1), (0, 4), (4, 0)) for c in (0, 1, 2, 15, 16, 17)]
    s = helpers.ragged_sizes_set(sizes * 4, seed=91)
    passing = []
    for f in (1.0, 100.0, 1e6):
        cuts = dict(msd_max=(0.03 * f * f, 0.025 * f * f))
        passing.append(int(assert_parity(gpu, s, test, form, f"one tile x{f}", **cuts).sum()))
        for k, bad in enumerate((np.nan, np.inf, -3.4028235e38)):
            x = s.x.copy()
            x[k::7] = bad
            assert_parity(gpu, synth.EventSet(s.offsets, x, s.y, s.n_tracks), test, form, f"one tile x{f} {bad}", **cuts)
    assert passing[0] < passing[1] <= passing[2]


# ------------------------------------------------------------ per-hit z ---

@pytest.mark.parametrize("test", ("msd", "window"))
def test_per_hit_z_blocks(gpu, test):  # noqa: F811
    """Per-hit z from blocks of events in LDS: both event tables (blocks of up
    to 52 and up to 128 events), hit counts that end inside a 16-byte group,
    events of the general path (over 64 hits in both layers), blocks over the
    hit capacity, blocks with one malformed event or one hit whose z no bound
    covers, z scales at and past the range of the approximate slopes, and
    batches on both sides of the size where a wave takes an event alone."""
    rng = np.random.default_rng(61)
    base = {
        "small events": helpers.ragged_sizes_set([tuple(rng.integers(0, 9, 3)) for _ in range(700)], seed=62),
        "medium events": helpers.ragged_sizes_set([tuple(rng.integers(20, 45, 3)) for _ in range(300)], seed=63),
        "general path": helpers.ragged_sizes_set([(70, 66, 5), (3, 80, 4), (65, 65, 65)] * 8 + [(9, 9, 9)] * 60, seed=64),
        "over capacity": helpers.ragged_sizes_set([(5, 5, 5)] * 90 + [(800, 9, 1300), (10, 900, 1200)] + [(6, 5, 4)] * 90,
                                                  seed=65),
        "wave per event": helpers.ragged_sizes_set([tuple(rng.integers(60, 90, 3)) for _ in range(40)], seed=66),
    }
    for tail in (1, 2, 3):
        base[f"tail {tail}"] = helpers.ragged_sizes_set([(9, 8, 7)] * 40 + [(4, 4, 4 + (tail - 40 * 24 - 12) % 4)], seed=67)
        assert base[f"tail {tail}"].n_hits % 4 == tail
    for name, s0 in base.items():
        s = synth.staggered(s0)
        c = assert_parity(gpu, s, test, "pruned", f"z {name}")
        assert c.sum() > 0, name
        for k, bad_z in enumerate((0.0, -400.0, np.nan, np.inf)):
            z = s.z.copy()
            z[rng.integers(0, s.n_hits)] = bad_z
            bad = synth.EventSet(s.offsets, s.x, s.y, s.n_tracks, z=z)
            assert_parity(gpu, bad, test, "pruned", f"z {name} with a z of {bad_z}")
        off = s.offsets.copy()
        off[3 * (s.n_events // 2) + 1] = off[3 * (s.n_events // 2) + 2] + 1
        assert_parity(gpu, synth.EventSet(off, s.x, s.y, s.n_tracks, z=s.z), test, "pruned", f"z {name} malformed")
    s = synth.staggered(base["medium events"])
    for e in (-101, -92, -60, 40, 91, 93):  # z times 2^e: at 2^+-92 around the range's ends
        f = np.float32(2.0) ** np.float32(e)
        scaled = synth.EventSet(s.offsets, s.x, s.y, s.n_tracks, z=s.z * f)
        for w in (np.float32(0.005) / f, np.float32(1e30)):
            assert_parity(gpu, scaled, test, "pruned", f"z scale 2^{e}", slope_window=(float(w), float(w)))
        with np.errstate(over="ignore"):
            both = synth.EventSet(s.offsets, s.x * f, s.y * f, s.n_tracks, z=s.z * f)
        assert_parity(gpu, both, test, "pruned", f"all scales 2^{e}")


def test_per_hit_z_misaligned(gpu):  # noqa: F811
    """z (or x and y) starting 4 bytes past a 16-byte boundary."""
    from paper_1810_11966_amd import trig
    from tests.test_gpu_parity import oracle_result
    from oracle import reference as R
    s = synth.staggered(synth.make_event_set(synth.SMALL_10K, n_events=900))
    want = oracle_result(s, R.OracleConfig())[0]
    off = gpu.from_numpy(s.offsets).cuda()
    for shift in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 2, 2)):
        a = []
        for v, k in zip((s.x, s.y, s.z), shift):
            t = gpu.zeros(s.n_hits + 4, dtype=gpu.float32, device="cuda")
            t[k:k + s.n_hits] = gpu.from_numpy(v).cuda()
            a.append(t[k:k + s.n_hits])
        print(f"[per-hit z misaligned] {shift}", flush=True)
        r = trig.select(off, a[0], a[1], hit_z=a[2], form="pruned")
        assert np.array_equal(r.counts.cpu().numpy(), want)


# ----------------------------------------------------------- compaction ---

@pytest.mark.parametrize("n_events", (1, 15, 16, 17, 4095, 4096, 4097, 61440, 65535, 65536, 65537, 131077))
def test_compaction_block_edges(gpu, n_events):  # noqa: F811
    """Accepted ids at the edges of a thread's 16 events, a block's 4,096 and
    the one-launch form's 65,536, few and many accepted, with the flags
    16-byte aligned and not, whole and at the end of a longer buffer."""
    from paper_1810_11966_amd import trig
    rng = np.random.default_rng(n_events)
    z = np.array([400.0, 410.0, 420.0])
    for share in (0.0, 0.002, 0.5, 1.0):
        hit = rng.random(n_events) < share
        hit[-1] = share > 0
        m = rng.uniform(-0.3, 0.3, n_events)
        x = (m[:, None] * z + np.where(hit, 0.0, 30.0)[:, None] * np.array([0.0, 1.0, 0.0])).astype(np.float32).ravel()
        d = [gpu.from_numpy(a).cuda() for a in (np.arange(3 * n_events + 1, dtype=np.int32), x, np.zeros_like(x))]
        for shift in (0, 1, 16):
            print(f"[compaction] events={n_events} share={share} shift={shift}", flush=True)
            counts = gpu.full((n_events,), -9, dtype=gpu.int32, device="cuda")
            flags = gpu.full((n_events + 40,), 7, dtype=gpu.uint8, device="cuda")
            accept = flags[shift:shift + n_events]
            r = trig.select(*d, form="pruned", compact=True, min_triplets=1, out=(counts, accept))
            gpu.cuda.synchronize()
            assert np.array_equal(accept.cpu().numpy() != 0, hit)
            assert int(r.n_accepted.cpu()[0]) == int(hit.sum())
            assert np.array_equal(r.ids.cpu().numpy()[: int(hit.sum())], np.flatnonzero(hit))
            assert (flags[:shift].cpu().numpy() == 7).all() and (flags[shift + n_events:].cpu().numpy() == 7).all()


# --------------------------------------------------- window prefilter ---

@pytest.mark.parametrize("form", ("pruned", "persistent_pruned"))
def test_window_prefilter_layer_positions(gpu, form):  # noqa: F811
    """The batched window test's approximate slopes: pairs at the window's
    edge far from the axis, and layer positions whose reciprocals are
    subnormal, overflow, or sit at either end of the normal range."""
    edge = synth.concat([helpers.window_boundary_events(100, 6, seed=71, rel=1e-6),
                         helpers.window_boundary_events(100, 6, seed=72, rel=3e-8)])
    c = assert_parity(gpu, edge, "window", form, "window edge")
    assert c.sum() > 0
    far = synth.EventSet(edge.offsets, edge.x * np.float32(512), edge.y * np.float32(512), edge.n_tracks)
    for w in (2.56, 2.5600002, 1e-3, 300.0):
        assert_parity(gpu, far, "window", form, f"far from the axis, window {w}", slope_window=(w, w))
    s = helpers.ragged_sizes_set([(9, 8, 7), (20, 25, 22), (40, 3, 5)] * 20, seed=73)
    for z in ((1e-42, 2e-42, 3e-42), (2e-38, 2.1e-38, 2.2e-38), (1e-3, 1e-38, 5.0), (3e38, 3.1e38, 3.2e38),
              (8e37, 9e37, 1e38), (1e38, 1e-38, 1.0), (1e30, 1e30, 1e30)):
        for w in (0.0, 1e-38, 1e-30, 1.0, 1e30, 3e38):
            assert_parity(gpu, s, "window", form, f"z {z} window {w}", z=z, slope_window=(w, w))


# ----------------------------------------------------- direct pair scan ---

@pytest.mark.parametrize("test", ("msd", "msd_basis", "window", "msd_z", "window_z"))
def test_direct_scan_edges(gpu, test):  # noqa: F811
    """The batched form's scan of staged pairs, two hits per lane: layer sizes
    around the copies' counts (1 to 64 lanes per copy, 16 copies to one), its
    limit of 128 hits in the lanes, 1,023 steps over the other layer and 64
    entries of the exact pass; overlapping last copies; every pair of an event
    close; layers at the ends of the scan's range of z ratios and beyond."""
    ns = (1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 21, 22, 31, 32, 33, 42, 43, 63, 64, 65, 127, 128, 129)
    sizes = [(a, b, 5) for a in ns for b in ns]
    sizes += [p for n in (1022, 1023, 1024) for m in (65, 127, 129) for p in ((n, m, 3), (m, n, 3))]
    s = helpers.ragged_sizes_set(sizes, seed=91)
    dup = duplicated_track_events([(a, b, 3) for a in (1, 2, 9, 30, 70) for b in (1, 2, 9, 30, 70)], 4, seed=92)
    near = synth.concat([helpers.near_threshold_events(40, n, seed=95, rel=1e-6) for n in (5, 16, 33)]
                        + [helpers.pair_boundary_events(40, 12, seed=96), helpers.window_boundary_events(40, 12, seed=97)])
    if test.endswith("_z"):
        s, dup, near = (synth.staggered(v) for v in (s, dup, near))
    t = test.replace("_z", "")
    for label, v in (("sizes", s), ("close pairs", dup), ("near the bounds", near)):
        for form in ("pruned",) if test.endswith("_z") else ("pruned", "persistent_pruned"):
            c = assert_parity(gpu, v, t, form, f"direct scan, {label}, {test}")
            assert c.sum() > 0
    if not test.endswith("_z"):
        few = helpers.ragged_sizes_set([(30, 33, 31), (5, 40, 9), (64, 17, 20)] * 10, seed=98)
        for z in ((1.0, 1e18, 2e18), (1e18, 1.0, 2e18), (1.0, 2e18, 3e18), (1e-18, 1.0, 2.0), (4e-19, 4.1e-19, 1.0),
                  (1e30, 1.0, 1e30), (1e-20, 1e20, 1e20)):
            for cut in (0.0, 1e-3, 1e20):
                assert_parity(gpu, few, t, "pruned", f"direct scan, z {z} cut {cut}", z=z, msd_max=(cut, cut),
                              slope_window=(cut, cut))


@pytest.mark.parametrize("hit_z", (False, True))
def test_block_offset_checks(gpu, hit_z):  # noqa: F811
    """Blocks with one malformed offset at each place of an event: below 0,
    the ends of int32 (whose differences wrap) and one beyond its neighbour or
    the hits; and one to 130 events per block, among them empty layers."""
    base = helpers.ragged_sizes_set([(3, 4, 5), (0, 2, 1), (6, 0, 2), (7, 7, 0), (9, 8, 11)] * 26, seed=99)
    n = int(base.offsets[-1])
    lo, hi = -2 ** 31, 2 ** 31 - 1
    for n_events in (1, 2, 63, 65, 130):
        off = base.offsets[: 3 * n_events + 1].copy()
        whole = synth.EventSet(off, base.x[: off[-1]], base.y[: off[-1]], base.n_tracks[:n_events])
        whole = synth.staggered(whole) if hit_z else whole
        assert_parity(gpu, whole, "msd", "pruned", f"block of {n_events}")
        for at in sorted({0, 1, 2, 3 * (n_events // 2) + 1, 3 * n_events - 1, 3 * n_events}):
            for bad in (lo, lo + 1, -1, hi, hi - 1, n + 1, int(off[min(at + 1, 3 * n_events)]) + 1):
                o = off.copy()
                o[at] = bad
                s = synth.EventSet(o, whole.x, whole.y, whole.n_tracks)
                if hit_z:
                    s.z = whole.z
                assert_parity(gpu, s, "msd", "pruned", f"block of {n_events}, offset {at} = {bad}")


# --------------------------------------------------------- binned cells ---

@pytest.mark.parametrize("test", ("msd", "msd_basis", "window"))
def test_binned_cell_edges(gpu, test):  # noqa: F811
    """The binned form's cells: layer sizes at its rounds of 64 and its limit
    of 256 (layer 0 beyond it), tracks through the outermost cells, |y| far
    larger than |x| and the reverse, all x equal to 0, coordinate scales from
    subnormal to huge, and one infinite or NaN hit per event."""
    ns = (1, 2, 63, 64, 65, 128, 129, 192, 193, 255, 256)
    s = helpers.ragged_sizes_set([(a, b, 9) for a in (1, 64, 65, 255, 256, 257, 600) for b in ns], seed=81)
    c = assert_parity(gpu, s, test, "binned", "cell sizes")
    assert (c > 0).all()
    rng = np.random.default_rng(82)
    t = helpers.ragged_sizes_set([(30, 40, 20), (100, 120, 70), (7, 250, 5)] * 6, seed=83, spread=150.0)
    x, y = t.x.copy(), t.y.copy()
    for e in range(t.n_events):  # a track whose layer-1 hit is the event's outermost in x
        o = t.offsets[3 * e: 3 * e + 4]
        sign = 1.0 if e % 2 else -1.0
        for layer, z in enumerate((400.0, 410.0, 420.0)):
            x[o[layer]] = np.float32(sign * 0.45 * z)
            y[o[layer]] = np.float32(0.1 * z)
    edge = synth.EventSet(t.offsets, x, y, t.n_tracks)
    c = assert_parity(gpu, edge, test, "binned", "outermost cells")
    assert (c > 0).all()
    one = np.float32(1)
    for fx, fy in ((one, np.float32(2e4)), (np.float32(2e4), one), (np.float32(0), one), (one, np.float32(0)),
                   (np.float32(1e-43), np.float32(1e-43)), (np.float32(1e-30), one), (np.float32(1e30), np.float32(1e30)),
                   (np.float32(1e36), np.float32(1e36))):
        scaled = synth.EventSet(t.offsets, x * fx, y * fy, t.n_tracks)
        w = (max(float(0.005 * fx), 1e-45), max(float(0.005 * fy), 1e-45))
        assert_parity(gpu, scaled, test, "binned", f"scales {fx} {fy}", slope_window=w)
    for bad in (np.inf, -np.inf, np.nan):
        for plane in (0, 1):
            v = [x.copy(), y.copy()]
            for e in range(t.n_events):
                v[plane][rng.integers(t.offsets[3 * e], t.offsets[3 * e + 3])] = bad
            assert_parity(gpu, synth.EventSet(t.offsets, v[0], v[1], t.n_tracks), test, "binned", f"{bad} in plane {plane}")


@pytest.mark.parametrize("n_events", (1, 5, 255, 98303, 98304, 98311, 400003))
def test_binned_runs_and_slices(gpu, n_events):  # noqa: F811
    """The binned form's runs of one, two and eight events per wave with a
    remainder, and its stealing form's 64 slices (fewer workgroups than
    slices, slices of unequal size), with malformed events in between."""
    rng = np.random.default_rng(n_events)
    counts = rng.integers(0, 4, 3 * n_events)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    m = rng.uniform(-0.3, 0.3, (n_events, 2))
    ev = np.repeat(np.arange(n_events), counts.reshape(-1, 3).sum(1))
    z = np.repeat(np.tile([400.0, 410.0, 420.0], n_events), counts)
    shift = np.where(rng.random(len(ev)) < 0.7, 0.0, 25.0)  # most hits on the event's track
    x, y = ((m[ev, k] * z + shift).astype(np.float32) for k in range(2))
    bad = off.copy()
    for e in rng.integers(0, n_events, max(1, n_events // 500)):
        bad[3 * e + 1] = -1
    tracks = np.zeros(n_events, np.int8)
    for form in ("binned", "persistent_binned"):
        for o in (off, bad):
            c = assert_parity(gpu, synth.EventSet(o, x, y, tracks), "msd", form, "runs")
        assert n_events < 100 or c.max() > 8


# -------------------------------------------------------- event building ---

@pytest.mark.parametrize("off", (0, 1))
def test_event_building_edges(gpu, off):  # noqa: F811
    """Stream sizes around a lane's two hits, the rounds of 128, the batches
    of 256, the wave's 4,096 and the workgroup's 16,384, on 16-byte aligned
    times and on times 8 bytes further; every hit an event, none, a start or a
    time reversal on each side of those edges; capacities up to all offsets."""
    from paper_1810_11966_amd import events as EB
    for n in (1, 2, 3, 63, 64, 127, 128, 129, 255, 256, 257, 4095, 4096, 4097, 16383, 16384, 16385, 50001):
        edges = [e for e in (1, 2, 3, 127, 128, 129, 255, 256, 257, 4095, 4096, 4097, 16383, 16384, 16385) if e < n]
        steps = [np.full(n, 6), np.zeros(n, np.int64), np.where(np.arange(n) % 3 == 2, 6, 5)]
        for sign in (6, -1):
            step = np.zeros(n, np.int64)
            step[edges] = sign
            steps.append(step)
        for k, step in enumerate(steps):
            t = -(2 ** 40) + np.cumsum(step).astype(np.int64)
            want, st = R.build_events_numpy(t, 5)
            d = gpu.from_numpy(np.concatenate([np.zeros(off, np.int64), t])).cuda()[off:]
            for cap in sorted({len(want), max(1, len(want) - 1), 1}):
                print(f"[events] hits={n} offset={off} stream {k} capacity {cap}", flush=True)
                r = EB.build_events(d, 5, capacity=cap)
                gpu.cuda.synchronize()
                assert int(r.n_events.cpu()[0]) == len(want) - 1
                assert np.array_equal(r.offsets.cpu().numpy(), want[:cap])
                assert int(r.status.cpu()[0]) == (st | (4 if cap < len(want) else 0))


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("n", (1024 * 16384, 1024 * 16384 + 1, 48 << 20, (48 << 20) + 1))
def test_event_building_long_streams(gpu, n, off):  # noqa: F811
    """Both sides of the largest stream whose waves sum the totals themselves
    (1,024 workgroups) and of the largest one read with cached loads."""
    from paper_1810_11966_amd import events as EB
    rng = np.random.default_rng(5)
    t = np.cumsum(rng.choice(np.array([0, 1, 2, 9], np.int64), n))
    print(f"[events] hits={n}", flush=True)
    want, st = R.build_events_numpy(t, 3)
    d = gpu.from_numpy(np.concatenate([np.zeros(off, np.int64), t])).cuda()[off:]
    r = EB.build_events(d, 3)
    gpu.cuda.synchronize()
    assert int(r.n_events.cpu()[0]) == len(want) - 1 and int(r.status.cpu()[0]) == st
    assert np.array_equal(r.offsets.cpu().numpy()[:len(want)], want)


@pytest.mark.parametrize("n", (1536 * 16384, 1536 * 16384 + 1, 40 << 20, (40 << 20) + 1))
def test_event_building_totals(gpu, n):  # noqa: F811
    """Both sides of the largest stream whose waves sum the totals themselves
    and of the largest one read with cached loads: a start every 1,000 hits."""
    from paper_1810_11966_amd import events as EB
    h = gpu.arange(n, dtype=gpu.int64, device="cuda")
    r = EB.build_events(h + 5 * (h // 1000), 3)
    k = -(-n // 1000)
    assert int(r.n_events.cpu()[0]) == k and int(r.status.cpu()[0]) == 0
    assert gpu.equal(r.offsets[:k], h[::1000]) and int(r.offsets[k]) == n

"""GPU parity at the edges of single kernels' tiles, groups and dispatch
rules, bit-exact against the CPU oracle.  Every case prints its name before it
touches the GPU."""
import numpy as np
import pytest

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

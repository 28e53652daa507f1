"""GPU parity where a prefilter's own arithmetic leaves binary32's range:
products and sums of accepted inputs that overflow, interval ends that are
infinite.  Bit-exact against the CPU oracle; every case prints its name before
it touches the GPU."""
import numpy as np
import pytest

from paper_1810_11966_amd import synth
from tests import helpers
from tests.test_gpu_parity import assert_parity, gpu  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

FLT_MAX = float(np.finfo(np.float32).max)


def events_of(*events):
    """One event per tuple of three x lists (y = 0)."""
    return synth.from_layers([[[(float(np.float32(v)), 0.0) for v in layer] for layer in e] for e in events])


@pytest.mark.parametrize("form", ("pruned", "persistent_pruned"))
def test_scaled_products_that_overflow(gpu, form):  # noqa: F811
    """The batched form's scan multiplies the lane layer by the ratio of the
    layer positions: with hits near the largest binary32 that product, or the
    sum, is infinite for a pair that passes."""
    z = (465.54053, 409.91873, 381.8398)
    e = events_of(([1.0], [1.0], [1.0]), ([FLT_MAX], [2.9962613e38], [5.0, 2.7910212e38]))
    c = assert_parity(gpu, e, "window", form, "quotients of FLT_MAX", z=z)
    assert c[1] == 1
    rng = np.random.default_rng(11)
    for zs in (z, (400.0, 410.0, 420.0), (420.0, 410.0, 400.0), (1.0, 3.0, 2.0), (1e10, 1.0, 1.0), (1.0, 1e10, 1.0)):
        zz = np.asarray(zs)
        for scale in (3.4e38, 1.7e38, 8e37, 1e37):
            m = scale / zz.max() * rng.uniform(0.9, 1.0, 24) * rng.choice([-1.0, 1.0], 24)
            ev = []
            for k in range(24):
                layers = [[m[k] * zz[layer], -m[k] * zz[layer] * 0.5, 3.0 * layer, m[(k + 1) % 24] * zz[layer]]
                          for layer in range(3)]
                ev.append([np.clip(v, -FLT_MAX, FLT_MAX) for v in layers])
            s = events_of(*ev)
            w = float(np.float32(abs(m).max() * 1e-6))
            for test in ("window", "msd_basis", "msd"):
                c = assert_parity(gpu, s, test, form, f"z {zs} scale {scale}", z=zs, slope_window=(w, w),
                                  msd_max=(1e37, 1e37))
            wide = (FLT_MAX, FLT_MAX)
            c = assert_parity(gpu, s, "window", form, f"widest windows, z {zs} scale {scale}", z=zs, slope_window=wide,
                              msd_max=(1e37, 1e37))
            assert c.sum() > 0


@pytest.mark.parametrize("form", ("binned", "persistent_binned"))
def test_cells_without_a_scale(gpu, form):  # noqa: F811
    """The binned form's cells where the largest key is 0, infinite or so large
    that its reciprocal is 0, with interval ends that overflow."""
    e = events_of(([3.0], [2.9, 150.0], [2.9]), ([3.0], [150.0, 2.9, -7.0], [2.9, 1.0]))
    c = assert_parity(gpu, e, "window", form, "keys beyond binary32", z=(2e-38, 2.1e-38, 2.2e-38),
                      slope_window=(3e38, 3e38))
    assert (c > 0).all()
    origin = events_of(([0.0, 5.0], [0.0, 0.0], [0.0, 1.0]), ([1.0], [0.0], [2.0]), ([0.0], [-0.0], [0.0]))
    for w in (FLT_MAX, 3e38, 1.0, 1e-38):
        c = assert_parity(gpu, origin, "window", form, f"layer 1 at the origin, window {w}", slope_window=(w, w))
        assert c.sum() > 0
    s = helpers.ragged_sizes_set([(9, 8, 7), (20, 25, 22), (40, 3, 5)] * 20, seed=73)
    for z in ((1e-42, 2e-42, 3e-42), (2e-38, 2.1e-38, 2.2e-38), (1e-3, 1e-38, 5.0), (3e38, 3.1e38, 3.2e38),
              (8e37, 9e37, 1e38), (1e38, 1e-38, 1.0), (1e30, 1e30, 1e30), (0.25, 0.5, 0.75)):
        for w in (0.0, 1e-38, 1e-30, 1.0, 1e30, 3e38, FLT_MAX):
            assert_parity(gpu, s, "window", form, f"z {z} window {w}", z=z, slope_window=(w, w))
    big = synth.EventSet(s.offsets, s.x * np.float32(1e36), s.y * np.float32(1e36), s.n_tracks)
    for z in ((400.0, 410.0, 420.0), (0.25, 0.5, 0.75), (1e18, 1.0, 1.0), (1.0, 1e18, 1.0)):
        for test in ("window", "msd", "msd_basis"):
            for cut in (0.0, 1e20, FLT_MAX):
                assert_parity(gpu, big, test, form, f"huge hits, z {z} cut {cut}", z=z, slope_window=(cut, cut),
                              msd_max=(cut, cut))
                assert_parity(gpu, s, test, form, f"z {z} cut {cut}", z=z, slope_window=(cut, cut), msd_max=(cut, cut))

"""GPU parity where a prefilter's own arithmetic leaves binary32's range:
products and sums of accepted inputs that overflow.  Bit-exact against the CPU
oracle; every case prints its name before it touches the GPU."""
import numpy as np
import pytest

from paper_1810_11966_amd import synth
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

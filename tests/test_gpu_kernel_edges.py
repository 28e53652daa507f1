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

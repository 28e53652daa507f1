"""The autotuner records what it measured (GPU): a recorded fill stands for the
events per block that were timed, in a batch of any size, so that it means the
same for another batch of its class."""
import numpy as np
import pytest

from paper_1810_11966_amd import synth
from tests.test_gpu_parity import gpu, to_dev  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

RULE_FILL = 0.92  # the built-in rule's record: the shape is chosen anew for each batch


@pytest.mark.parametrize("n_events", (300, 1000, 4096, 20000))
@pytest.mark.parametrize("test", ("msd", "window"))
def test_recorded_fill_was_measured(gpu, n_events, test, tmp_path):  # noqa: F811
    from paper_1810_11966_amd import trig
    s = synth.make_event_set(synth.SMALL_10K, n_events=n_events)
    mean = s.n_hits / n_events
    dev = to_dev(gpu, s)
    for attempt in range(4):
        print(f"[autotune record] events={n_events} {test} {attempt}", flush=True)
        trig.trig_autotune_reset()
        r, info = trig.autotune(*dev, test=test, reps=2)
        path = tmp_path / f"cache{attempt}"
        trig.autotune_save(str(path))
        line = path.read_text().splitlines()[1].split()
        form, hb, nw, fill, steal = line[3], int(line[4]), int(line[5]), float(line[6]), int(line[7])
        assert info.binned == (form == "binned")
        if form == "binned" or (fill == RULE_FILL and not steal):
            continue
        eb = max(1, min(128, int(fill * hb / mean)))
        eb -= eb % nw if eb >= nw else 0
        assert (info.block_hits, info.block_waves, info.block_events, info.persistent) == (hb, nw, eb, steal)
    trig.trig_autotune_reset()

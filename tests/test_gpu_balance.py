"""GPU: a form's time must not hang on the order of the batch's events or on
how close the cuts are.  Each case times two batches or two cuts in the same
process, in turn, and compares the best times with a wide margin."""
import numpy as np
import pytest

from tests.test_gpu_parity import gpu  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def batch(torch, per_layer, seed, spread=200.0):
    """Noise events with per_layer[e] hits in each layer, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    per = torch.as_tensor(per_layer, dtype=torch.int64, device="cuda")
    off = torch.zeros(3 * per.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(per.repeat_interleave(3), 0, out=off[1:])
    x, y = ((torch.rand(int(off[-1]), generator=g, device="cuda") * 2 - 1) * spread for _ in range(2))
    return off.int(), x, y


def best_ms(torch, calls, rounds=7, reps=4):
    """The best time of each call, ms, taken in turn."""
    best = [float("inf")] * len(calls)
    for r in range(rounds + 1):
        for k, call in enumerate(calls):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            call()
            a.record()
            for _ in range(reps):
                call()
            b.record()
            b.synchronize()
            if r:  # the first round warms up
                best[k] = min(best[k], a.elapsed_time(b) / reps)
    return best


def test_binned_stealing_clustered_events(gpu):  # noqa: F811
    """2 % of the events 30 times as large as the others, at the front or
    spread out: the stealing binned form shares a cluster among all slices."""
    from paper_1810_11966_amd import trig
    n = 300_000
    e = np.arange(n)
    calls = []
    for large in (e < n // 50, e % 50 == 0):
        b = batch(gpu, np.where(large, 300, 10), seed=3)
        calls.append(lambda b=b: trig.select(*b, form="persistent_binned"))
    print("[balance] persistent_binned, 300,000 events", flush=True)
    front, spread = best_ms(gpu, calls)
    print(f"front {front:.3f} ms, spread {spread:.3f} ms", flush=True)
    assert front < 2.5 * spread


@pytest.mark.parametrize("form", ("plain", "persistent"))
def test_every_triplet_loops_at_loose_cuts(gpu, form):  # noqa: F811
    """Cuts that reject next to nothing cost the every-triplet loops the full
    test of each triplet and no more (window test, 20,000 events of 30 hits per
    layer: 7 to 9 times the default cuts' time where each group of triplets went
    through the rejecting test and was then tested hit by hit)."""
    from paper_1810_11966_amd import trig
    b = batch(gpu, np.full(20_000, 30), seed=4)
    calls = [lambda w=w: trig.select(*b, test="window", form=form, slope_window=(w, w)) for w in (0.15, 0.005)]
    print(f"[balance] loose cuts, {form}", flush=True)
    loose, tight = best_ms(gpu, calls)
    print(f"loose {loose:.3f} ms, tight {tight:.3f} ms", flush=True)
    assert loose < 5 * tight


def test_stolen_units_of_wide_events(gpu):  # noqa: F811
    """The stealing every-triplet form's units cost their own pairs: events of
    3 x 200,000 pairs against as many pairs of 775 x 775 (50 times as long
    where each unit read the whole layer for its bound)."""
    from paper_1810_11966_amd import trig
    calls = []
    for n0, n1 in ((3, 200_000), (775, 775)):
        g = gpu.Generator(device="cuda")
        g.manual_seed(5)
        per = gpu.tensor([n0, n1, 3], device="cuda").repeat(20)
        off = gpu.zeros(61, dtype=gpu.int64, device="cuda")
        gpu.cumsum(per, 0, out=off[1:])
        x, y = ((gpu.rand(int(off[-1]), generator=g, device="cuda") * 2 - 1) * 200 for _ in range(2))
        calls.append(lambda b=(off.int(), x, y): trig.select(*b, form="persistent"))
    print("[balance] wide events, persistent", flush=True)
    wide, square = best_ms(gpu, calls)
    print(f"wide {wide:.3f} ms, square {square:.3f} ms", flush=True)
    assert wide < 4 * square


def test_binned_cells_at_loose_cuts(gpu):  # noqa: F811
    """The binned form where many pairs pass (window test, decisions only,
    20,000 events of 150 hits per layer, windows 10 times the default): layer 2
    in cells at once, without listing pairs first (3.7 times the default
    windows' time where every event first listed its pairs)."""
    from paper_1810_11966_amd import trig
    b = batch(gpu, np.full(20_000, 150), seed=6)
    calls = [lambda w=w: trig.select(*b, test="window", form="binned", slope_window=(w, w),
                                     extra_flags=trig.TRIG_DECISION_ONLY) for w in (0.05, 0.005)]
    print("[balance] loose cuts, binned", flush=True)
    loose, tight = best_ms(gpu, calls)
    print(f"loose {loose:.4f} ms, tight {tight:.4f} ms", flush=True)
    assert loose < 2.5 * tight


def test_batched_scan_at_close_pairs(gpu):  # noqa: F811
    """The batched form leaves its scan out for events that are expected to have
    close pairs (100,000 events of 100 hits per layer, cuts 10 times the
    default in cm: 1.9 times the default cuts' time with the scan, 1.4
    without)."""
    from paper_1810_11966_amd import trig
    b = batch(gpu, np.full(100_000, 100), seed=7)
    calls = [lambda f=f: trig.select(*b, form="pruned", msd_max=(0.03 * f, 0.025 * f)) for f in (100.0, 1.0)]
    print("[balance] close pairs, pruned", flush=True)
    close, few = best_ms(gpu, calls)
    print(f"close {close:.4f} ms, few {few:.4f} ms", flush=True)
    assert close < 1.65 * few

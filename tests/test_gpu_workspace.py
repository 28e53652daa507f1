"""Workspaces of earlier releases, smaller than trig_workspace_bytes() now
reports, are still accepted (GPU: trig_select and trig_autotune)."""
import numpy as np
import pytest

from oracle import reference as R
from paper_1810_11966_amd import synth
from tests.test_gpu_parity import gpu, oracle_result, to_dev  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def earlier_bytes(n_events, compact):
    """256 bytes of counters and, with compaction, one count per 1,024 events
    and their total."""
    a = lambda v: (v + 255) & ~255
    return 256 + (a(4 * (-(-n_events // 1024) + 1)) if compact else 0)


@pytest.mark.parametrize("form", ("persistent_pruned", "persistent_binned", "auto"))
@pytest.mark.parametrize("compact", (False, True))
def test_earlier_workspace_sizes(gpu, form, compact):  # noqa: F811
    from paper_1810_11966_amd import trig
    s = synth.make_event_set(synth.SMALL_10K, n_events=9000)
    want, accept, _, _ = oracle_result(s, R.OracleConfig())
    off, x, y = to_dev(gpu, s)
    n = s.n_events
    ev, hits = trig.TrigEventsCsr(n, off.data_ptr()), trig.TrigHits(s.n_hits, x.data_ptr(), y.data_ptr(), None)
    p = trig.make_params(flags=trig.FORMS[form] | (trig.TRIG_OUT_COMPACT if compact else 0))
    counts = gpu.zeros(n, dtype=gpu.int32, device="cuda")
    flags = gpu.zeros(n, dtype=gpu.uint8, device="cuda")
    ids = gpu.zeros(n, dtype=gpu.int32, device="cuda")
    n_accepted = gpu.zeros(1, dtype=gpu.int32, device="cuda")
    if compact:
        p.out_accepted_ids, p.out_n_accepted = ids.data_ptr(), n_accepted.data_ptr()
    small = earlier_bytes(n, compact)
    assert small < trig.trig_workspace_bytes(n, p)
    guard = 512
    ws = gpu.full((small + 256 + guard,), 0x5A, dtype=gpu.uint8, device="cuda")
    start = (-ws.data_ptr()) % 256
    p.workspace, p.workspace_bytes = ws.data_ptr() + start, small
    for run in ("select", "autotune") if form == "auto" else ("select", "select"):
        print(f"[workspace] {form} compact={compact} {small} bytes, {run}", flush=True)
        if run == "select":
            rc = trig.trig_select(ev, hits, p, counts.data_ptr(), flags.data_ptr(), 0)
        else:
            rc, _ = trig.trig_autotune(ev, hits, p, counts.data_ptr(), flags.data_ptr(), 1, 0)
            trig.trig_autotune_reset()
        gpu.cuda.synchronize()
        assert rc == trig.TRIG_OK, trig.trig_last_error_detail()
        assert np.array_equal(counts.cpu().numpy(), want) and np.array_equal(flags.cpu().numpy(), accept)
        if compact:
            assert np.array_equal(ids.cpu().numpy()[: int(n_accepted.cpu()[0])], R.accepted_ids(accept))
        assert (ws[start + small:].cpu().numpy() == 0x5A).all()  # nothing past the workspace
    p.workspace_bytes = (small - 256) if compact else 255  # less than any layout
    assert trig.trig_select(ev, hits, p, counts.data_ptr(), flags.data_ptr(), 0) == trig.TRIG_EWORKSPACE

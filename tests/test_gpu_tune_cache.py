"""The batched form's tuning cache: an entry that an earlier double-precision
kernel was tuned to (its key named no kernel) is not taken for the present one;
single precision, whose kernels are those of such entries, takes it."""
import re

import numpy as np
import pytest

import synth
from gpu_util import PROCESS_TEXT, dev, torch_cuda

pytestmark = pytest.mark.gpu
TUNED = "192 64 256 0"                           # tile, block, grid, helicity split: no default


@pytest.mark.parametrize("precision,old_entry_used", [(0, False), (1, True)])
def test_entries_of_another_kernel(tmp_path, monkeypatch, precision, old_entry_used):
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("RWGT_TUNE_CACHE", str(cache))
    n = 500
    p, w = dev(synth.events("uu_eeg", n)), dev(np.ones(n))
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    ctx = rw.rwgt_create(PROCESS_TEXT["uu_eeg"], synth.ORIG_EW.slha(), precision)

    def schedule():
        b = rw.rwgt_batch_create([ctx])
        try:
            segs, keep = rw.make_segments([(0, p, w, synth.NEW_UU.row("uu_eeg"), out)])
            if not cache.exists():
                rw.rwgt_batch_tune(b, segs, reps=1)
            else:
                rw.rwgt_batch_eval(b, segs)
            torch.cuda.synchronize()
            return rw.rwgt_batch_get_schedule(b)
        finally:
            rw.rwgt_batch_destroy(b)
    try:
        tuned = schedule()
        assert precision or tuned["hel_split"] == 0   # one kernel for both settings: not searched
        key = cache.read_text().split("|")[0]
        assert schedule() == tuned               # its own entry
        cache.write_text(f"{key}|{TUNED}\n")
        got = schedule()
        assert (got["tile_events"], got["block"], got["grid"]) == (192, 64, 256)
        cache.write_text(re.match(r".*log2events=\d+", key).group(0) + f"|{TUNED}\n")
        assert (schedule()["tile_events"] == 192) == old_entry_used
    finally:
        rw.rwgt_destroy(ctx)

"""The double-precision batch kernel at the sizes where its dealing of tiles can
go wrong: segment counts around the 64 and 64^2 of its segment search, tiles
smaller than, equal to and not a multiple of the 64 events of a piece, segments
of one event, and launches of fewer waves than tiles and of more.  Every segment
equals the plain call bit for bit (the same code on the same momenta).
"""
import numpy as np
import pytest

import synth
from gpu_util import PROCESS_TEXT, dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nseg,top,schedule", [
    (1, 1, (64, 64, 1)), (1, 1000, (1, 64, 1)), (63, 70, (63, 128, 1)), (64, 70, (64, 256, 2)),
    (65, 130, (65, 192, 1)), (129, 300, (100, 256, 8)), (4096, 3, (256, 256, 2)), (4097, 3, (2, 64, 1)),
])
def test_segments_equal_plain_calls(nseg, top, schedule):
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    rng = np.random.default_rng(nseg + top)
    counts = rng.integers(1, top + 1, nseg)
    procs = rng.integers(0, 2, nseg)
    names = ("ee_mumu", "uu_eeg")
    cards = synth.batch_grid()
    pool = [dev(synth.events(n, max(int(counts[procs == k].sum()), 1))) for k, n in enumerate(names)]
    w = dev(rng.uniform(0.5, 2.0, int(counts.sum())))
    out = torch.full((int(counts.sum()) + 1,), -5.0, dtype=torch.float64, device="cuda")
    ctxs = [rw.rwgt_create(PROCESS_TEXT[n], synth.ORIG_EW.slha(), rw.RWGT_FP64) for n in names]
    b = rw.rwgt_batch_create(ctxs)
    try:
        rw.rwgt_batch_set_schedule(b, *schedule, 0)
        jobs, at, used = [], 0, [0, 0]
        for k in range(nseg):
            j, m = int(procs[k]), int(counts[k])
            jobs.append((j, pool[j][used[j]:used[j] + m], w[at:at + m], cards[k % 64].row(names[j]), out[at:at + m]))
            used[j], at = used[j] + m, at + m
        segs, keep = rw.make_segments(jobs)
        rw.rwgt_batch_eval(b, segs)
        torch.cuda.synchronize()
        assert float(out[-1]) == -5.0
        for k in np.unique(np.linspace(0, nseg - 1, 40).astype(int)):
            j, mom, wk, row, got = jobs[k]
            want = torch.empty((1, mom.shape[0]), dtype=torch.float64, device="cuda")
            rw.rwgt_set_stream(ctxs[j], None)
            rw.rwgt_eval(ctxs[j], mom, wk.contiguous(), row, want)
            assert torch.equal(got, want[0]), f"segment {k}"
        assert bool(torch.isfinite(out).all()) and bool((out[:-1] > 0).all())
        del keep
    finally:
        rw.rwgt_batch_destroy(b)
        for c in ctxs:
            rw.rwgt_destroy(c)

"""The half-wave-per-event kernels of g g -> t t~ g g and g g -> t t~ t t~ (FP64)
at the sizes where their launch can go wrong: one event, odd counts (the last
wave's second half repeats the last event), several cards, and as the mixed
path's re-evaluation of an odd list of flagged events.  |M|^2 against the
oracle at 1e-10, w' against the exact ratio at 1e-12 and, re-evaluated, against
the FP64 path at 4e-15: the bars of the full-size tests of these processes.
"""
import numpy as np
import pytest

import synth
from gpu_util import dev, gpu_me2, rel_err, torch_cuda
from oracle import reweight

pytestmark = pytest.mark.gpu
TEXT = {"gg_ttgg": "g g > t t~ g g", "gg_tttt": "g g > t t~ t t~"}


@pytest.mark.parametrize("proc", list(TEXT))
@pytest.mark.parametrize("n,ncards", [(1, 1), (1, 3), (2, 1), (3, 2), (65, 1), (129, 5)])
def test_small_and_odd_counts(n, ncards, proc):
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    p = synth.events(proc, 130)[-n:]
    w = np.linspace(0.5, 2.0, n)
    alphas = np.linspace(0.11, 0.13, ncards)
    cards = [synth.Card(aS=float(a)) for a in alphas]
    me = gpu_me2(proc, p, synth.ORIG_QCD, cards)
    pick = np.unique(np.linspace(0, n - 1, min(n, 4)).astype(int))
    ref = reweight.me2(proc, p[pick], cards[0])
    assert rel_err(me[0][pick], ref).max() < 1e-10
    for k in range(ncards):
        assert rel_err(me[k] / me[0], np.full(n, (alphas[k] / alphas[0]) ** 4)).max() < 1e-12
    # outputs exactly fill their array
    buf = torch.full((ncards * n + 7,), -3.0, dtype=torch.float64, device="cuda")
    with rw.Reweighter(TEXT[proc], synth.ORIG_QCD.slha(), rw.RWGT_FP64) as r:
        r.eval(dev(p), dev(w), np.stack([c.row(proc) for c in cards]), buf[:ncards * n])
        torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.all(got[ncards * n:] == -3.0)
    want = w[None, :] * ((alphas / 0.118) ** 4)[:, None]
    assert rel_err(got[:ncards * n].reshape(ncards, n), want).max() < 1e-12


@pytest.mark.parametrize("proc", list(TEXT))
@pytest.mark.parametrize("n", [1, 7, 130])
def test_reevaluation_of_flagged_events(n, proc):
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    p = synth.events(proc, n)
    rows = np.stack([synth.NEW_QCD.row(proc), synth.ORIG_QCD.row(proc)])
    out = {}
    for prec in (rw.RWGT_FP64, rw.RWGT_MIXED_FP16):
        with rw.Reweighter(TEXT[proc], synth.ORIG_QCD.slha(), prec) as r:
            if prec:
                rw.rwgt_set_mixed_guard(r.ctx, 1e-3)             # kappa > 1 / (terms per flow): every event
            out[prec] = torch.empty((2, n), dtype=torch.float64, device="cuda")
            r.eval(dev(p), dev(np.ones(n)), rows, out[prec])
            if prec:
                assert rw.rwgt_mixed_guard_count(r.ctx) == n
    a, b = (out[k].cpu().numpy() for k in (rw.RWGT_FP64, rw.RWGT_MIXED_FP16))
    assert rel_err(b, a).max() <= 4e-15

"""Cards as launch arguments and as an uploaded table (double precision): the
same outputs on both sides of the limit (32 cards, the original included), and
the count of non-finite outputs that the kernels make themselves, on both sides
of theirs (4096 workgroups of two events for the QCD processes).

Both sources hold the same numbers and the kernels' arithmetic is the same:
electroweak weights agree to the bit (fixed roundings); the QCD kernels may
contract differently, 4e-15 as their re-evaluation test."""
import numpy as np
import pytest

import synth
from gpu_util import dev, rel_err, torch_cuda

pytestmark = pytest.mark.gpu
TEXT = {"ee_mumu": "e+ e- > mu+ mu-", "uu_eeg": "u u~ > e+ e- g", "gg_ttgg": "g g > t t~ g g",
        "gg_tttt": "g g > t t~ t t~"}


def _rows(proc, k):
    orig = synth.ORIG_EW if proc in ("ee_mumu", "uu_eeg") else synth.ORIG_QCD
    row = np.asarray(orig.row(proc), dtype=np.float64)
    rows = np.tile(row, (k, 1))
    if proc in ("ee_mumu", "uu_eeg"):
        rows[:, -2] *= 1.0 + 0.001 * np.arange(k)                # M_Z
    else:
        rows[:, 0] *= 1.0 + 0.002 * np.arange(k)                 # alpha_s
    return orig, rows


@pytest.mark.parametrize("proc", list(TEXT))
@pytest.mark.parametrize("nsets", [30, 31, 32, 65])
def test_arguments_and_table_agree(proc, nsets):
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    n = 67
    orig, rows = _rows(proc, nsets)
    p, w = dev(synth.events(proc, n)), dev(np.linspace(0.5, 2.0, n))
    tol = 0.0 if proc in ("ee_mumu", "uu_eeg") else 4e-15
    with rw.Reweighter(TEXT[proc], orig.slha(), rw.RWGT_FP64) as r:
        out = torch.full((nsets, n), -3.0, dtype=torch.float64, device="cuda")
        one = torch.empty((1, n), dtype=torch.float64, device="cuda")
        r.eval(p, w, rows, out)
        me, me1 = torch.empty_like(out), torch.empty_like(one)
        r.me2(p, rows, me)
        for k in {0, 1, nsets // 2, nsets - 1}:
            r.eval(p, w, rows[k:k + 1], one)
            r.me2(p, rows[k:k + 1], me1)
            assert rel_err(out[k].cpu().numpy(), one[0].cpu().numpy()).max() <= tol
            assert rel_err(me[k].cpu().numpy(), me1[0].cpu().numpy()).max() <= tol


@pytest.mark.parametrize("proc", list(TEXT))
@pytest.mark.parametrize("n", [1, 65, 8192, 8193])
def test_nonfinite_count(proc, n):
    """Events of infinite input weight and, for |M|^2, of NaN momenta."""
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    orig, rows = _rows(proc, 3)
    base = synth.events(proc, 64)
    p = np.tile(base, (n // 64 + 1, 1, 1))[:n].copy()
    w = np.ones(n)
    bad = np.unique(np.linspace(0, n - 1, 7).astype(int))
    w[bad] = np.inf
    with rw.Reweighter(TEXT[proc], orig.slha(), rw.RWGT_FP64) as r:
        out = torch.empty((3, n), dtype=torch.float64, device="cuda")
        r.eval(dev(p), dev(w), rows, out)
        assert rw.rwgt_nonfinite(r.ctx) == 3 * len(bad) == int((~torch.isfinite(out)).sum())
        p[bad] = np.nan
        r.me2(dev(p), rows, out)
        assert rw.rwgt_nonfinite(r.ctx) == int((~torch.isfinite(out)).sum()) == 3 * len(bad)

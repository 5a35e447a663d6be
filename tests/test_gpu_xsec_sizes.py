"""The one-pass cross-section reduction at the sizes where its pieces can go
wrong: one event, around the 2048 weights of a chunk, more chunks than blocks
(512 x 2048 and a ragged rest), and weights whose spread is tiny beside their
mean, against the oracle's two-pass sums.  1e-11 on sigma' and 1e-9 on dsigma'
are the bars of the other cross-section tests; with dsigma = 0 and w' constant
to 1e-7 the standard deviation alone is compared, at 1e-6 of itself (rounding
of the weights, 1e-16, over their spread).
"""
import numpy as np
import pytest

import synth
from gpu_util import dev, rel_err, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nsets", [(1, 1), (2, 3), (2047, 2), (2048, 2), (2049, 2), (512 * 2048 + 5, 1),
                                     (3 * 512 * 2048 - 1, 1), (100_003, 65)])
def test_sizes(n, nsets):
    torch_cuda()
    import paper_2510_05100_amd as rw
    from oracle import xsec as oxsec
    rng = np.random.default_rng(n + nsets)
    w = rng.uniform(0.5, 2.0, n)
    w[:: 7] = 0.0
    wp = rng.uniform(0.2, 1.8, (nsets, n)) * np.where(w == 0.0, 0.0, 1.0) + (1.0 if n == 1 else 0.0)
    with rw.Reweighter("g g > t t~ g g", synth.ORIG_QCD.slha()) as r:
        xs, xe, fb = rw.rwgt_xsec(r.ctx, dev(w), dev(wp), 12.5, 0.3, 12.5 / n)
        again = rw.rwgt_xsec(r.ctx, dev(w), dev(wp), 12.5, 0.3, 12.5 / n)
    np.testing.assert_array_equal(xs, again[0])
    np.testing.assert_array_equal(xe, again[1])
    for k in range(nsets):
        rx, re_, rb = oxsec.xsec(w, wp[k], 12.5, 0.3, 12.5 / n)
        assert rel_err(xs[k], rx).max() < 1e-11 and rel_err(xe[k], re_).max() < 1e-9 and fb[k] == np.any(rb)


def test_small_spread():
    torch_cuda()
    import paper_2510_05100_amd as rw
    n = 1_300_001
    rng = np.random.default_rng(5)
    wp = 1.0 + 1e-7 * rng.standard_normal(n)
    wp += np.linspace(0.0, 3e-7, n)                # pieces with different means
    with rw.Reweighter("g g > t t~ g g", synth.ORIG_QCD.slha()) as r:
        _, xe, _ = rw.rwgt_xsec(r.ctx, dev(np.ones(n)), dev(wp[None, :]), 1.0, 0.0, 1.0 / n)
    assert abs(xe[0] / np.std(wp) - 1.0) < 1e-6

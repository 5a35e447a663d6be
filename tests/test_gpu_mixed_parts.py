"""The mixed path with a wave per helicity (small launches) against the kernel
that loops over them (large ones): the same events as a small call and at the
start of a call beyond the form's range.  The single-precision amplitudes are
the same code and the sums over helicities are double precision in the same
order: 1e-15 relative, and the same events flagged."""
import numpy as np
import pytest

import synth
from gpu_util import dev, rel_err, torch_cuda

pytestmark = pytest.mark.gpu
TEXT = {"ee_mumu": "e+ e- > mu+ mu-", "uu_eeg": "u u~ > e+ e- g", "gg_ttgg": "g g > t t~ g g",
        "gg_tttt": "g g > t t~ t t~"}
BEYOND = 327_681                              # 10242 waves of the many-flow form, 5121 of the other


@pytest.mark.parametrize("precision", ["RWGT_MIXED_FP16", "RWGT_MIXED_BF16"])
@pytest.mark.parametrize("proc", list(TEXT))
def test_small_calls_equal_large_ones(proc, precision):
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    qcd = proc.startswith("gg")
    orig = synth.ORIG_QCD if qcd else synth.ORIG_EW
    rows = np.tile(np.asarray(orig.row(proc), dtype=np.float64), (3, 1))
    rows[:, 0 if qcd else -2] *= 1.0 + 0.01 * np.arange(1, 4)
    base = synth.events(proc, 1000)
    p = dev(np.tile(base, (BEYOND // 1000 + 1, 1, 1))[:BEYOND])
    w = torch.linspace(0.5, 2.0, BEYOND, dtype=torch.float64, device="cuda")
    with rw.Reweighter(TEXT[proc], orig.slha(), getattr(rw, precision)) as r:
        for guard in (0.0, 30.0):             # off; some events flagged
            rw.rwgt_set_mixed_guard(r.ctx, guard)
            big = torch.empty((3, BEYOND), dtype=torch.float64, device="cuda")
            r.eval(p, w, rows, big)
            big_me = torch.empty_like(big)
            r.me2(p, rows, big_me)
            big_kappa = torch.empty(BEYOND, dtype=torch.float64, device="cuda")
            rw.rwgt_cancellation(r.ctx, p, rows, big_kappa)
            for n in (1, 63, 65, 1000):
                out = torch.full((3 * n + 5,), -3.0, dtype=torch.float64, device="cuda")
                r.eval(p[:n].contiguous(), w[:n].contiguous(), rows, out[:3 * n])
                if guard:
                    kappa = big_kappa[:n].cpu().numpy()
                    # the call's kappa includes the original card: at least the new cards' maximum
                    assert rw.rwgt_mixed_guard_count(r.ctx) >= int((kappa > guard).sum())
                got = out.cpu().numpy()
                assert np.all(got[3 * n:] == -3.0)
                assert rel_err(got[:3 * n].reshape(3, n), big[:, :n].cpu().numpy()).max() <= 1e-15
                me = torch.empty((3, n), dtype=torch.float64, device="cuda")
                r.me2(p[:n].contiguous(), rows, me)
                assert rel_err(me.cpu().numpy(), big_me[:, :n].cpu().numpy()).max() <= 1e-15
                k = torch.empty(n, dtype=torch.float64, device="cuda")
                rw.rwgt_cancellation(r.ctx, p[:n].contiguous(), rows, k)
                assert rel_err(k.cpu().numpy(), big_kappa[:n].cpu().numpy()).max() <= 1e-15


@pytest.mark.parametrize("precision", ["RWGT_MIXED_FP16", "RWGT_MIXED_BF16"])
@pytest.mark.parametrize("proc,sizes", [("ee_mumu", (32_769,)), ("uu_eeg", (16_385, 77_777)),
                                        ("gg_ttgg", (4097, 20_011)), ("gg_tttt", (4097, 20_011))])
def test_a_wave_for_all_cards_equals_large_calls(proc, sizes, precision):
    """From two waves per SIMD on, a wave takes every card in turn instead of
    one: the first size that does, and a ragged one, bit for bit."""
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    qcd = proc.startswith("gg")
    orig = synth.ORIG_QCD if qcd else synth.ORIG_EW
    rows = np.tile(np.asarray(orig.row(proc), dtype=np.float64), (4, 1))
    rows[:, 0 if qcd else -2] *= 1.0 + 0.01 * np.arange(1, 5)
    p = dev(np.tile(synth.events(proc, 1000), (BEYOND // 1000 + 1, 1, 1))[:BEYOND])
    w = torch.linspace(0.5, 2.0, BEYOND, dtype=torch.float64, device="cuda")
    with rw.Reweighter(TEXT[proc], orig.slha(), getattr(rw, precision)) as r:
        for guard in (0.0, 30.0):
            rw.rwgt_set_mixed_guard(r.ctx, guard)
            big, big_me = (torch.empty((4, BEYOND), dtype=torch.float64, device="cuda") for _ in range(2))
            big_kappa = torch.empty(BEYOND, dtype=torch.float64, device="cuda")
            r.eval(p, w, rows, big)
            r.me2(p, rows, big_me)
            rw.rwgt_cancellation(r.ctx, p, rows, big_kappa)
            for n in sizes:
                ps, out = p[:n].contiguous(), torch.full((4 * n + 5,), -3.0, dtype=torch.float64, device="cuda")
                r.eval(ps, w[:n].contiguous(), rows, out[:4 * n])
                assert torch.equal(out[:4 * n].view(4, n), big[:, :n])
                assert bool((out[4 * n:] == -3.0).all())
                r.me2(ps, rows, out[:4 * n])
                assert torch.equal(out[:4 * n].view(4, n), big_me[:, :n])
                k = torch.empty(n, dtype=torch.float64, device="cuda")
                rw.rwgt_cancellation(r.ctx, ps, rows, k)
                assert torch.equal(k, big_kappa[:n])

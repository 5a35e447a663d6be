"""The training step as two kernels (rows, then the sums over rows) and as one:
every sum is in the same order, so gradients, loss and the parameters after
Adam steps are the same bits.  Rows: one tile and less, tiles beyond a round of
the sums kernel (16), a ragged last one; inputs given, and made from the pairs
of an event-card grid under every feature map."""
import ctypes

import numpy as np
import pytest

import synth
from gpu_util import dev, torch_cuda

pytestmark = pytest.mark.gpu
ONE, TWO = 0, 256                                # row tiles up to which a network takes two kernels


def _network(rw, form, n_in, width, depth):
    from paper_2510_05100_amd import _abi
    m = rw.rwgt_mlp_create(n_in, width, depth, 2, rw.RWGT_MLP_BF16, 5)
    rw.rwgt_mlp_set_stream(m, None)
    rw.rwgt_mlp_set_training(m, 0.01)
    force = _abi.load().rwgt_mlp_train_rows_tiles
    force.argtypes, force.restype = [ctypes.c_void_p, ctypes.c_int64], ctypes.c_int
    assert force(m, form) == 0
    return m


def _bits(x):
    return np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("width,depth", [(128, 2), (128, 3), (128, 9), (256, 4), (256, 9)])
def test_given_rows(width, depth):
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    gen = torch.Generator().manual_seed(width + depth)
    for n in (1, 63, 129, 1000, 2049, 4096, 5000):
        x = torch.zeros(((n + 63) // 64 * 64, 32))
        x[:n, :18] = torch.randn((n, 18), generator=gen)
        x, y = x.cuda(), torch.randn(n, generator=gen).cuda()
        got = []
        for form in (ONE, TWO):
            m = _network(rw, form, 18, width, depth)
            try:
                rw.rwgt_mlp_set_target_scale(m, 0.1, 0.7)
                loss = torch.zeros(4, dtype=torch.float32, device="cuda")
                rw.rwgt_mlp_train_step(m, x, y, n, 0.0, loss[:1])
                out = [rw.rwgt_mlp_get_grads(m)]
                for k in range(3):
                    rw.rwgt_mlp_train_step(m, x, y, n, 1e-3, loss[k + 1:k + 2])
                got.append([*out, rw.rwgt_mlp_get_grads(m), rw.rwgt_mlp_get_params(m), loss.cpu().numpy()])
            finally:
                rw.rwgt_mlp_destroy(m)
        for a, b in zip(*got):
            assert np.all(np.isfinite(a)) and np.any(a)
            np.testing.assert_array_equal(_bits(a), _bits(b), err_msg=f"{n} rows")


@pytest.mark.parametrize("proc,kind", [("ee_mumu", 0), ("ee_mumu", 1), ("uu_eeg", 0), ("uu_eeg", 1)])
def test_rows_of_a_grid(proc, kind):
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    p = dev(synth.events(proc, 700))
    npart = p.shape[1]
    cards = torch.as_tensor(np.stack([[c.MZ, c.WZ, c.sw2] for c in synth.batch_grid()[:5]]).astype(np.float32)).cuda()
    y = torch.randn((5, 700), generator=torch.Generator().manual_seed(2)).cuda()
    got = []
    for form in (ONE, TWO):
        m = _network(rw, form, rw.n_features(kind, npart), 128, 3)
        try:
            rw.rwgt_mlp_set_features(m, kind, npart, (2, 3), (91.188, 2.441))
            rw.rwgt_mlp_fit_grid(m, p, cards, y)
            losses = rw.rwgt_mlp_train(m, p, cards, y, 1100, 2, 1e-3, 1e-4, 3, 2)
            got.append((rw.rwgt_mlp_get_params(m), losses))
        finally:
            rw.rwgt_mlp_destroy(m)
    for a, b in zip(*got):
        assert np.all(np.isfinite(a))
        np.testing.assert_array_equal(_bits(a), _bits(b))

"""Training steps where the workspace of the two-kernel form cannot be had (too
little device memory): the one kernel gives the same bits, so the step is not
refused."""
import numpy as np
import pytest

from gpu_util import torch_cuda
from test_gpu_mixed_workspace import _fill

pytestmark = pytest.mark.gpu


def _network(rw, width, depth, stream=None):
    m = rw.rwgt_mlp_create(18, width, depth, 2, rw.RWGT_MLP_BF16, 5)
    rw.rwgt_mlp_set_stream(m, stream)
    rw.rwgt_mlp_set_target_scale(m, 0.0, 1.0)
    rw.rwgt_mlp_set_training(m, 0.01)
    return m


def _rows(torch, n):
    gen = torch.Generator().manual_seed(9)
    x = torch.zeros((n, 32))
    x[:, :18] = torch.randn((n, 18), generator=gen)
    return x.cuda(), torch.randn(n, generator=gen).cuda()


def test_nearly_full_card():
    """16,384 rows of the nine-layer network of width 256 want 296 MB of rows; the
    one kernel's workspace is there from a step on more rows."""
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    x, y = _rows(torch, 65_536)
    m, other = _network(rw, 256, 9), _network(rw, 256, 9)
    try:
        rw.rwgt_mlp_train_step(other, x, y, 16_384, 0.0)
        want = np.asarray(rw.rwgt_mlp_get_grads(other))
        rw.rwgt_mlp_destroy(other)
        other = None
        rw.rwgt_mlp_train_step(m, x, y, 65_536, 0.0)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        held = _fill(torch)
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(290 << 20, dtype=torch.uint8, device="cuda")
        rw.rwgt_mlp_train_step(m, x, y, 16_384, 0.0)
        torch.cuda.synchronize()
        del held
        torch.cuda.empty_cache()
        np.testing.assert_array_equal(np.asarray(rw.rwgt_mlp_get_grads(m)), want)
    finally:
        rw.rwgt_mlp_destroy(m)
        if other is not None:
            rw.rwgt_mlp_destroy(other)

"""Training steps where the workspace of the two-kernel form cannot be had (a
stream capture, too little device memory): the one kernel gives the same bits,
so the step is not refused."""
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


@pytest.mark.parametrize("width,depth", [(128, 3), (256, 4)])
@pytest.mark.parametrize("before", [(65_536,), (65_536, 1024), (1024,)])
def test_capture_of_a_small_step(width, depth, before):
    """The captured gradients of 1024 rows after steps on 65,536 rows (one
    kernel), on 1024 (two) and on both, and eager steps on the same network
    between the replays; on more rows, which replace a workspace, where the
    graph keeps the one kernel's."""
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    x, y = _rows(torch, 65_536)
    stream = torch.cuda.Stream()
    m, other = _network(rw, width, depth, stream.cuda_stream), _network(rw, width, depth)
    try:
        rw.rwgt_mlp_train_step(other, x, y, 1024, 0.0)
        torch.cuda.synchronize()
        want = np.asarray(rw.rwgt_mlp_get_grads(other))
        for n in before:
            rw.rwgt_mlp_train_step(m, x, y, n, 0.0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            rw.rwgt_mlp_train_step(m, x, y, 1024, 0.0)
        for n in (512, 1000, 900) if before == (1024,) else (2048, 4096, 65_536):
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(np.asarray(rw.rwgt_mlp_get_grads(m)), want)
            rw.rwgt_mlp_train_step(m, x, y, n, 0.0)
            torch.cuda.synchronize()
            assert np.any(np.asarray(rw.rwgt_mlp_get_grads(m)) != want)
    finally:
        rw.rwgt_mlp_destroy(m)
        rw.rwgt_mlp_destroy(other)


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

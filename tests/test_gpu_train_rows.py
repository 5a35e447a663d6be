"""The training step's two forms: rows and sums as two kernels (up to 256 row
tiles: 32768 rows at width 128, 16384 at 256) and the one-kernel form beyond.

Row counts are powers of two, so that the 1/n in every gradient scales the
BF16 operands exactly and two row counts differ in the order of FP32 sums only.
2e-4 relative in the 2-norm per layer: at most about 300 additions in sequence
(6e-8 each), times 10 for the cancellation of rows of either sign.
"""
import numpy as np
import pytest

from gpu_util import torch_cuda

pytestmark = pytest.mark.gpu
TOL = 2e-4


def _network(rw, width, depth):
    m = rw.rwgt_mlp_create(18, width, depth, 2, rw.RWGT_MLP_BF16, 5)
    rw.rwgt_mlp_set_stream(m, None)
    rw.rwgt_mlp_set_target_scale(m, 0.0, 1.0)
    rw.rwgt_mlp_set_training(m, 0.01)
    return m


def _grads(rw, m, x, y, n):
    rw.rwgt_mlp_train_step(m, x, y, n, 0.0)                      # gradients only
    return np.asarray(rw.rwgt_mlp_get_grads(m), dtype=np.float64)


def _check(got, want, width, depth):
    at = 0
    for layer in range(depth + 1):
        size = (18 if layer == 0 else width) * (width if layer < depth else 2)
        for count in (size, width if layer < depth else 2):
            a, b = got[at:at + count], want[at:at + count]
            assert np.linalg.norm(a - b) <= TOL * np.linalg.norm(b), (layer, count)
            at += count
    assert at == got.size


def _rows(torch, rw, m, n, seed):
    gen = torch.Generator().manual_seed(seed)
    x = torch.zeros((rw.rwgt_mlp_input_bytes(m, n) // 128, 32), dtype=torch.float32)
    x[:n, :18] = torch.randn((n, 18), generator=gen)
    return x, torch.randn(n, generator=gen)


@pytest.mark.parametrize("width,depth", [(128, 2), (128, 3), (256, 4), (256, 9)])
@pytest.mark.parametrize("n", [2, 16, 64, 256])
def test_rows_add_up(width, depth, n):
    """A step on n rows against the n steps on one row each."""
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    m = _network(rw, width, depth)
    try:
        x, y = _rows(torch, rw, m, n, 11 + n)
        want = 0.0
        one = torch.zeros((rw.rwgt_mlp_input_bytes(m, 1) // 128, 32), dtype=torch.float32, device="cuda")
        for i in range(n):
            one[0] = x[i].cuda()
            want = want + _grads(rw, m, one, y[i:i + 1].cuda(), 1) / n
        got = _grads(rw, m, x.cuda(), y.cuda(), n)
    finally:
        rw.rwgt_mlp_destroy(m)
    _check(got, want, width, depth)


@pytest.mark.parametrize("width,depth", [(128, 3), (256, 4)])
def test_two_kernels_against_one(width, depth):
    """1024 rows, and the same rows 64 times over (more tiles than the
    two-kernel form takes)."""
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    m = _network(rw, width, depth)
    try:
        x, y = _rows(torch, rw, m, 1024, 3)
        few = _grads(rw, m, x.cuda(), y.cuda(), 1024)
        many = _grads(rw, m, x[:1024].repeat(64, 1).cuda(), y.repeat(64).cuda(), 65536)
    finally:
        rw.rwgt_mlp_destroy(m)
    _check(many, few, width, depth)

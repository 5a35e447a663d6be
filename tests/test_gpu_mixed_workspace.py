"""Mixed-precision calls where the workspace of the wave-per-helicity form
cannot be had (a stream capture, too little device memory): the kernel without
it gives the same results, so the call is not refused."""
import numpy as np
import pytest

import synth
from gpu_util import PROCESS_TEXT, dev, torch_cuda

pytestmark = pytest.mark.gpu
BEYOND = 400_000                                 # events: a call without the workspace


def _setup(proc, nsets):
    torch = torch_cuda()
    qcd = proc.startswith("gg")
    orig = synth.ORIG_QCD if qcd else synth.ORIG_EW
    rows = np.tile(np.asarray(orig.row(proc), dtype=np.float64), (nsets, 1))
    rows[:, 0 if qcd else -2] *= 1.0 + 0.01 * np.arange(1, nsets + 1)
    p = dev(np.tile(synth.events(proc, 1000), (BEYOND // 1000, 1, 1)))
    return torch, orig, rows, p, torch.linspace(0.5, 2.0, BEYOND, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("proc,n", [("uu_eeg", 1000), ("gg_ttgg", 777), ("gg_tttt", 5000)])
def test_capture_of_a_small_call_after_a_large_one(proc, n):
    """The large call has allocated every buffer but the workspace; the graph
    of the small one is replayed between eager calls that allocate and replace
    it."""
    torch, orig, rows, p, w = _setup(proc, 2)
    import paper_2510_05100_amd as rw
    ps, ws = p[:n].contiguous(), w[:n].contiguous()
    stream = torch.cuda.Stream()
    with rw.Reweighter(PROCESS_TEXT[proc], orig.slha(), rw.RWGT_MIXED_FP16) as r:
        rw.rwgt_set_stream(r.ctx, stream.cuda_stream)
        torch.cuda.synchronize()
        big = torch.empty((2, BEYOND), dtype=torch.float64, device="cuda")
        r.eval(p, w, rows, big)
        torch.cuda.synchronize()
        small = torch.zeros((2, n), dtype=torch.float64, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            r.eval(ps, ws, rows, small)
        for m in (n, 2 * n, 4 * n):
            small.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(small, big[:, :n])
            out = torch.empty((2, m), dtype=torch.float64, device="cuda")
            r.eval(p[:m].contiguous(), w[:m].contiguous(), rows, out)
            torch.cuda.synchronize()
            assert torch.equal(out, big[:, :m])


def _fill(torch):
    """Allocations that leave 128 to 256 MB of device memory."""
    spare, held = torch.empty(128 << 20, dtype=torch.uint8, device="cuda"), []
    for size in (32 << 30, 4 << 30, 512 << 20, 128 << 20):
        while True:
            try:
                held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
            except torch.OutOfMemoryError:
                break
    del spare
    torch.cuda.empty_cache()
    return held


def test_nearly_full_card():
    """60,000 g g -> t t~ g g events under 9 cards want 276 MB of workspace."""
    torch, orig, rows, p, w = _setup("gg_ttgg", 8)
    import paper_2510_05100_amd as rw
    n = 60_000
    ps, ws = p[:n].contiguous(), w[:n].contiguous()
    with rw.Reweighter(PROCESS_TEXT["gg_ttgg"], orig.slha(), rw.RWGT_MIXED_FP16) as r:
        big, out = (torch.empty((8, m), dtype=torch.float64, device="cuda") for m in (BEYOND, n))
        r.eval(p, w, rows, big)
        assert rw.rwgt_nonfinite(r.ctx) == 0
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        held = _fill(torch)
        print("free", torch.cuda.mem_get_info()[0] >> 20, "MB", flush=True)
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(276_480_000, dtype=torch.uint8, device="cuda")
        r.eval(ps, ws, rows, out)
        torch.cuda.synchronize()
        del held
        torch.cuda.empty_cache()
        assert torch.equal(out, big[:, :n])
        r.eval(ps, ws, rows, out)                # with the workspace
        torch.cuda.synchronize()
        assert torch.equal(out, big[:, :n])

"""The count of non-finite outputs after a call whose kernel was not launched
(its stream's capture had been invalidated): nothing was evaluated, so 0 and not
what an earlier call left."""
import ctypes

import numpy as np
import pytest

import synth
from gpu_util import PROCESS_TEXT, dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("proc", ["ee_mumu", "gg_ttgg"])
def test_no_count_after_a_failed_launch(proc):
    torch = torch_cuda()
    import paper_2510_05100_amd as rw
    with open("/proc/self/maps") as f:           # the runtime that torch and the library share
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    orig = synth.ORIG_QCD if proc.startswith("gg") else synth.ORIG_EW
    p = dev(synth.events(proc, 40))
    w = torch.full((40,), float("nan"), dtype=torch.float64, device="cuda")
    out = torch.empty((1, 40), dtype=torch.float64, device="cuda")
    row = orig.row(proc)
    stream, graph, memory = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    torch.cuda.synchronize()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    with rw.Reweighter(PROCESS_TEXT[proc], orig.slha(), rw.RWGT_FP64) as r:
        rw.rwgt_set_stream(r.ctx, stream.value)
        r.eval(p, w, row, out)
        assert rw.rwgt_nonfinite(r.ctx) == 40
        assert hip.hipStreamBeginCapture(stream, 1) == 0          # thread-local: an allocation invalidates it
        assert hip.hipMalloc(ctypes.byref(memory), ctypes.c_size_t(1 << 20)) != 0
        with pytest.raises(rw.RwgtError, match="EDEVICE"):
            r.eval(p, w, row, out)
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) != 0
        hip.hipGetLastError()
        assert rw.rwgt_nonfinite(r.ctx) == 0
        r.eval(p, w, row, out)
        assert rw.rwgt_nonfinite(r.ctx) == 40
        torch.cuda.synchronize()
        assert np.all(np.isnan(out.cpu().numpy()))
        rw.rwgt_set_stream(r.ctx, None)
    assert hip.hipStreamDestroy(stream) == 0

"""Double-precision QCD calls of any number of events: half a wave per event,
and a launch holds fewer than 2^32 work-items.  The ranges the call is launched
in (tests/host/launch_shape.cpp, the library's own function) on the CPU, and a
call beyond one launch on the GPU."""
import os
import shutil
import subprocess

import pytest

import synth
from gpu_util import PROCESS_TEXT, dev, torch_cuda

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("shape") / "launch_shape")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "paper_2510_05100_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "launch_shape.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.mark.parametrize("nevt", [1, 2, 3, 8192, 1_000_001, 2**26 - 1, 2**26, 2**26 + 1, 2**27 - 1, 2**27, 2**27 + 1,
                                  2**30, 2**31 + 3])
def test_launches_cover_every_event_once(exe, nevt):
    r = subprocess.run([exe, str(nevt)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    at = 0
    for line in r.stdout.splitlines():
        first, groups = map(int, line.split())
        assert first == at
        assert 1 <= groups and groups * 64 < 2**32
        at = first + 2 * groups                   # a workgroup: two events
    assert nevt <= at <= nevt + 1


@pytest.mark.gpu
@pytest.mark.parametrize("proc", ["gg_ttgg", "gg_tttt"])
def test_more_events_than_one_launch_holds(proc):
    """2^27 + 1 events (26 GB of momenta), a sample of 1000 over and over:
    every copy of an event gets that event's |M|^2, the same bits."""
    import paper_2510_05100_amd as rw
    torch = torch_cuda()
    n, base = 2**27 + 1, dev(synth.events(proc, 1000))
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of free device memory")
    row = synth.ORIG_QCD.row(proc)
    torch.cuda.empty_cache()
    p = torch.empty((n, 6, 4), dtype=torch.float64, device="cuda")
    whole = n // 1000 * 1000
    p[:whole].view(-1, 1000, 6, 4).copy_(base.expand(whole // 1000, 1000, 6, 4))
    p[whole:].copy_(base[:n - whole])
    me = torch.full((1, n), -1.0, dtype=torch.float64, device="cuda")
    want = torch.empty((1, 1000), dtype=torch.float64, device="cuda")
    with rw.Reweighter(PROCESS_TEXT[proc], synth.ORIG_QCD.slha(), rw.RWGT_FP64) as r:
        r.me2(base, row, want)
        r.me2(p, row, me)
        assert rw.rwgt_nonfinite(r.ctx) == 0
        assert bool((me[0, :whole].view(-1, 1000) == want[0]).all())
        assert torch.equal(me[0, whole:], want[0, :n - whole])
    del p, me
    torch.cuda.empty_cache()

"""Where the mixed path takes a wave per helicity, on the CPU: at sizes where that
was measured to be the faster form, and not where the kernel that loops over
the helicities was, whose full rounds of waves have nothing idle."""
import ctypes

import pytest

EE, UU, TTGG, TTTT = range(4)


def _parts(proc, nevt, ncards):
    from paper_2510_05100_amd import _abi
    f = getattr(_abi.load(), "_ZN4rwgt14me_parts_bytesEili")      # rwgt::me_parts_bytes(int, int64_t, int)
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int64, ctypes.c_int], ctypes.c_size_t
    return f(proc, nevt, ncards)


@pytest.mark.parametrize("proc,ncards,nevt", [
    (TTGG, 2, 1), (TTGG, 2, 777), (TTGG, 2, 26_214), (TTGG, 2, 34_406), (TTGG, 2, 58_982), (TTGG, 2, 91_750),
    (TTGG, 2, 100_000), (TTGG, 2, 212_992), (TTTT, 2, 29_491), (TTTT, 2, 49_152), (TTTT, 2, 88_473), (TTTT, 2, 147_456),
    (TTTT, 2, 209_715), (TTTT, 2, 301_465), (UU, 2, 1), (UU, 4, 77_777), (UU, 2, 140_000), (UU, 2, 212_992),
    (EE, 4, 10_000), (EE, 8, 163_840)])
def test_taken_where_faster(proc, ncards, nevt):
    assert _parts(proc, nevt, ncards) > 0


@pytest.mark.parametrize("proc,ncards,nevt", [
    (TTGG, 2, 31_129), (TTGG, 2, 32_768), (TTGG, 2, 65_536), (TTGG, 2, 98_304), (TTGG, 4, 98_304), (TTGG, 2, 131_072),
    (TTGG, 2, 327_680), (TTTT, 2, 32_768), (TTTT, 2, 62_259), (TTTT, 2, 95_027), (TTTT, 4, 131_072), (TTTT, 2, 163_840),
    (TTTT, 2, 222_822), (TTTT, 2, 327_680), (UU, 2, 196_608), (UU, 2, 245_760), (UU, 2, 262_144), (UU, 4, 262_144),
    (EE, 4, 196_608), (EE, 8, 262_144), (EE, 2, 1000), (TTGG, 2, 1_000_000), (UU, 2, 500_000)])
def test_not_taken_where_slower(proc, ncards, nevt):
    assert _parts(proc, nevt, ncards) == 0

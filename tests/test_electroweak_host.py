"""The weights of the double-precision electroweak kernels (csrc/electroweak.h),
compiled for the host, against the oracle's explicit Dirac matrices: generic
events, momenta rounded to ten digits (neither exactly massless nor exactly
conserved, as an event file holds them), and particles along the axis where a
spinor's phase is undefined.

1e-12 (e+ e- > mu+ mu-) and 1e-11 (u u~ > e+ e- g, whose two diagrams cancel):
the bars of the device's FP64 path against the same oracle.
"""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth
from oracle import reweight

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROC = {"ee_mumu": (4, 0.25, 1e-12), "uu_eeg": (5, 1.0 / 36.0, 1e-11)}


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("electroweak") / "electroweak_me")
    cmd = [hipcc, "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2510_05100_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "electroweak_me.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


def _run(exe, name, p, card):
    npart, average, _ = PROC[name]
    e, gs = math.sqrt(4 * math.pi / card.aEWM1), math.sqrt(4 * math.pi * card.aS)
    gz = e / math.sqrt(card.sw2 * (1 - card.sw2))
    charge, t3 = (-1.0, -1.0, 2 / 3, 2 / 3), (-0.5, -0.5, 0.5, 0.5)
    c = [gs] + [-e * q for q in charge] + [-gz * (t - q * card.sw2) for q, t in zip(charge, t3)]
    c += [gz * q * card.sw2 for q in charge] + [card.MZ, card.WZ]
    text = f"{npart} {p.shape[0]} {average!r}\n" + " ".join("%.17g" % x for x in c) + "\n"
    text += "\n".join(" ".join("%.17g" % x for x in ev.reshape(-1)) for ev in p)
    r = subprocess.run([exe], input=text, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return np.array([float(x) for x in r.stdout.split()])


@pytest.mark.parametrize("name", list(PROC))
@pytest.mark.parametrize("digits", [17, 10])
def test_weights_against_oracle(exe, name, digits):
    p = synth.events(name, 300, seed=41)
    p = np.vectorize(lambda x: float(f"{x:.{digits - 1}e}"))(p)
    for card in (synth.ORIG_EW, synth.NEW_UU):
        np.testing.assert_allclose(_run(exe, name, p, card), reweight.me2(name, p, card), rtol=PROC[name][2])


@pytest.mark.parametrize("name,particle", [("ee_mumu", 2), ("ee_mumu", 3), ("uu_eeg", 2), ("uu_eeg", 3), ("uu_eeg", 4)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_particle_along_the_axis(exe, name, particle, sign):
    """One event whose momenta are permuted to beams along x and rotated so
    that the given particle lies exactly on +z or -z."""
    p = synth.events(name, 1, seed=43)[0]
    v = p[particle, 1:] / p[particle, 0]
    a = np.cross(v, [0.0, 0.0, sign])
    s, c = np.linalg.norm(a), v[2] * sign
    k = a / s
    for n in range(p.shape[0]):
        u = p[n, 1:].copy()
        p[n, 1:] = u * c + np.cross(k, u) * s + k * (k @ u) * (1 - c)
    p[particle, 1:] = [0.0, 0.0, sign * p[particle, 0]]
    got = _run(exe, name, p[None], synth.ORIG_EW)
    np.testing.assert_allclose(got, reweight.me2(name, p[None], synth.ORIG_EW), rtol=PROC[name][2])

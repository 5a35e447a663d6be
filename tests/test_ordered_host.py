"""The colour-ordered recursions of the double-precision kernels of
g g -> t t~ g g (csrc/ordered.h) and g g -> t t~ t t~ (csrc/ordered_pairs.h), compiled for the host with one thread per lane
(tests/host/ordered_me.cpp), against the oracle: the tasks' index arithmetic,
the relations between orderings and the vertices, without a GPU.

1e-12 relative, the bar of the generated code on the host: both sides are
double-precision sums of the same flows (24, 12) in different orders.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth
from oracle import reweight

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build(tmp_path_factory, *flags):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("ordered") / "ordered_me")
    cmd = [hipcc, *flags, "-O1", "-std=c++17", "-pthread", "-I" + os.path.join(ROOT, "paper_2510_05100_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "ordered_me.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return _build(tmp_path_factory)


def _run(exe, p, card):
    text = f"{p.shape[0]} {card.aS!r} {card.MT!r}\n" + "\n".join(
        " ".join("%.17g" % x for x in ev.reshape(-1)) for ev in p)
    r = subprocess.run([exe], input=text, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return np.array([float(x) for x in r.stdout.split()])


def test_recursion_on_host_against_oracle(exe):
    p = synth.events("gg_ttgg", 200)[::10]
    for card in (synth.ORIG_QCD, synth.NEW_QCD):
        np.testing.assert_allclose(_run(exe, p, card), reweight.me2("gg_ttgg", p, card), rtol=1e-12)


def test_gluons_along_the_beam(exe):
    """Azimuth undefined (a final gluon along -z or +z): still the oracle's value."""
    p = synth.events("gg_ttgg", 8)
    q = p.copy()
    for e, (which, sign) in enumerate([(4, -1.0), (4, 1.0), (5, -1.0), (5, 1.0)]):
        # rotate the final state so that the gluon lies on the axis
        v = p[e, which, 1:] / p[e, which, 0]
        a = np.cross(v, [0.0, 0.0, sign])
        s, c = np.linalg.norm(a), v[2] * sign
        k = a / s
        for n in range(2, 6):
            u = p[e, n, 1:]
            q[e, n, 1:] = u * c + np.cross(k, u) * s + k * (k @ u) * (1 - c)
        q[e, which, 1:] = [0.0, 0.0, sign * p[e, which, 0]]
        q[e, 2, 1:] -= q[e, 2:, 1:].sum(axis=0)                  # rounding of the rotation
    # collinear with a beam the squared amplitude is singular: take the beams along x instead
    q[:, 0, 1:] = q[:, 0, [3, 1, 2]]
    q[:, 1, 1:] = q[:, 1, [3, 1, 2]]
    got, want = _run(exe, q[:4], synth.ORIG_QCD), reweight.me2("gg_ttgg", q[:4], synth.ORIG_QCD)
    np.testing.assert_allclose(got, want, rtol=1e-11)


def test_pairs_on_host_against_oracle(tmp_path_factory):
    pairs = _build(tmp_path_factory, "-DPAIRS")
    p = synth.events("gg_tttt", 200)[::10]
    for card in (synth.ORIG_QCD, synth.NEW_QCD):
        np.testing.assert_allclose(_run(pairs, p, card), reweight.me2("gg_tttt", p, card), rtol=1e-12)

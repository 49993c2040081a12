"""The sphere lists that a step's setup reads for its ground point, and the rule when a
search over them is worth it.

CPU: the host builder's lists against brute force.  GPU: records of showers over large
arrays, with few and many bunches a step (both sides of the rule), are the oracle's, and
time at 60 degrees, where the light lands a kilometre from the axis's ground point, grows
less than the array (with every step past all spheres: five to seven times as long for
1024 spheres as for 100)."""
import dataclasses
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2006_14927_amd import synth
from test_light_cone_directions import _us

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lists_program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("reach") / "check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2006_14927_amd/csrc",
                    f"{ROOT}/tests/golden/reach_lists_check.cpp", "-o", out], check=True)
    return out


@pytest.mark.parametrize("n,half,cx", [(32, 500.0, 0.0), (33, 500.0, 0.0), (33, 0.001, 0.0), (100, 1000.0, 0.0),
                                       (400, 2000.0, 3e5), (1024, 3200.0, -1e4), (1024, 4.9e5, 0.0),
                                       (64, 6e5, 0.0)])
def test_lists_hold_every_near_sphere(lists_program, n, half, cx):
    r = subprocess.run([lists_program, str(n), repr(half), repr(cx)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def disk(n):
    return synth.telescopes_disk(n, disk_radius=1000.0 * np.sqrt(n / 100.0))


def shower(zenith, n):
    return synth.shower_segments(1, n, synth.layered_atmosphere(), zenith_deg=zenith, xmax=400.0)


@pytest.mark.gpu
@pytest.mark.parametrize("bunch", [0.5, 5.0, 50.0, 500.0])
@pytest.mark.parametrize("zenith,scale", [(20.0, 1.0), (60.0, 1.0), (75.0, 1.0), (60.0, 30.0), (60.0, 400.0)])
def test_large_arrays_match_the_oracle(bunch, zenith, scale):
    from gpu_helpers import compare_records, gpu_run
    from paper_2006_14927_amd import ckv
    t = disk(1024)
    # spread arrays keep a cluster of spheres about the shower
    far = np.hypot(t.x, t.y) > 900.0
    tels = synth.Telescopes(np.where(far, t.x * scale, t.x), np.where(far, t.y * scale, t.y), t.r)
    n = 400 if bunch < 1 else 3000
    wl = dataclasses.replace(synth.single_tev(1000), segs=shower(zenith, n), tels=tels, bunch_size=bunch)
    cfg = oracle.Config.from_workload(wl)
    compare_records(wl, cfg, oracle.run(cfg, wl.segs, nthreads=8), gpu_run(wl, ckv.CKV_FP64), ckv.CKV_FP64)


@pytest.mark.gpu
@pytest.mark.parametrize("bunch", [5.0, 50.0])
def test_inclined_showers_over_large_arrays(bunch):
    from gpu_helpers import handles, params
    from paper_2006_14927_amd import ckv
    us = []
    for n in (100, 1024):
        wl = dataclasses.replace(synth.single_tev(1000), segs=shower(60.0, 200_000), tels=disk(n), bunch_size=bunch)
        atmo, tels = handles(wl)
        us.append(_us(ckv.Runner(ckv.DeviceSegments(wl.segs), atmo, tels, params(wl, ckv.CKV_MIXED), 1 << 21)))
    print(f"100 spheres {us[0]:.0f} us, 1024 {us[1]:.0f} us")
    assert us[1] < 3.0 * us[0]

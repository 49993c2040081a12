"""Directions that are unit only to the precision they were stored in.

The azimuth sectors' bound of a step (test_light_cone restates it) holds for directions of
length other than 1 as well, widened by a multiple of off = |length^2 - 1|.  On the CPU:
every crossing bunch of the oracle has its sector set, with directions rounded to FP32 or to
five digits.  On the GPU: such a shower's records are the oracle's, and it takes about as
long as the same shower with unit directions (without a bound every bunch is propagated:
three times as long)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2006_14927_amd import synth
from test_light_cone import R_EARTH, light_cone, sector_masks


def rounded(segs, how):
    f = (lambda x: x.astype(np.float32).astype(np.float64)) if how == "fp32" else (lambda x: np.round(x, 5))
    return dataclasses.replace(segs, u=f(segs.u), v=f(segs.v), w=f(segs.w))


def widened(segs, sd, base, w_unit, tels, h_obs, earth_r, psi):
    """The terms in off added to the unit step's bound (looser for shells: the unit step's
    smallest cosine of any of its rays)."""
    off = np.abs(segs.u ** 2 + segs.v ** 2 + segs.w ** 2 - 1)
    st, ct = sd["sin_t"], sd["cos_t"]
    wp = w_unit * ct - np.sqrt(np.maximum(0, 1 - w_unit ** 2)) * st - (0.51 + 1.7 * st) * off
    dh0 = segs.h0 - h_obs
    if earth_r > 0:
        return base + off / wp ** 2 * ((8 + 12 * st) * dh0 / wp + (4 + 4 * st) * tels.r.max() + 3 * base), off
    wo2 = wp ** 2
    if not np.all(np.diff(psi) <= 0):
        wo2 = 1 - (1 + psi.max()) / (1 + psi.min()) * (1 - wp ** 2)
    return base + off * ((5 + 8 * st) * dh0 / wp ** 2 + (5 + 8 * st) * tels.r.max() / wo2 + 3 * base), off


def cases():
    yield "tev_fp32", synth.single_tev(3000), "fp32", 0.0
    yield "tev_5_digits", synth.single_tev(3000), "digits", 0.0
    yield "hadron_60_5_digits", synth.hadron_like(60.0, 2000), "digits", 0.0
    wl = synth.single_tev(2000)
    bumpy = dataclasses.replace(wl.atmo, eta=wl.atmo.eta * (1 + 0.05 * np.sin(wl.atmo.alt / 900.0)))
    yield "not_monotone_5_digits", dataclasses.replace(wl, atmo=bumpy), "digits", 0.0
    yield "curved_40_fp32", synth.inclined(40.0, 1500), "fp32", R_EARTH
    yield "curved_70_fp32", synth.inclined(70.0, 4000), "fp32", R_EARTH


@pytest.mark.parametrize("name,wl,how,earth_r", list(cases()), ids=[c[0] for c in cases()])
def test_every_crossing_has_its_sector(name, wl, how, earth_r):
    segs = rounded(wl.segs, how)
    cfg = oracle.Config(oracle.build_tables(wl.atmo.alt, wl.atmo.eta, wl.atmo.obs_level), wl.tels.x, wl.tels.y,
                        wl.tels.r, seed=wl.seed, earth_radius=earth_r)
    sd = oracle.segment_details(cfg, segs)
    length = np.sqrt(segs.u ** 2 + segs.v ** 2 + segs.w ** 2)
    unit = dataclasses.replace(segs, u=segs.u / length, v=segs.v / length, w=segs.w / length)
    ok, px, py, base = light_cone(unit, sd, cfg.tables.grid(), cfg.psi, wl.tels, wl.atmo.obs_level, earth_r)
    base, off = widened(segs, sd, base, unit.w, wl.tels, wl.atmo.obs_level, earth_r, cfg.psi)
    assert off.max() > 1e-8
    ok &= off <= (1e-6 if earth_r else 1e-4)
    mask, _ = sector_masks(segs, sd, ok, px, py, base, wl.tels, wl.atmo.obs_level)
    nb = sd["n_b"].astype(np.int64)
    seg = np.repeat(np.arange(len(nb)), nb)
    k = np.arange(len(seg)) - np.repeat(np.cumsum(nb) - nb, nb)
    bd = oracle.bunch_details(cfg, segs, seg, k)
    assert np.all(bd["status"][ok[seg]] < 0)
    dx = bd["x_g"][:, None] - wl.tels.x[None, :]
    dy = bd["y_g"][:, None] - wl.tels.y[None, :]
    b = dx * bd["u_o"][:, None] + dy * bd["v_o"][:, None]
    crosses = (bd["status"] < 0) & (b * b - (dx * dx + dy * dy - wl.tels.r[None, :] ** 2) >= 0).any(1)
    taken = mask[seg, bd["r"][:, 1] >> 24]
    assert crosses.sum() > 20
    assert np.all(taken[crosses])
    assert taken.mean() < 0.5


def _us(runner, reps=5):
    import torch
    runner.run()
    t = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            runner.run()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b) * 250.0)
    return sorted(t)[reps // 2]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_rounded_directions_keep_their_bound(precision):
    from gpu_helpers import compare_records, gpu_run, handles, params
    from paper_2006_14927_amd import ckv
    for wl, how, earth_r in ((synth.single_tev(3000), "fp32", 0.0), (synth.single_tev(3000), "digits", 0.0),
                             (synth.hadron_like(60.0, 4000), "digits", 0.0), (synth.inclined(70.0, 4000), "fp32", R_EARTH)):
        segs = rounded(wl.segs, how)
        cfg = oracle.Config(oracle.build_tables(wl.atmo.alt, wl.atmo.eta, wl.atmo.obs_level), wl.tels.x, wl.tels.y,
                            wl.tels.r, seed=wl.seed, earth_radius=earth_r)
        g = gpu_run(wl, precision, segs=segs, earth_radius=earth_r)
        compare_records(wl, cfg, oracle.run(cfg, segs, nthreads=8), g, precision, segs=segs)
    big = synth.single_tev(300_000)
    atmo, tels = handles(big)
    us = [_us(ckv.Runner(ckv.DeviceSegments(s), atmo, tels, params(big, precision), 1 << 20))
          for s in (big.segs, rounded(big.segs, "fp32"))]
    print(f"unit {us[0]:.0f} us, rounded to FP32 {us[1]:.0f} us")
    assert us[1] < 1.5 * us[0]

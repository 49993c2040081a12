"""The bunch kernel's azimuth sectors, checked on the oracle's bunches (CPU).

A bunch goes through the first pass only if the sector of its azimuth, the top bits of
its second draw, is set in its step's mask: the mask holds the windows of azimuth in
which the step's light can reach some sphere, from a bound of the distance between the
observed line and the straight emission line.  This test restates the bound in numpy and
checks that every bunch that crosses a sphere has its sector set, and that no bunch of a
step with a bound is dropped, for gamma and hadron-like showers (muons, wide cones) at
several zenith angles, node tables, spheres of very uneven size, a profile whose index is
not monotone, and spherical shells."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2006_14927_amd import synth

W_MIN = 0.1
SECTORS = 256
R_EARTH = 6.371e6


def altitude(R, x, y, z):
    q = x * x + y * y
    rz = R + z
    return (q + z * (2.0 * R + z)) / (np.sqrt(q + rz * rz) + R)


def light_cone(segs, sd, h_nodes, psi, tels, h_obs, earth_r=0.0, w_min=W_MIN):
    """Per step: whether the bound holds, the shifted start point and the bound."""
    falls = bool(np.all(np.diff(psi) <= 0))
    slope = np.max(np.abs(np.diff(psi)) / np.diff(h_nodes))
    p_max, p_min, h_top = psi.max(), psi.min(), h_nodes[-1]
    rmax, dmax = tels.r.max(), np.hypot(tels.x, tels.y).max()
    u, v, w, L, ct, st = segs.u, segs.v, segs.w, segs.length, sd["cos_t"], sd["sin_t"]
    dh0 = segs.h0 - h_obs
    ok = (sd["status"] < 0) & (sd["n_b"] > 0) & (np.abs(u * u + v * v + w * w - 1) <= 1e-9) & (w >= 0.05)
    with np.errstate(all="ignore"):
        s_hi = st * (1 + 1e-9) + 1e-12
        sa = np.sqrt(np.maximum(0, (1 - w) * (1 + w)))
        wp = w * ct - sa * s_hi - 1e-12
        ok &= (wp >= 0.03) & (wp > w_min + 1e-6)
        x_psi = (np.maximum(p_max - (sd["n_mid"] ** 2 - 1) + slope * 0.5 * L, 0) if falls
                 else np.full_like(L, p_max - p_min))
        iw = 1 / wp
        m = 0.05 + dh0 * 1e-6 * iw
        px, py = segs.x0.copy(), segs.y0.copy()
        if earth_r > 0:
            R = earth_r
            r0 = np.sqrt(segs.x0 ** 2 + segs.y0 ** 2 + (R + segs.h0) ** 2)
            x1, y1, h1 = segs.x0 + L * u, segs.y0 + L * v, segs.h0 - L * w
            alt0, alt1 = altitude(R, segs.x0, segs.y0, segs.h0), altitude(R, x1, y1, h1)
            c1 = (w * (R + h1) - u * x1 - v * y1) / (R + alt1)
            c_lo = c1 * ct - np.sqrt(np.maximum(0, (1 - c1) * (1 + c1))) * s_hi - 1e-12
            s_max = r0 / (R + h_obs) * np.sqrt((1 - c_lo) * (1 + c_lo)) * (1 + 1e-9)
            ok &= falls & (c1 > 0.03) & (c_lo > 0.03) & (s_max < 0.9995) & (alt0 < h_top - 1)
            c_ray = np.sqrt((1 - s_max) * (1 + s_max))
            bend = s_max / c_ray * 0.5 * x_psi * (1 + 1e-6)
            ok &= wp - bend >= 0.03
            reach = rmax / (wp - bend)
            base = (bend * (alt0 - h_obs) / c_ray + 0.51 * (dmax + reach) ** 2 / (R + h_obs) + reach * bend
                    + m + 1e-6 * (alt0 - h_obs) / c_ray)
            ok &= alt1 - h_obs > rmax + base + 1
        else:
            x0 = x_psi / (1 + p_min)
            ok &= (x0 * iw * iw <= 0.5) & (segs.h0 < h_top - 1)
            B = (0.5 if falls else 0.8) * x0 * iw * iw
            t_max = np.sqrt((1 - wp) * (1 + wp)) * iw
            beta0 = 0.5 * B if falls else 0 * B
            wo2 = wp * wp
            if not falls:
                wo2 = 1 - (1 + p_max) / (1 + p_min) * (1 - wp) * (1 + wp)
                ok &= wo2 > 1e-3
            m = m + dh0 * ((1e-6 * st + 2e-9) * (iw + iw * iw) + 4e-6 * p_max * iw ** 3)
            base = ((B - beta0) * t_max * dh0 + beta0 * (s_hi * iw / w * dh0 + sa * L)
                    + rmax / np.sqrt(wo2) * (0.51 * x0 * (1 + 2 * iw)) + m)
            px = segs.x0 - beta0 * dh0 * u / w
            py = segs.y0 - beta0 * dh0 * v / w
        ok &= dh0 - L * w > rmax + base + 1
    return ok, px, py, base


def sector_masks(segs, sd, ok, px, py, base, tels, h_obs):
    """(steps, SECTORS) booleans; all set where there is no bound."""
    mask = np.zeros((segs.n, SECTORS), dtype=bool)
    mask[~ok] = True
    i = np.nonzero(ok)[0]
    ct, st = sd["cos_t"][i], sd["sin_t"][i]
    t = st / ct
    b1, b2 = (np.stack([sd[f + c][i] for c in "xyz"], 1) for f in ("b1", "b2"))
    pairs = 0
    for k in range(tels.n):
        q = np.stack([tels.x[k] - px[i], tels.y[k] - py[i], h_obs - segs.h0[i]], 1)
        A = q[:, 0] * segs.u[i] + q[:, 1] * segs.v[i] - q[:, 2] * segs.w[i]
        v1, v2 = (q * b1).sum(1), (q * b2).sum(1)
        n = np.hypot(v1, v2)
        rho = tels.r[k] * 1.00001 + base[i]
        rc = rho / ct + 1e-5 * n
        hit = (n <= t * A + rc) & (n >= t * (A - segs.length[i]) - rc)
        pairs += hit.sum()
        for j in np.nonzero(hit)[0]:
            q2 = (rho[j] / n[j]) ** 2 if n[j] > 0 else 1.0
            if not q2 < 0.64:
                mask[i[j]] = True
                continue
            half = np.sqrt(q2 / (1 - q2)) * 0.15916 + 2e-5
            mid = np.arctan2(v2[j], v1[j]) / (2 * np.pi)
            lo, hi = int(np.floor((mid - half) * SECTORS)), int(np.floor((mid + half) * SECTORS))
            mask[i[j], np.arange(lo, hi + 1) % SECTORS] = True
    return mask, pairs


def cases():
    for z in (0.0, 20.0, 45.0, 60.0):
        wl = synth.hadron_like(z, 1500)
        yield f"hadron_{z:.0f}", wl, {}
    yield "gamma", synth.vertical_gamma(2500), {}
    yield "tev", synth.single_tev(3000), {}
    wl = synth.single_tev(2000)
    r = np.where(np.arange(wl.tels.n) % 7 == 0, 60.0, 2.0)
    yield "uneven_spheres", dataclasses.replace(wl, tels=dataclasses.replace(wl.tels, r=r)), {}
    bumpy = dataclasses.replace(wl.atmo, eta=wl.atmo.eta * (1 + 0.05 * np.sin(wl.atmo.alt / 900.0)))
    yield "not_monotone", dataclasses.replace(wl, atmo=bumpy), {}
    yield "node_tables", dataclasses.replace(wl, atmo=synth.sparse_atmosphere()), dict(nodes=True)
    yield "inclined_70", synth.inclined(70.0, 2500), {}
    for z in (0.0, 60.0, 70.0, 80.0):
        yield f"curved_{z:.0f}", synth.inclined(z, 1500 if z < 65 else 4000), dict(earth_radius=R_EARTH)


@pytest.mark.parametrize("name,wl,kw", list(cases()), ids=[c[0] for c in cases()])
def test_every_crossing_has_its_sector(name, wl, kw):
    earth_r = kw.get("earth_radius", 0.0)
    build = oracle.build_node_tables if kw.get("nodes") else oracle.build_tables
    cfg = oracle.Config(build(wl.atmo.alt, wl.atmo.eta, wl.atmo.obs_level), wl.tels.x, wl.tels.y, wl.tels.r,
                        seed=wl.seed, earth_radius=earth_r)
    sd = oracle.segment_details(cfg, wl.segs)
    ok, px, py, base = light_cone(wl.segs, sd, cfg.tables.grid(), cfg.psi, wl.tels, wl.atmo.obs_level, earth_r)
    mask, pairs = sector_masks(wl.segs, sd, ok, px, py, base, wl.tels, wl.atmo.obs_level)
    nb = sd["n_b"].astype(np.int64)
    seg = np.repeat(np.arange(len(nb)), nb)
    k = np.arange(len(seg)) - np.repeat(np.cumsum(nb) - nb, nb)
    bd = oracle.bunch_details(cfg, wl.segs, seg, k)
    # no drop among the steps with a bound
    assert np.all(bd["status"][ok[seg]] < 0)
    dx = bd["x_g"][:, None] - wl.tels.x[None, :]
    dy = bd["y_g"][:, None] - wl.tels.y[None, :]
    b = dx * bd["u_o"][:, None] + dy * bd["v_o"][:, None]
    disc = b * b - (dx * dx + dy * dy - wl.tels.r[None, :] ** 2)
    crosses = (bd["status"] < 0) & (disc >= 0).any(1)
    taken = mask[seg, bd["r"][:, 1] >> 24]
    assert crosses.sum() > 20
    assert np.all(taken[crosses])
    print(f"{name}: bound on {ok[sd['status'] < 0].mean():.3f} of the steps, {nb[mask.any(1)].sum() / nb.sum():.3f} of "
          f"the bunches in the pass, {taken.mean():.4f} taken, {crosses.mean():.4f} cross, "
          f"{pairs / max(ok.sum(), 1):.2f} spheres a step")
    if not name.startswith("curved_80"):
        assert taken.mean() < 0.5

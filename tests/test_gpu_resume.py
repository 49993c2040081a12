"""Runs cut short by a full output and resumed at their cursors until done: per (shower,
telescope) the records, ids and counts of the parts concatenate to the whole run's, through
the small tiles of short default runs (a cursor then lies inside a shower) and on both sides
of the finalize's switches.  (The crossings of each fit the workspace's staging, so every part makes way.)"""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import gpu_run, handles, params
from paper_2006_14927_amd import ckv, synth

pytestmark = pytest.mark.gpu


def by_group(offsets, *arrays):
    return [np.split(a, offsets[1:-1]) for a in arrays]


def workload(kind, n, n_tel):
    if kind == "grazing":
        return synth.grazing_tracks(n)
    wl = synth.single_tev(1000)
    if kind == "showers":
        segs = synth.Segments.concat([synth.shower_segments(s, n // 7 + 31 * s, wl.atmo, zenith_deg=20.0, xmax=400.0,
                                                            shower_id=s) for s in range(7)])
    else:
        segs = synth.shower_segments(3, n, wl.atmo, zenith_deg=20.0, xmax=400.0)
    tels = synth.telescopes_disk(n_tel, disk_radius=100.0 * np.sqrt(n_tel))
    return dataclasses.replace(wl, segs=segs, tels=tels)


@pytest.mark.parametrize("kind,n,n_tel,parts,kw", [
    ("one", 300, 9, 2, {}), ("one", 5000, 31, 6, {}), ("one", 5000, 127, 6, {}), ("one", 20_000, 100, 9, {}),
    ("one", 40_000, 100, 9, {}), ("one", 3000, 512, 5, {}), ("one", 3000, 513, 5, {}),
    ("showers", 6000, 100, 8, {}), ("showers", 30_000, 9, 8, {}), ("showers", 40_000, 100, 8, {}),
    ("showers", 6000, 100, 8, dict(tile_segments=16)), ("showers", 6000, 100, 8, dict(precision=ckv.CKV_FP64)),
    ("grazing", 400, 400, 5, dict(grazing_exact=True)), ("grazing", 9000, 400, 3, dict(grazing_exact=True)),
    ("showers", 6000, 100, 8, dict(grazing_exact=True)), ("showers", 6000, 100, 8, dict(earth_radius=6.371e6)),
])
def test_parts_concatenate_to_the_whole_run(kind, n, n_tel, parts, kw):
    wl = workload(kind, n, n_tel)
    kw = dict(kw)
    precision = kw.pop("precision", ckv.CKV_MIXED)
    whole = gpu_run(wl, precision, **kw)
    n_rec = whole["result"]["n_records"]
    assert whole["result"]["overflow"] == 0 and n_rec > 20 * parts
    atmo, tels = handles(wl)
    r = ckv.Runner(ckv.DeviceSegments(wl.segs), atmo, tels, params(wl, precision, **kw), n_rec // parts + n_rec // 10)
    at, got, runs = (0, 0), None, 0
    while True:
        out = r.run(resume_from=at)
        res = out.result()
        offs = out.tel_offsets.cpu().numpy()
        k = res["n_records"]
        assert res["error"] == 0 and offs[-1] == k
        part = by_group(offs, out.records[:k].cpu().numpy().view(np.uint32), out.ids[:k].cpu().numpy())
        got = part if got is None else [[np.concatenate(x) for x in zip(a, b)] for a, b in zip(got, part)]
        runs += 1
        if not res["overflow"]:
            break
        assert (res["resume_step"], res["resume_shower"]) > at
        at = (res["resume_step"], res["resume_shower"])
    assert runs > 1
    want = by_group(whole["offsets"], whole["rec"].view(np.uint32), whole["ids"])
    for a, b in zip(got, want):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("zenith", [60.0, 80.0, 83.0])
def test_listed_soft_forward_where_cones_straddle_w_min(zenith):
    """The screening pass bounds a step's azimuths with w no lower than w_min, below which
    the FP64 pass drops a bunch: with and without the list S and A are the same sums."""
    dw = synth.diff_showers(4, 3000, zenith_deg=zenith)
    spec = ckv.ParamSpec(dw.eta0, dw.layer_bounds, dw.n_knots, dw.knot_top, dw.obs_level, dw.step, dw.top)
    out = []
    for use_list in (True, False):
        m = ckv.SoftModel(dw.segs, dw.tels, spec, dw.theta0, dw.sigma, seed=dw.seed, use_list=use_list,
                          list_capacity=2_000_000)
        S, A = m.forward(dw.theta0)
        out.append((S.cpu().numpy(), A.cpu().numpy()))
        if use_list:
            count, cap = m.list_state()
            assert 0 < count <= cap
    (S, A), (So, Ao) = out
    assert So.sum() > 10
    # (sums of at most 1e6 weights in another order)
    np.testing.assert_allclose(S, So, rtol=1e-10, atol=1e-12 * So.max())
    np.testing.assert_allclose(A, Ao, rtol=1e-10, atol=1e-12 * np.abs(Ao).max())

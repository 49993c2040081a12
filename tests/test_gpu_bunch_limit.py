"""Default tiles past the 2^30 bunches that a tile's offsets allow.

A tile of the report's size (32 steps) with more bunches is refused whole: error bit 1, its
bunches left out.  Short runs of default tiles work in smaller ones inside; the refusal,
like the report and the cut, stays that of 32 steps, whether one step passes the limit by
itself, or only all of the tile's steps together do, with no smaller tile past it."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_run
from paper_2006_14927_amd import ckv, synth

pytestmark = pytest.mark.gpu


def with_long_steps(segs, at, length, split=0):
    """Steps `at` nearly horizontal, 1 GeV, `length` long (1.8e-9 x 2^30 bunches a metre); two
    showers from step `split`."""
    f = {k: getattr(segs, k).copy() for k in segs.FIELDS}
    w = 5e-6
    for k in at:
        f["length"][k], f["w"][k], f["u"][k], f["v"][k], f["h0"][k] = length, w, np.sqrt(1.0 - w * w), 0.0, 13000.0
        f["energy"][k] = 1000.0
    offsets, t_ref, ids = segs.seg_offsets, segs.t_ref, segs.shower_ids
    if split:
        offsets, t_ref, ids = np.array([0, split, segs.n]), np.repeat(t_ref, 2), np.arange(2, dtype=np.uint32)
    return synth.Segments(*[f[n] for n in segs.FIELDS], segs.ptype, offsets, t_ref, ids)


@pytest.mark.parametrize("n,at,length,refused,split", [
    (3000, (100,), 2e9, (96, 128), 0),                        # 8-step tiles, one step
    (3000, (97, 105, 113, 121, 127), 1.4e8, (96, 128), 0),      # its four tiles together
    (20_000, (1025, 1030, 1041, 1050), 1.6e8, (1024, 1056), 0),  # 16-step tiles, two together
    (3000, (1012, 1019, 1030, 1041), 1.6e8, (1010, 1042), 1010),  # across 1024 steps
], ids=["one_step", "four_tiles", "two_tiles", "second_shower"])
@pytest.mark.parametrize("precision", [ckv.CKV_FP64, ckv.CKV_MIXED])
def test_default_tiles_past_the_bunch_limit_are_refused(precision, n, at, length, refused, split):
    wl = synth.vertical_gamma(n)
    segs = with_long_steps(wl.segs, at, length, split)
    cfg = oracle.Config.from_workload(wl)
    nb = np.asarray(oracle.segment_details(cfg, segs)["n_b"], dtype=np.int64)
    a, b = refused
    assert nb[a:b].sum() >= 1 << 30
    if len(at) > 1:
        small = 8 if n <= 8192 else 16
        assert max(nb[i:i + small].sum() for i in range(a, b, small)) < 1 << 30
    res = gpu_run(wl, precision, segs=segs)["result"]
    assert res["error"] == 2
    assert res["n_bunches"] == int(nb.sum() - nb[a:b].sum())


@pytest.mark.parametrize("grazing", [False, True])
def test_a_resumed_run_refuses_from_its_cursor(grazing):
    """Tiles count from the cursor: resumed at step 110, the 32 steps from there hold all
    of the long ones; from the start they are in two tiles, neither past the limit."""
    wl = synth.vertical_gamma(3000)
    cfg = oracle.Config.from_workload(wl)
    segs = with_long_steps(wl.segs, (111, 120, 130, 141), 1.6e8)
    nb = np.asarray(oracle.segment_details(cfg, segs)["n_b"], dtype=np.int64)
    assert nb[110:142].sum() >= 1 << 30 and max(nb[96:128].sum(), nb[128:160].sum()) < 1 << 30
    atmo = ckv.Atmosphere(wl.atmo.alt, wl.atmo.eta, wl.atmo.obs_level)
    tels = ckv.TelescopeArray(wl.tels.x, wl.tels.y, wl.tels.r)
    r = ckv.Runner(ckv.DeviceSegments(segs), atmo, tels, ckv.make_params(grazing_exact=grazing, seed=wl.seed), 65536)
    res = r.run(resume_from=(110, 0)).result()
    assert res["error"] == 2
    assert res["n_bunches"] == int(nb[142:].sum())

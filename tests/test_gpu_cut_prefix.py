"""How much a cut run writes.  A run whose crossings pass its capacity writes a prefix of its
steps: the longest that fits, unless the staging area (the capacity and two blocks of 256 for
each of 4096 waves) fills while an earlier tile is still worked on.  The waves' first tiles
are worked on at once; over an array with up to 16 crossings a step the area holds them all,
so what fits of them is written, whatever comes after."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_helpers import handles, params
from paper_2006_14927_amd import ckv, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [ckv.CKV_FP64, ckv.CKV_MIXED])
@pytest.mark.parametrize("capacity", [30_000, 300_000, 1_500_000])
def test_cut_runs_over_a_dense_array_write_a_full_prefix(precision, capacity):
    wl = synth.single_tev(1000)
    segs = synth.shower_segments(3, 400_000, wl.atmo, zenith_deg=20.0, xmax=400.0)
    tels = synth.telescopes_disk(400, disk_radius=250.0, r_min=4.0, r_max=6.0)
    wl = dataclasses.replace(wl, segs=segs, tels=tels)
    atmo, t = handles(wl)
    d = ckv.DeviceSegments(segs)
    whole = ckv.Runner(d, atmo, t, params(wl, precision), 4_500_000)
    out = whole.run()
    n = out.result()["n_records"]
    assert 3_000_000 < n < 4_500_000
    per_tile = np.bincount(out.ids[:n, 0].cpu().numpy() // 32, minlength=-(-segs.n // 32))
    cum = np.cumsum(per_tile)
    fits = int(cum[cum <= capacity][-1])
    first = torch.cuda.get_device_properties(0).multi_processor_count * 16     # waves
    assert cum[first - 1] + 128 * first < capacity + 2 * 256 * first           # (half a block of each is empty)
    res = ckv.Runner(d, atmo, t, params(wl, precision), capacity).run().result()
    assert res["overflow"] == 1 and res["n_hits"] == n
    assert res["n_records"] in cum
    assert min(fits, cum[first - 1]) <= res["n_records"] <= fits

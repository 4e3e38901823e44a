"""The patch-size tuner (pic_autotune_patch): it times temporary simulations
at each candidate patch edge and workgroup size, writes the fastest into the
descriptor, reuses a cached choice, and the tuned descriptor runs the same
physics as the oracle with that patch."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1511_03878_amd import workloads as W
from paper_1511_03878_amd.sim import autotune_patch
from tests.helpers import compare_fields, gpu_sim, oracle_run

pytestmark = pytest.mark.gpu


def test_patch_tuner(tmp_path):
    print("[gpu-test] pic_autotune_patch on the small laser box", flush=True)
    wl = W.lwfa_2d_small()
    cache = str(tmp_path / "tune.txt")
    grid, tune, r = autotune_patch(wl, 32, candidates=(8, 16, 32, 24), warm=5, steps=5, cache=cache)
    assert grid["patch"][0] == grid["patch"][1] in (8, 16, 32)
    assert tune["block"] in (256, 512, 1024)
    assert r["from_cache"] == 0 and r["trials"] >= 3 and r["ms_per_step"] > 0
    assert r["patch"][:2] == grid["patch"]
    grid2, tune2, r2 = autotune_patch(wl, 32, candidates=(8, 16, 32, 24), warm=5, steps=5, cache=cache)
    assert r2["from_cache"] == 1 and grid2 == grid and tune2 == tune
    tuned = dict(wl, grid=grid)
    g = gpu_sim(tuned, 64, **tune)
    g.step(20)
    o = oracle_run(tuned, 20)
    e, b = compare_fields(g, o)
    assert e < 1e-11 and b < 1e-11, (e, b)
    assert np.array_equal(g.counts(), o.counts())


def test_choices_stored_by_an_earlier_version_are_not_taken(tmp_path):
    # a line as stored when field_tile 0 was a tile shape and 2-D Yee had no strips
    print("[gpu-test] both tuners with a cache file of an earlier version", flush=True)
    from tests import fixtures as F
    wl = F.uniform_2d(n=(64, 64), patch=(16, 16), ppc=8)
    cache = tmp_path / "tune.txt"
    cache.write_text("pic-tune nd=2 prec=32 n=64,64,1 patch=16,16,1 np2=15 1024 3 8 256\n"
                     "pic-patch nd=2 prec=32 n=64,64,1 profile=0 load=0 ppc=8 32 32 1 1024\n")
    g = gpu_sim(wl, 32)
    r = g.autotune(steps=2, cache=str(cache))
    assert r["from_cache"] == 0 and r["trials"] > 0
    box = W.uniform_2d(n=(64, 64), patch=(16, 16), ppc=8)
    r = autotune_patch(box, 32, candidates=(16, 32), warm=2, steps=2, cache=str(cache))[2]
    assert r["from_cache"] == 0 and r["trials"] > 0
    # the choices stored now are
    assert gpu_sim(wl, 32).autotune(steps=2, cache=str(cache))["from_cache"] == 1
    assert autotune_patch(box, 32, candidates=(16, 32), warm=2, steps=2, cache=str(cache))[2]["from_cache"] == 1


def test_tuner_tries_every_lane_stride_of_3d():
    # the settings as they are, three workgroup sizes, strides 2, 4 and 8, four chunks
    print("[gpu-test] tuner candidates of a 3-D box", flush=True)
    from tests import fixtures as F
    g = gpu_sim(F.blob_3d(n=(16, 16, 16), patch=(8, 8, 8), ppc0=2), 32)
    r = g.autotune(steps=2)
    assert r["trials"] >= 1 + 3 + 3 + 4 and r["lane_stride"] in (1, 2, 4, 8)

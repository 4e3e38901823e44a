"""Choices of the step and of the read-back that depend on sizes, at the sizes
where they change: shared launches against separate ones, work items of other
sizes, the depth of 3-D field-update blocks, the lanes of the re-binning check,
and read-backs that end inside a slot or a patch."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests import fixtures as W
from tests.brute import rho_2d, rho_3d
from tests.helpers import compare_fields, gpu_sim, neighbour_patch, neighbour_patch3

pytestmark = pytest.mark.gpu

FIELDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx", "Jy", "Jz")
S6 = 75.0 / 64.0 + 25.0 / 384.0 + 3.0 / 640.0


def _announce(msg):
    print(f"[gpu-test] {msg}", flush=True)


def _box(case):
    if case == "2d_open":
        return W.lwfa_2d_small(n=(256, 64), patch=(16, 16), nsteps=12), {}
    if case == "2d_sixth":
        return W.uniform_2d(n=(72, 40), patch=(12, 8), ppc=6, T_keV=20.0, cfl=0.9 / S6), {"maxwell_order": 6}
    if case == "3d":
        return W.blob_3d(n=(24, 16, 20), patch=(8, 8, 4), T_keV=20.0, ppc0=3), {}
    return W.blob_3d(n=(16, 12, 20), patch=(4, 4, 4), T_keV=20.0, ppc0=3, cfl=0.9 / S6), {"maxwell_order": 6}


@pytest.mark.parametrize("case", ["2d_open", "2d_sixth", "3d", "3d_sixth"])
def test_shared_launches_give_the_bits_of_separate_ones(case):
    # timing every kernel group takes the separate launches on two streams
    _announce(f"field update and re-binning in shared launches: {case}")
    wl, kw = _box(case)
    runs = []
    for timed in (False, True):
        g = gpu_sim(wl, 32, deterministic=1, **kw)
        g.timing_enable(timed)
        g.step(12)
        runs.append([g.field(c) for c in FIELDS] + [g.history(0, 12)[0], g.counts(), *g.particles()[0], g.perm()])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("case", ["2d_sixth", "3d"])
@pytest.mark.parametrize("chunk", [64, 1000])
def test_item_size_does_not_change_the_state(case, chunk):
    # (64: more items than workgroups, so most are claimed from the counter)
    _announce(f"items of {chunk} particles against the default: {case}")
    wl = (W.uniform_2d(n=(192, 160), patch=(32, 32), ppc=16, T_keV=20.0, cfl=0.9 / S6) if case == "2d_sixth"
          else W.blob_3d(n=(32, 24, 16), patch=(8, 8, 8), T_keV=20.0, ppc0=6))
    kw = {"maxwell_order": 6} if case == "2d_sixth" else {}
    runs = []
    for c in (0, chunk):
        g = gpu_sim(wl, 32, deterministic=1, chunk=c, **kw)
        g.step(8)
        runs.append([g.field(f) for f in FIELDS] + [g.counts(), *g.particles()[0], g.perm()])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("case", ["2d_fp64", "3d_fp64", "3d_fp32"])
def test_workgroup_size_does_not_change_the_state(case):
    # enough items that 256 threads are chosen, against 512
    _announce(f"particle workgroups chosen against 512 threads: {case}")
    wl = (W.uniform_2d(n=(256, 128), patch=(8, 8), ppc=4, T_keV=20.0) if case == "2d_fp64"
          else W.blob_3d(n=(64, 32, 64) if case == "3d_fp32" else (32, 32, 32), patch=(4, 4, 4), T_keV=20.0,
                         ppc0=2))
    runs = []
    for block in (0, 512):
        g = gpu_sim(wl, 32 if case == "3d_fp32" else 64, deterministic=1, block=block)
        g.step(6)
        runs.append([g.field(f) for f in FIELDS] + [g.counts(), *g.particles()[0], g.perm()])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [32, 64])
def test_patch_shapes_mixed_in_a_3d_batch(precision):
    # one kernel for all shapes of the batch; tiles of different sizes follow
    # each other in a workgroup (small items: several per workgroup)
    _announce(f"3-D batch of 8x8x8 and 4x4x8 patches fp{precision}")
    from paper_1511_03878_amd.sim import Batch
    wls = [W.blob_3d(n=(24, 16, 16), patch=(8, 8, 8), T_keV=20.0, ppc0=3),
           W.blob_3d(n=(16, 24, 16), patch=(4, 4, 8), T_keV=20.0, ppc0=3, seed=6)]
    runs = []
    for together in (False, True):
        sims = [gpu_sim(wl, precision, deterministic=1, chunk=64) for wl in wls]
        if together:
            b = Batch(precision, ndim=3)
            for g in sims:
                b.add(g, 6)
            b.step(6)
        else:
            for g in sims:
                g.step(6)
        runs.append([v for g in sims for v in [*(g.field(f) for f in FIELDS), g.counts(), *g.particles()[0]]])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [(40, 12, 18), (256, 128, 36)])
def test_shallow_field_blocks_match_oracle(n):
    # 4 and 8 planes per block; the last block of the z axis is partial
    _announce(f"3-D vacuum fields {n} fp64")
    d = (0.1, 0.13, 0.11)
    grid = dict(ndim=3, n=list(n), d=list(d), dt=W.cfl_dt(d), patch=[4, 4, 2 if n[2] % 4 else 4],
                periodic=[1, 1, 1], q=-1.0, m=1.0)
    from paper_1511_03878_amd.sim import Sim
    g = Sim(grid, 64)
    g.set_particles([np.zeros(0)] * 3, [np.zeros(0)] * 3, np.zeros(0))
    o = oracle.Sim(grid)
    rng = np.random.default_rng(5)
    for c in FIELDS[:6]:
        f = rng.standard_normal(n[::-1])
        g.set_field(c, f)
        o.set_field(c, f)
    steps = 8 if n[0] < 100 else 2
    g.step(steps)
    o.step(steps)
    e, b = compare_fields(g, o)
    assert e < 1e-12 and b < 1e-12, (e, b)
    U, Uo = g.history(steps - 1, 1)[0][0], o.energy()[0]
    assert abs(U - Uo) <= 1e-12 * abs(Uo)


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("periodic", [1, 0])
@pytest.mark.parametrize("n", [(64, 8), (60, 12), (184, 42), (8, 5000), (976, 602)])
def test_field_strips_give_the_bits_of_tiles(n, periodic, precision):
    # strips of 61 columns and 4 or 8 rows (partial ones, a grid narrower than a
    # strip, the x = L ghost in the first and last lanes) against 2-D tiles
    _announce(f"2-D vacuum fields {n} periodic {periodic} fp{precision}: strips against tiles")
    from paper_1511_03878_amd.sim import Sim
    d = (0.1, 0.13)
    grid = dict(ndim=2, n=list(n), d=list(d), dt=W.cfl_dt(d), patch=[4, 2], periodic=[periodic, 1], q=-1.0, m=1.0)
    runs = []
    for tile in (0, 1):
        g = Sim(grid, precision, field_tile=tile)
        g.set_particles([np.zeros(0)] * 2, [np.zeros(0)] * 3, np.zeros(0))
        rng = np.random.default_rng(11)
        for c in FIELDS[:6]:
            g.set_field(c, rng.standard_normal(g.field(c).shape))
        if not periodic:
            t = np.arange(6)[:, None] + 0.1 * np.arange(n[1])[None]
            g.set_laser(ey=np.sin(t), ez=np.cos(t))
            g.add_laser(dict(a0=1.0, omega0=1.0, w0=5.0, tau=4.0, t0=1.0, x_focus=3.0, y_center=2.0, phase=0.2))
        g.step(6)
        runs.append(([g.field(c) for c in FIELDS[:6]], g.history(0, 6)[0]))
    for a, b in zip(runs[0][0], runs[1][0]):
        assert np.array_equal(a, b)
    # the energies add the same squares in another order
    assert np.abs(runs[0][1] - runs[1][1]).max() <= 1e-12 * np.abs(runs[1][1]).max()


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("share", [0.0, 0.0005, 0.2])
def test_particles_at_rest_without_fields(share, precision):
    # weightless particles make no field: at rest they are passed over, but a
    # share of them moves (units with and without a moving particle, slots
    # that hold the code of a particle which left)
    _announce(f"particles at rest without fields, {share} of them moving, fp{precision}")
    wl = W.uniform_2d(n=(64, 48), patch=(16, 16), ppc=12, T_keV=200.0, seed=4)
    if precision == 32:
        wl = W.to_float32_state(wl)
    go = np.random.default_rng(8).random(wl["w"].size) < share
    wl["w"] = np.zeros_like(wl["w"])
    wl["u"] = [np.where(go, v, 0.0) for v in wl["u"]]
    from paper_1511_03878_amd.sim import Sim
    g = Sim(wl["grid"], precision, chunk=300)
    g.set_particles(wl["x"], wl["u"], wl["w"])
    o = oracle.Sim(wl["grid"])
    o.set_particles(wl["x"], wl["u"], wl["w"])
    for steps in (1, 1, 12):
        g.step(steps)
        o.step(steps)
        if precision == 64:
            assert np.array_equal(g.counts(), o.counts()) and np.array_equal(g.perm(), o.particles()[3])
            for a, b in zip(g.particles()[0], o.particles()[0]):
                assert np.abs(np.asarray(a) - np.asarray(b)).max() < 1e-11
    gx, gu, _, ids = g.particles()
    back = np.argsort(ids)
    for a in range(3):
        assert np.array_equal(gu[a][back], np.asarray(wl["u"][a]))  # no field changes a momentum
    for a in range(2):
        assert np.array_equal(gx[a][back][~go], np.asarray(wl["x"][a])[~go])
    assert not any(np.any(g.field(c)) for c in FIELDS)


@pytest.mark.parametrize("nd", [2, 3])
@pytest.mark.parametrize("moving", [0.001, 0.35, 1.0])
def test_rebin_check_searches_any_number_of_vacated_slots(nd, moving):
    # a few, thousands and all of a patch's particles leave
    _announce(f"re-binning check: {nd}-D, {moving} of the particles leave")
    wl = (W.uniform_2d(n=(128, 128), patch=(64, 64), ppc=2) if nd == 2
          else W.blob_3d(n=(16, 16, 16), patch=(8, 8, 8), ppc0=8))
    from paper_1511_03878_amd.sim import Sim
    g = Sim(wl["grid"], 64)
    g.set_particles(wl["x"], wl["u"], wl["w"])
    counts, ids = g.counts(), g.perm()
    rng = np.random.default_rng(9)
    ndir = 9 if nd == 2 else 27
    go = rng.random(ids.size) < moving
    codes = np.full(ids.size, ndir // 2, dtype=np.uint8)
    codes[go] = rng.integers(0, ndir, int(go.sum()))
    codes[rng.random(ids.size) > 0.99] = 255
    np_ = [wl["grid"]["n"][a] // wl["grid"]["patch"][a] for a in range(nd)]
    owner = np.repeat(np.arange(counts.size), counts)
    to = (lambda p, c: neighbour_patch(p, c, np_, (1, 1))) if nd == 2 else (lambda p, c: neighbour_patch3(p, c, np_))
    dest = np.array([-1 if c == 255 else to(p, int(c)) for p, c in zip(owner, codes)], dtype=np.int32)
    newcount, src = oracle.rebin(counts, dest)
    g.rebin_codes(codes)
    assert np.array_equal(g.counts(), newcount)
    assert np.array_equal(g.perm(), ids[src])


@pytest.mark.parametrize("ppc,moving", [(255, 0.005), (260, 0.005), (20, 0.05)])
def test_rebin_of_patches_of_many_batches(ppc, moving):
    # waves whose 65536 slots still fit a listed slot number, one more row, and
    # lists of leavers near the room kept for them (256 per wave before the last batch)
    _announce(f"re-binning of patches of {ppc * 1024} particles, {moving} of them leave")
    wl = W.uniform_2d(n=(96, 32), patch=(32, 32), ppc=ppc)
    from paper_1511_03878_amd.sim import Sim
    g = Sim(wl["grid"], 32)
    g.set_particles(wl["x"], wl["u"], wl["w"])
    counts, ids = g.counts(), g.perm()
    rng = np.random.default_rng(4)
    codes = np.full(ids.size, 4, dtype=np.uint8)
    go = rng.random(ids.size) < moving
    codes[go] = rng.integers(0, 9, int(go.sum()))
    owner = np.repeat(np.arange(counts.size), counts)
    table = np.array([[neighbour_patch(p, c, [3, 1], (1, 1)) for c in range(9)] for p in range(3)])
    newcount, src = oracle.rebin(counts, table[owner, codes].astype(np.int32))
    g.rebin_codes(codes)
    assert np.array_equal(g.counts(), newcount)
    assert np.array_equal(g.perm(), ids[src])


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("n,patch", [((52, 20), (4, 20)), ((1000, 524), (50, 4)), ((1000, 525), (50, 25))])
def test_fields_read_back_whole(n, patch, precision):
    # below and above the size from which a grid is read in parts (2^19 nodes)
    _announce(f"field read-back {n} fp{precision}")
    from paper_1511_03878_amd.sim import Sim
    d = (0.1, 0.1)
    g = Sim(dict(ndim=2, n=list(n), d=list(d), dt=W.cfl_dt(d), patch=list(patch), periodic=[1, 1]), precision)
    rng = np.random.default_rng(3)
    for c in ("Ex", "Bz"):
        f = rng.standard_normal(n[::-1]).astype(np.float32).astype(np.float64)
        g.set_field(c, f)
        assert np.array_equal(g.field(c), f)


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("nd,count", [(2, 0), (2, 1), (2, 65536), (2, 65537), (3, 3000), (3, 131075)])
def test_particles_read_back_whole(nd, count, precision):
    # runs of 2^16 particles: none, one, one exactly, and rests of 1 and 3
    _announce(f"particle read-back {nd}-D {count} fp{precision}")
    from paper_1511_03878_amd.sim import Sim
    n, patch = ([48, 40], [8, 20]) if nd == 2 else ([16, 8, 24], [8, 4, 6])
    d = [0.1] * nd
    g = Sim(dict(ndim=nd, n=n, d=d, dt=W.cfl_dt(d), patch=patch, periodic=[1] * nd), precision)
    rng = np.random.default_rng(count + nd)
    # multiples of 2^-12: exact in FP32 as offsets in a patch and in the grid
    x = [np.floor(rng.random(count) * n[a] * 4096) / 4096 for a in range(nd)]
    x[0] = np.where(rng.random(count) < 0.3, x[0] % patch[0], x[0])  # uneven patches, some may be empty
    u = [rng.standard_normal(count).astype(np.float32).astype(np.float64) for _ in range(3)]
    w = rng.random(count).astype(np.float32).astype(np.float64)
    g.set_particles(x, u, w)
    gx, gu, gw, ids = g.particles()
    assert np.array_equal(np.sort(ids), np.arange(count)) and np.array_equal(ids, g.perm())
    pid = sum(np.floor(x[a]).astype(int) // patch[a] * int(np.prod([n[b] // patch[b] for b in range(a)]))
              for a in range(nd))
    assert np.array_equal(ids, np.argsort(pid, kind="stable"))
    for got, ref in zip([*gx, *gu, gw], [*x, *u, w]):
        assert np.array_equal(got, ref[ids])


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("n,patch", [((64, 64), (64, 64)), ((60, 35), (20, 7)), ((12, 10, 14), (6, 5, 7)),
                                     ((8, 8, 4), (4, 8, 1))])
def test_charge_density_of_any_patch_shape(n, patch, precision):
    _announce(f"rho {n} patches {patch} fp{precision}")
    wl = (W.uniform_2d(n=n, patch=patch, ppc=5, T_keV=20.0) if len(n) == 2
          else W.blob_3d(n=n, patch=patch, ppc0=3, T_keV=20.0, blob_radius=3.0))
    g = gpu_sim(wl, precision)
    if patch != (64, 64):  # (the particle kernel's tiles of such a patch do not fit into LDS)
        g.step(2)
    x, _, w, _ = g.particles()
    ref = rho_2d(x[0], x[1], w, -1.0, n) if len(n) == 2 else rho_3d(x, w, -1.0, n)
    got = g.field("rho")
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("start", [0, 9])
def test_merges_and_jumps_are_launched_when_due(start):
    # merges every 7 steps and a jump every 16: a run that stops for larger
    # patches on the way and graph replays (whose launches serve any step)
    # give the bits of single steps
    _announce(f"window from step {start} and merges: long runs against single steps")
    from tests.test_gpu_window import _gapped, _thermal_open
    runs = []
    for calls, kw in (((1,) * 80, {}), ((1, 20, 59), dict(capacity_factor=1.0, min_capacity=16)), ((80,), dict(graph=1))):
        g = gpu_sim(_thermal_open(T_keV=5.0, ppc=9), 64, deterministic=1, **kw)
        g.set_window(start, 1.0, (3, 3), _gapped())
        g.set_merge(7, 8, 4)
        for n in calls:
            g.step(n)
        d = g.diag()
        assert d["window_cells"] >= 32 and d["merged"] > 0 and (d["relayouts"] > 0) == ("min_capacity" in kw)
        runs.append([d["merged"], d["window_cells"], *(g.field(c) for c in FIELDS), g.counts(), *g.particles()[0],
                     *g.particles()[1], g.perm()])
    for r in runs[1:]:
        for a, b in zip(runs[0], r):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("case", ["2d_open", "2d_sixth", "3d", "3d_sixth"])
def test_alone_and_beside_a_large_box_give_the_same_bits(case, precision):
    # alone the field update shares launches with the re-binning, beside a grid
    # of more than 3 * 2^18 nodes it has kernels of its own on a second stream
    _announce(f"shared launches alone against separate ones in a large batch: {case} fp{precision}")
    from paper_1511_03878_amd.sim import Batch, Sim
    wl, kw = _box(case)
    nd = wl["grid"]["ndim"]
    n, patch = ([1024, 1024], [64, 8]) if nd == 2 else ([128, 96, 80], [8, 8, 8])
    runs = []
    for together in (False, True):
        g = gpu_sim(wl, precision, deterministic=1, **kw)
        if together:
            d = [0.1] * nd
            big = Sim(dict(ndim=nd, n=n, d=d, dt=0.5 * W.cfl_dt(d), patch=patch, periodic=[1] * nd), precision, **kw)
            x = [np.full(3, 0.5 * v) for v in n]
            big.set_particles(x, [np.zeros(3)] * 3, np.full(3, 0.1))
            b = Batch(precision, ndim=nd)
            b.add(g, 12)
            b.add(big, 12)
            b.step(12)
            b.close()
        else:
            g.step(12)
        runs.append([g.field(c) for c in FIELDS] + [g.history(0, 12)[0], g.counts(), *g.particles()[0],
                                                    *g.particles()[1], g.perm()])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


def test_large_reads_of_work_queued_on_a_per_thread_stream():
    # a handle on hipStreamPerThread (2): the threads that read a large array have
    # streams of their own there, and the density they read is queued on the
    # caller's (one crowded patch keeps its kernel running for milliseconds)
    _announce("large reads with the per-thread default stream, 1024x1024 fp32 and fp64")
    from paper_1511_03878_amd.sim import Sim
    n, d, count = (1024, 1024), (0.1, 0.1), 2000000
    # dyadic positions and weights: every sum is exact; in the last thread's part
    x, w = [np.full(count, 8.25), np.full(count, 1000.25)], np.full(count, 2.0 ** -10)
    ref = rho_2d([8.25], [1000.25], [count * 2.0 ** -10], -1.0, n)
    rng = np.random.default_rng(6)
    for precision in (32, 64):
        g = Sim(dict(ndim=2, n=list(n), d=list(d), dt=W.cfl_dt(d), patch=[16, 16], periodic=[1, 1], q=-1.0, m=1.0),
                precision, stream=2, torch_alloc=False)
        g.set_particles(x, [np.zeros(count)] * 3, w)
        for _ in range(3):
            assert np.array_equal(g.field("rho"), ref)
        f = rng.standard_normal(n).astype(np.float32).astype(np.float64)
        g.set_field("Ey", f)
        assert np.array_equal(g.field("Ey"), f)

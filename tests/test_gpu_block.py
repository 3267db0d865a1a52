"""Several steps per launch on LDS blocks (k_block) against single steps:
with kernel timing on, every step is a pass of its own; without, runs go
through k_block where the domain has a plan for it.  Fields, masses, wall
force, counters and the first unstable step are the same bit for bit, at
lattices narrower than a block's region, at multiples of a tile and one node
either side, for every rule, fix, EOS and storage form, and the total mass has
the same bits for every tile shape."""
import sys

import numpy as np
import pytest

from lbm_inputs import configs as cfg

from tests._random_cases import random_case

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    from paper_1908_09235_amd import lbm
    lbm.lib()
    return lbm


RUNS = (1, 2, 3, 7, 26, 1, 8)


def _same(L, p, storage, runs=RUNS, **kw):
    with L.Domain(p, storage=storage, history_capacity=256, **kw) as a, \
            L.Domain(p, storage=storage, history_capacity=256, **kw) as b:
        L.lbm_set_profiling(a.h, 1)  # single steps
        for n in runs:
            for d in (a, b):
                try:
                    d.step(n)
                except L.LbmError as e:
                    assert e.code == L.LBM_EUNSTABLE
            tag = (p.name, storage, a.t)
            assert a.t == b.t
            for x, y in zip(a.moments(), b.moments()):
                assert np.array_equal(x, y, equal_nan=True), tag
            assert np.array_equal(a.mass_history(), b.mass_history(), equal_nan=True), tag
            assert np.array_equal(a.wall_force(), b.wall_force(), equal_nan=True), tag
        assert a.negative_rest() == b.negative_rest()
        assert a.degenerate_b() == b.degenerate_b()
        assert L.lbm_unstable_step(a.h) == L.lbm_unstable_step(b.h)


STORAGES = ["f64", "f32", "f32_arith32", "f32dev", "f16dev"]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("case", [
    ("mls", "A"), ("mls", "B"), ("mls", "bao"), ("fh", "B"), ("halfway", "none"),
    ("ibb_linear", "A"), ("ibb_quadratic", "A"), ("zhao_yong", "none")])
def test_every_rule(L, case, storage):
    p = cfg.droplet_on_cylinder(rule=case[0], fix=case[1], tau=0.8, collision="mrt",
                                rho_wall=0.05, name="_".join(case))
    say(f"[gpu] blocks vs single steps {case} {storage}")
    _same(L, p, storage)


@pytest.mark.parametrize("storage", ["f64", "f16dev"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 40), (31, 33), (32, 32), (48, 24), (96, 95),
                                   (97, 96), (289, 97)])
def test_sizes_around_a_tile(L, nx, ny, storage):
    say(f"[gpu] blocks vs single steps {nx}x{ny} {storage}")
    p = cfg.free_droplet(max(nx, ny), 0.25 * min(nx, ny), eos="exp")
    rho0 = np.ascontiguousarray(p.rho0[:ny, :nx])
    _same(L, p.with_(nx=nx, ny=ny, solid=np.zeros((ny, nx), np.uint8), rho0=rho0,
                     rho_wall=np.ones((ny, nx))), storage)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("nx,ny", [(3, 5), (8, 8), (9, 7), (23, 24), (24, 25), (100, 50),
                                   (128, 121), (129, 129)])
def test_small_single_phase_sizes(L, nx, ny, storage):
    say(f"[gpu] blocks vs single steps, single phase {nx}x{ny} {storage}")
    y, x = np.mgrid[:ny, :nx]
    p = cfg.couette(10, rule="halfway", fix="none")
    rho0 = 1.0 + 0.01 * np.cos(0.7 * x + 0.3) * np.sin(1.1 * y)
    _same(L, p.with_(nx=nx, ny=ny, solid=np.zeros((ny, nx), np.uint8), links=p.links[:0],
                     rho0=rho0, rho_wall=np.ones((ny, nx)), gravity=(1e-5, 2e-5)), storage)


@pytest.mark.parametrize("make", [
    lambda: cfg.couette(10, rule="mls", fix="A"),              # moving walls
    lambda: cfg.cylinder_flow(20.0, fix="B", d=8.0),           # open x
    lambda: cfg.sloped_channel(16, fix="B", g0=1e-3),          # walls through every tile
    lambda: cfg.static_gravity(0.3, rule="mls", fix="A", nx=40, ny=30),
    lambda: cfg.cfg2a(scale=5.0)])                             # more tiles than CUs
@pytest.mark.parametrize("storage", ["f64", "f32dev"])
def test_flows(L, make, storage):
    p = make()
    say(f"[gpu] blocks vs single steps {p.name} {storage}")
    _same(L, p, storage)


@pytest.mark.parametrize("k", range(12))
def test_random_cases(L, k):
    p = random_case(k)[0]
    say(f"[gpu] blocks vs single steps random {k} {p.nx}x{p.ny} {p.rule}/{p.fix}")
    _same(L, p, STORAGES[k % 5])


@pytest.mark.parametrize("storage", ["f64", "f32", "f32dev", "f16node"])
def test_mass_does_not_depend_on_the_tiles(L, storage):
    p = cfg.cfg1("mls", "B")
    got = []
    for tw, th in ((64, 3), (128, 16), (256, 7), (256, 4000)):
        with L.Domain(p, storage=storage, tile_w=tw, tile_h=th, history_capacity=64) as d:
            L.lbm_set_profiling(d.h, 1)
            d.step(20)
            got.append(d.mass_history())
    say(f"[gpu] masses for four tile shapes, {storage}: {got[0][-1]!r}")
    assert all(np.array_equal(got[0], g) for g in got[1:])


def _mixed(eos):
    """Instances of a batch, some of which break down within the run: with the
    mean density at the walls and a tau near a half the droplets do."""
    if eos == "none":
        return [cfg.couette(10, rule="mls", fix="A"), cfg.sloped_channel(16, fix="B", g0=1e-3),
                cfg.sloped_channel(44, rule="ibb_quadratic", fix="A", g0=1e-3)]
    ps = []
    for k, tau in enumerate((0.505, 0.52, 0.55, 0.9, 0.505, 0.55)):
        p = cfg.batch_instance(k, seed=11, side_lo=40, side_hi=90)
        mean = 0.5 * (p.rho0.max() + p.rho0.min())
        ps.append(p.with_(tau=tau, collision="bgk", rho_wall=np.full_like(p.rho_wall, mean)))
    return ps


@pytest.mark.parametrize("runs", [RUNS + (46,), (94,)], ids=["short", "long"])
@pytest.mark.parametrize("storage,eos", [(s, "cs") for s in STORAGES] + [("f64", "none")])
def test_batch(L, storage, eos, runs):
    ps = _mixed(eos)
    total = [90, 33, 94, 12, 61, 94][:len(ps)]
    say(f"[gpu] batch in blocks vs single steps {storage} {eos} {[p.nx for p in ps]}")
    with L.Batch(storage=storage, eos=eos, max_instances=8, arena_bytes=1 << 28) as b:
        slots = [b.add(p, n, history_capacity=128) for p, n in zip(ps, total)]
        doms = [L.Domain(p, storage=storage, history_capacity=128) for p in ps]
        try:
            for d in doms:
                L.lbm_set_profiling(d.h, 1)  # single steps
            for n in runs:
                b.run(n)
                for k, d in enumerate(doms):
                    t, rem, u = b.status(slots[k])
                    if L.lbm_unstable_step(d.h) < 0:
                        try:
                            d.step(min(n, total[k] - d.t))
                        except L.LbmError as e:
                            assert e.code == L.LBM_EUNSTABLE
                    alone = L.lbm_unstable_step(d.h)
                    assert u == alone, (k, u, alone)
                    assert t == (u if u >= 0 else d.t) and rem == (0 if u >= 0 else total[k] - t)
                    if u < 0:
                        for x, y in zip(b.moments(slots[k]), d.moments()):
                            assert np.array_equal(x, y, equal_nan=True), (k, t)
                    h = b.mass_history(slots[k])
                    assert np.array_equal(h, d.mass_history()[:len(h)], equal_nan=True), (k, t)
            ends = [b.status(s)[2] for s in slots]
            say(f"    unstable at {ends}")
            assert eos == "none" or (max(ends) > 0 and min(ends) < 0)
        finally:
            for d in doms:
                d.close()


@pytest.mark.parametrize("storage", ["f32_arith32", "f32dev"])
def test_two_steps_per_pass_without_walls(L, storage):
    """Asked for two steps per pass, lattices without walls go through blocks
    up to three million nodes and through the two-step kernel beyond."""
    for nx, ny in ((1733, 1731), (1733, 1733)):
        x = np.arange(nx)[None, :] * (2.0 * np.pi / nx)
        y = np.arange(ny)[:, None] * (2.0 * np.pi / ny)
        p = cfg.free_droplet(64, 16.0, eos="exp")
        p = p.with_(nx=nx, ny=ny, solid=np.zeros((ny, nx), np.uint8), rho_wall=np.ones((ny, nx)),
                    rho0=200.0 + np.sin(3 * x) * np.cos(2 * y))
        say(f"[gpu] two steps per pass without walls {nx}x{ny} {storage}")
        with L.Domain(p, storage=storage, history_capacity=64) as a, \
                L.Domain(p, storage=storage, history_capacity=64) as b:
            L.lbm_set_profiling(a.h, 1)
            L.lbm_set_steps_per_pass(b.h, 2)
            for n in (5, 2, 8):
                a.step(n)
                b.step(n)
                for u, v in zip(a.moments(), b.moments()):
                    assert np.array_equal(u, v)
                assert np.array_equal(a.mass_history(), b.mass_history())

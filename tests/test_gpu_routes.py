"""Which launches a run goes through (lbm_get_blocks, lbm_batch_get_blocks): the
cases of test_gpu_block.py that are meant to compare blocks of several steps
with single steps have a plan for them, each number of lanes is used, and what
is meant to fall back to single steps does, with the same fields."""
import sys

import numpy as np
import pytest

from lbm_inputs import configs as cfg
from lbm_inputs.problem import LINK_DTYPE

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


STORAGES = ["f64", "f32", "f32_arith32", "f32dev", "f16dev"]


def _drop(rule, fix):
    return cfg.droplet_on_cylinder(rule=rule, fix=fix, tau=0.8, collision="mrt", rho_wall=0.05)


def _free(nx, ny, eos="exp"):
    p = cfg.free_droplet(64, 16.0, eos="exp")
    return p.with_(nx=nx, ny=ny, solid=np.zeros((ny, nx), np.uint8), eos=eos,
                   rho_wall=np.ones((ny, nx)), rho0=np.full((ny, nx), p.rho0[0, 0]))


def _plan(L, p, storage):
    with L.Domain(p, storage=storage, history_capacity=16) as d:
        return d.blocks()


def _pillars(nx, ny, period):
    """Single solid nodes, one per square of `period`: eight links each."""
    solid = np.zeros((ny, nx), np.uint8)
    solid[::period, ::period] = 1
    return _halfway(solid)


def _halfway(solid):
    ny, nx = solid.shape
    rows = []
    for a, (cx, cy) in enumerate(zip((1, 0, -1, 0, 1, -1, -1, 1), (0, 1, 0, -1, 1, 1, -1, -1)), 1):
        y, x = np.nonzero((solid == 0) & (np.roll(solid, (-cy, -cx), (0, 1)) != 0))
        r = np.zeros(len(x), LINK_DTYPE)
        r["x"], r["y"], r["dir"], r["q"] = x, y, a, 0.5
        rows.append(r)
    y, x = np.mgrid[:ny, :nx]
    rho0 = 1.0 + 0.01 * np.cos(2.0 * np.pi * x / nx) * np.sin(4.0 * np.pi * y / ny)
    return cfg.couette(10, rule="halfway", fix="none").with_(
        nx=nx, ny=ny, solid=solid, links=np.concatenate(rows), rho0=rho0,
        rho_wall=np.ones((ny, nx)), gravity=(1e-5, 2e-5))


@pytest.mark.parametrize("storage", STORAGES)
def test_blocks_where_they_are_compared(L, storage):
    say(f"[gpu] plans of the compared cases, {storage}")
    for rule, fix in (("mls", "A"), ("mls", "B"), ("mls", "bao"), ("fh", "B"),
                      ("halfway", "none"), ("ibb_linear", "A"), ("ibb_quadratic", "A")):
        assert _plan(L, _drop(rule, fix), storage)[0] >= 2, (rule, fix)
    for nx, ny in ((3, 3), (5, 40), (31, 33), (32, 32), (48, 24), (96, 95), (97, 96), (289, 97)):
        assert _plan(L, _free(nx, ny), storage)[0] >= 2, (nx, ny)
    for nx, ny in ((3, 5), (8, 8), (23, 24), (24, 25), (100, 50), (128, 121), (129, 129)):
        assert _plan(L, _free(nx, ny, "none"), storage)[0] >= 2, (nx, ny)
    for p in (cfg.couette(10, rule="mls", fix="A"), cfg.cylinder_flow(20.0, fix="B", d=8.0),
              cfg.sloped_channel(16, fix="B", g0=1e-3), cfg.cfg2a(scale=5.0),
              cfg.static_gravity(0.3, rule="mls", fix="A", nx=40, ny=30)):
        assert _plan(L, p, storage)[0] >= 2, p.name
    for k in range(12):
        p = random_case(k)[0]
        assert (_plan(L, p, storage)[0] >= 2) == (p.rule != "zhao_yong"), k


def test_lanes_of_a_block(L):
    ncu = 256
    for p, lanes in ((_free(100, 50, "none"), 576), (_free(128, 128), 1024),
                     (_free(700, 600), 512), (_free(700, 600, "none"), 512)):
        steps, got, blocks = _plan(L, p, "f64")
        say(f"[gpu] {p.nx}x{p.ny} {p.eos}: {steps} steps, {got} lanes, {blocks} blocks")
        assert steps >= 2 and got == lanes and (blocks > ncu) == (lanes == 512)


def test_no_blocks_where_single_steps_are_meant(L):
    assert _plan(L, _drop("zhao_yong", "none"), "f64") == (0, 0, 0)
    assert _plan(L, _drop("mls", "A"), "f16node") == (0, 0, 0)
    # FP64 arithmetic on FP32 storage: the halos cost more than the bytes saved
    assert _plan(L, cfg.cfg2a(), "f32") == (0, 0, 0)
    assert _plan(L, cfg.cfg2a(), "f64")[0] >= 2
    with L.Domain(_drop("mls", "A"), storage="f32", history_capacity=16) as d:
        on = d.blocks()
        assert on[0] >= 2
        L.lbm_set_profiling(d.h, 1)
        assert d.blocks() == (0, 0, 0)
        L.lbm_set_profiling(d.h, 0)
        L.lbm_set_steps_per_pass(d.h, 2)
        assert d.blocks() == on
        L.lbm_set_steps_per_pass(d.h, 2, 16)
        assert d.blocks() == (0, 0, 0)
        L.lbm_set_steps_per_pass(d.h, 2, 0)
        assert d.blocks() == on


def test_a_refused_setting_changes_nothing(L):
    with L.Domain(_drop("mls", "A"), storage="f32", history_capacity=16) as d:
        for tile_h in (0, 16):
            L.lbm_set_steps_per_pass(d.h, 2, tile_h)
            setting, on = L.lbm_get_steps_per_pass(d.h), d.blocks()
            assert (on[0] >= 2) == (tile_h == 0)
            for steps, refused in ((2, 3), (2, -1), (3, 0), (1, -1)):
                assert L.lib().lbm_set_steps_per_pass(d.h, steps, refused) == L.LBM_EINVAL
                assert L.lbm_get_steps_per_pass(d.h) == setting
                assert d.blocks() == on, (steps, refused)


@pytest.mark.parametrize("eos,nx,ny,period,blocks", [
    ("exp", 1700, 1700, 0, True), ("exp", 1800, 1700, 0, False),    # no walls
    ("none", 1800, 1700, 0, True),                                  # single phase
    ("exp", 3500, 3500, 64, True), ("exp", 3700, 3700, 64, False),  # few links
    ("exp", 3700, 3700, 32, True), ("none", 3700, 3700, 64, True)])
def test_blocks_or_the_two_step_kernel(L, eos, nx, ny, period, blocks):
    p = _free(nx, ny, eos)
    if period:
        w = _pillars(nx, ny, period)
        p = p.with_(solid=w.solid, links=w.links, rule="halfway", fix="none")
    with L.Domain(p, storage="f32_arith32", history_capacity=16) as d:
        assert d.blocks()[0] >= 2
        L.lbm_set_steps_per_pass(d.h, 2)
        say(f"[gpu] two steps per pass, {eos} {nx}x{ny}, {len(p.links)} links: {d.blocks()}")
        assert (d.blocks()[0] >= 2) == blocks
        before = d.total_mass()
        d.step(4)
        assert abs(d.total_mass() - before) <= 1e-6 * before


def test_default_tiles_of_the_per_node_form(L):
    """64 columns only where a lattice is small or narrow: a tile's LDS does not
    shrink with its columns."""
    for nx, ny, want in ((300, 300, (64, 3)), (1200, 1000, (256, 6)), (1408, 1408, (256, 9)),
                         (2048, 2048, (128, 9)), (50, 20000, (64, 6)), (4064, 3000, (256, 15))):
        with L.Domain(_free(nx, ny), storage="f16node", history_capacity=16) as d:
            i = d.info()
            say(f"[gpu] {nx}x{ny}: tiles of {i['tile_w']}x{i['tile_h']}")
            assert (i["tile_w"], i["tile_h"]) == want


def test_tables_that_do_not_fit_a_block(L):
    """With a third of the nodes solid a block of 32 x 32 has more links than a
    workgroup has lanes."""
    p = _halfway((np.random.default_rng(5).random((96, 96)) < 0.33).astype(np.uint8))
    say(f"[gpu] {len(p.links)} links in 96x96 nodes")
    with L.Domain(p, storage="f64", history_capacity=64) as a, \
            L.Domain(p, storage="f64", history_capacity=64) as b:
        assert a.blocks() == (0, 0, 0)
        L.lbm_set_profiling(b.h, 1)
        a.step(9)
        b.step(9)
        assert all(np.array_equal(x, y) for x, y in zip(a.moments(), b.moments()))
        assert np.array_equal(a.mass_history(), b.mass_history())


def test_batches(L):
    for storage in STORAGES + ["f16node"]:
        with L.Batch(storage=storage, eos="cs", max_instances=4, arena_bytes=1 << 27) as b:
            assert b.blocks() == (0, 0, 0)
            for k in range(3):
                b.add(cfg.batch_instance(k, seed=11, side_lo=40, side_hi=90), 20,
                      history_capacity=32)
            b.run(10)
            say(f"[gpu] batch {storage}: {b.blocks()}")
            assert (b.blocks()[0] >= 2) == (storage != "f16node")
            b.add(_drop("zhao_yong", "none"), 20, history_capacity=32)
            b.run(5)
            assert b.blocks() == (0, 0, 0)


def test_batch_without_room_for_its_tables(L):
    """Pillars five nodes apart: the tables of all four instances are larger
    than an eighth of the arena that holds them, those of one are not."""
    p = _pillars(255, 255, 5)
    with L.Domain(p, storage="f16dev", history_capacity=64) as d:
        L.lbm_set_profiling(d.h, 1)
        want = []
        for n in (12, 8):
            d.step(n)
            want.append((d.moments(), d.mass_history()))
    with L.Batch(storage="f16dev", eos="none", max_instances=4, arena_bytes=44 << 20) as b:
        slots = [b.add(p, 20, history_capacity=64) for _ in range(4)]
        b.run(12)
        say(f"[gpu] four instances: {b.blocks()}, {b.info()['arena_used']} bytes of the arena")
        assert b.blocks() == (0, 0, 0)
        for s in slots:
            assert all(np.array_equal(x, y) for x, y in zip(b.moments(s), want[0][0]))
            assert np.array_equal(b.mass_history(s), want[0][1])
        for s in slots[1:]:
            b.remove(s)
        b.run(8)
        say(f"[gpu] one instance: {b.blocks()}")
        assert b.blocks()[0] >= 2
        assert all(np.array_equal(x, y) for x, y in zip(b.moments(slots[0]), want[1][0]))
        assert np.array_equal(b.mass_history(slots[0]), want[1][1])

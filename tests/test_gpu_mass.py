"""The total mass against the sum of the densities that lbm_moments reads out,
added as rational numbers: a step's mass is that sum, rounded.  Domains of more
than 2^24 nodes whose densities all leave the same rest over the unit of the
sums, which is where the sum of the rests is largest; and densities far below
the unit."""
import sys
from fractions import Fraction

import numpy as np
import pytest

from lbm_inputs import configs as cfg

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    from paper_1908_09235_amd import lbm
    lbm.lib()
    return lbm


def _still(nx, ny, rho0):
    """A fluid without walls or forces, at rest but for the density given."""
    return cfg.couette(10, rule="halfway", fix="none").with_(
        nx=nx, ny=ny, solid=np.zeros((ny, nx), np.uint8),
        links=cfg.couette(10).links[:0], rho0=rho0, rho_wall=np.ones((ny, nx)),
        name=f"still_{nx}x{ny}")


def _sum(rho):
    v, n = np.unique(rho, return_counts=True)
    return sum((Fraction(float(x)) * int(k) for x, k in zip(v, n)), Fraction(0))


def _close(got, want):
    """Rounded once, and the sum of the three parts it is rounded from again."""
    ulp = np.spacing(abs(float(want)))
    return abs(Fraction(float(got)) - want) <= Fraction(float(ulp))


@pytest.mark.parametrize("rest", [0.44, -0.44])
@pytest.mark.parametrize("form", ["single steps", "blocks"])
def test_rests_of_one_sign(L, form, rest):
    # the unit is 2^-40 of the power of two above the largest density
    nx, ny = 4480, 4481
    assert abs(rest) * nx * ny > 2 ** 23
    p = _still(nx, ny, np.full((ny, nx), 0.75 + rest * 2.0 ** -40))
    say(f"[gpu] mass of {nx}x{ny} equal densities, rest {rest} units, {form}")
    with L.Domain(p, storage="f64", history_capacity=64) as d:
        if form == "single steps":
            L.lbm_set_profiling(d.h, 1)
        for n in (0, 1, 7):
            if n:
                d.step(n)
            want = _sum(d.moments()[0])
            got = d.total_mass()
            say(f"    t = {d.t}: off by {float(Fraction(got) - want)!r}")
            assert _close(got, want)
        for m in d.mass_history():
            assert abs(m - float(want)) <= 1e-13 * float(want)


def test_densities_below_the_unit(L):
    # e-folds over four nodes from 1 in the middle down to 2^-42, an eighth of
    # the unit, which most nodes have
    n = 400
    y, x = np.mgrid[:n, :n] - n // 2
    p = _still(n, n, np.maximum(np.exp(-np.hypot(x, y) / 4.0), 2.0 ** -42))
    say(f"[gpu] mass of {n}x{n} densities from 1 to 2^-42")
    with L.Domain(p, storage="f64", history_capacity=64) as a, \
            L.Domain(p, storage="f64", history_capacity=64) as b:
        L.lbm_set_profiling(b.h, 1)  # single steps
        a.step(10)                   # nine of them in launches of several
        for k, got in enumerate(a.mass_history()):
            want = _sum(b.moments()[0])
            alone = b.total_mass()
            say(f"    t = {k}: off by {float(Fraction(got) - want)!r}, single steps "
                f"{float(Fraction(alone) - want)!r} of {got!r}")
            assert np.isfinite(got) and _close(got, want) and _close(alone, want)
            assert got == alone
            b.step(1)


@pytest.mark.parametrize("rho", [3e-150, 3e-250, 1.3e-290, 3e-304, 3e200])
def test_densities_of_any_size(L, rho):
    n = 64
    p = _still(n, n, np.full((n, n), rho))
    say(f"[gpu] mass of {n}x{n} densities of {rho!r}")
    with L.Domain(p, storage="f64", history_capacity=64) as d:
        for k in (0, 1, 9):
            if k:
                d.step(k)
            want = _sum(d.moments()[0])
            say(f"    t = {d.t}: {d.total_mass()!r}, {float(want)!r}")
            assert _close(d.total_mass(), want)


@pytest.mark.parametrize("nx,ny", [(64, 64), (1300, 1250)])
@pytest.mark.parametrize("form", ["single steps", "blocks"])
def test_densities_beyond_the_units(L, form, nx, ny):
    # too large for the integers: the parts are FP64 sums, whose error is at
    # most a rounding a term
    p = _still(nx, ny, np.full((ny, nx), 1.7e280))
    say(f"[gpu] mass of {nx}x{ny} densities of 1.7e280, {form}")
    with L.Domain(p, storage="f64", history_capacity=64) as d:
        if form == "single steps":
            L.lbm_set_profiling(d.h, 1)
        d.step(9)
        want = _sum(d.moments()[0])
        hist = d.mass_history()
        say(f"    {hist[-1]!r}, {float(want)!r}")
        assert np.all(np.abs(hist - float(want)) <= nx * ny * 2.0 ** -53 * float(want))


@pytest.mark.parametrize("storage", ["f64", "f32", "f32_arith32", "f16dev", "f16node"])
def test_tall_tiles(L, storage):
    """Tiles of more rows than one lane adds up run as several."""
    ny, nx = 1300, 300
    y, x = np.mgrid[:ny, :nx]
    p = _still(nx, ny, 1.0 + 0.1 * np.cos(0.05 * x) * np.sin(0.01 * y))
    got = []
    for w, h in ((64, 3), (64, 511), (128, 512), (256, 513), (256, 1300), (64, 4000)):
        with L.Domain(p, storage=storage, tile_w=w, tile_h=h, history_capacity=16) as d:
            L.lbm_set_profiling(d.h, 1)
            d.step(3)
            got.append((w, h, d.mass_history()))
            if storage == "f64":
                assert _close(d.total_mass(), _sum(d.moments()[0]))
    say(f"[gpu] masses of tall tiles, {storage}: {got[0][2]}")
    for w, h, m in got[1:]:
        assert np.array_equal(m, got[0][2]), (w, h)


@pytest.mark.parametrize("ntiles", [3, 256, 257, 1024, 1025, 4096, 4097, 5120, 5121, 9217])
def test_any_number_of_partials(L, ntiles):
    """256 lanes sum the tiles' parts, 16 at a time and the last four: the edges
    of both."""
    nx = 62  # one strip of 64 columns, one row a tile
    y, x = np.mgrid[:ntiles, :nx]
    p = _still(nx, ntiles, 1.0 + 0.3 * np.cos(0.7 * x) * np.sin(0.9 * y))
    with L.Domain(p, storage="f64", tile_w=64, tile_h=1, history_capacity=16) as d:
        L.lbm_set_profiling(d.h, 1)
        d.step(2)
        want = _sum(d.moments()[0])
        say(f"[gpu] mass from {ntiles} parts: off by {float(Fraction(d.total_mass()) - want)!r}")
        assert _close(d.total_mass(), want)
        hist = d.mass_history()
    with L.Domain(p, storage="f64", tile_w=256, tile_h=16, history_capacity=16) as d:
        L.lbm_set_profiling(d.h, 1)
        d.step(2)
        assert np.array_equal(d.mass_history(), hist)


@pytest.mark.parametrize("storage", ["f32", "f32_arith32"])
@pytest.mark.parametrize("rule,fix", [("mls", "B"), ("ibb_quadratic", "A")])
def test_fp32_populations(L, storage, rule, fix):
    """Sums of FP32 populations, which are not split: the same bits from every
    tile, from two steps per pass and from blocks, and that of the densities."""
    p = cfg.cfg2a(rule=rule, fix=fix, scale=2.3)
    got = []
    for w, h, two in ((256, 9, 0), (64, 3, 0), (128, 37, 0), (256, 512, 0), (0, 0, 0), (0, 0, 8)):
        if two and rule == "ibb_quadratic":
            continue  # (refused)
        with L.Domain(p, storage=storage, tile_w=w, tile_h=h, history_capacity=64) as d:
            if two:
                L.lbm_set_steps_per_pass(d.h, 2, two)
            elif w:
                L.lbm_set_profiling(d.h, 1)
            d.step(40)
            got.append(((w, h, two, d.blocks()[0]), d.mass_history()))
            if storage == "f32":
                assert _close(d.total_mass(), _sum(d.moments()[0]))
    say(f"[gpu] masses of FP32 populations, {storage} {rule}: {got[0][1][-2:]}")
    assert got[4][0][3] > 0  # blocks among them
    for k, m in got[1:]:
        assert np.array_equal(m, got[0][1]), k

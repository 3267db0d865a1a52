"""The two-step kernel (k_main2) by its rows per tile, which keep runs off the
blocks: equal to single steps bit for bit for every rule, fix, EOS and storage
form it takes, masses, wall force and counters with them, and a state saved
after a two-step pass resumes in a domain of its own, into two-step passes,
single steps and blocks."""
import sys

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


CASES = {
    "cfg1_mls_B": lambda: cfg.cfg1("mls", "B"),
    "cfg1_mls_A": lambda: cfg.cfg1("mls", "A"),
    "cfg1_ibbl_none": lambda: cfg.cfg1("ibb_linear", "none"),
    "cfg1_halfway": lambda: cfg.cfg1("halfway", "none"),
    "cfg1_mls_bao": lambda: cfg.cfg1("mls", "bao"),
    "drop_fh_B_mrt": lambda: cfg.droplet_on_cylinder(rule="fh", fix="B", tau=0.8,
                                                     collision="mrt", rho_wall=0.05),
    "gravity_q03": lambda: cfg.static_gravity(0.3, rule="mls", fix="A", nx=40, ny=30),
    "sloped16_B": lambda: cfg.sloped_channel(16, fix="B", g0=1e-3),
    "exp_droplet": lambda: cfg.free_droplet(64, 12.0, eos="exp"),
    "couette10_mls_A": lambda: cfg.couette(10, rule="mls", fix="A"),
}
STORAGES = ["f32", "f32_arith32", "f32dev", "f16dev"]


def _step(L, d, n):
    try:
        d.step(n)
    except L.LbmError as e:
        assert e.code == L.LBM_EUNSTABLE


def _fluid_state(L, d, p, storage):
    """f*(t) of the fluid nodes (first in a saved state, after 32 bytes)."""
    st = L.lbm_get_state(d.h)
    es = 2 if storage == "f16dev" else 4
    pitch = (p.nx + 63) // 64 * 64
    plane = pitch * p.ny + 256
    f = np.frombuffer(st[32:32 + 9 * plane * es].tobytes(), np.uint16 if es == 2 else np.uint32)
    f = f.reshape(9, plane)[:, :pitch * p.ny].reshape(9, p.ny, pitch)[:, :, :p.nx]
    return f[:, ~p.solid.astype(bool)]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("case", sorted(CASES))
def test_two_step_kernel_equals_single_steps(L, case, storage):
    p = CASES[case]()
    say(f"[gpu] two-step kernel vs single steps: {case} {storage} {p.nx}x{p.ny}")
    with L.Domain(p, storage=storage, history_capacity=256) as a, \
            L.Domain(p, storage=storage, history_capacity=256) as b:
        L.lbm_set_steps_per_pass(a.h, 2, 16)
        assert a.blocks() == (0, 0, 0)
        L.lbm_set_profiling(b.h, 1)
        for n in (2, 1, 6, 51, 140):
            _step(L, a, n)
            _step(L, b, n)
            tag = (case, storage, a.t)
            if a.t % 2 == 0:  # a's last pass made two steps
                assert np.array_equal(_fluid_state(L, a, p, storage),
                                      _fluid_state(L, b, p, storage)), tag
            for x, y in zip(a.moments(), b.moments()):
                assert np.array_equal(x, y, equal_nan=True), tag
            assert np.array_equal(a.mass_history(), b.mass_history(), equal_nan=True), tag
            assert np.array_equal(a.wall_force(), b.wall_force(), equal_nan=True), tag
        assert a.negative_rest() == b.negative_rest()


def test_state_after_a_two_step_pass(L):
    p = cfg.cfg1("mls", "A")
    with L.Domain(p, storage="f32", history_capacity=256) as a:
        L.lbm_set_steps_per_pass(a.h, 2, 16)
        a.step(20)
        state, now = L.lbm_get_state(a.h), a.moments()
        a.step(30)
        want, hist = a.moments(), a.mass_history()
    for setting in ((2, 16), (1, 0), (2, 0)):
        say(f"[gpu] state of a two-step pass into steps per pass, rows {setting}")
        with L.Domain(p, storage="f32", history_capacity=256) as c:
            L.lbm_set_steps_per_pass(c.h, *setting)
            assert (c.blocks()[0] >= 2) == (setting != (2, 16))
            L.lbm_set_state(c.h, state)
            assert all(np.array_equal(x, y) for x, y in zip(c.moments(), now))
            c.step(30)
            assert all(np.array_equal(x, y) for x, y in zip(c.moments(), want))
            assert np.array_equal(c.mass_history(), hist)

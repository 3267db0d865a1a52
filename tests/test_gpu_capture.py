"""Step graphs of more than one step, on forms whose runs do not go through
blocks, against plain launches; and calls on a stream that the caller is
capturing, which keep to single steps.  A domain's are launches of its own
graphs, which HIP runs at once and does not record; a batch's are recorded, and
replayed several times with eager steps and synchronisations between."""
import ctypes as C
import sys

import numpy as np
import pytest

from lbm_inputs import configs as cfg

from _hip import hip

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    from paper_1908_09235_amd import lbm
    lbm.lib()
    return lbm


@pytest.mark.parametrize("rule,storage,rows", [
    ("zhao_yong", "f64", 0), ("mls", "f16node", 0), ("mls", "f32", 16)])
def test_graphs_of_several_steps(L, rule, storage, rows):
    p = cfg.cfg1(rule, "B") if rule == "mls" else cfg.static_gravity(0.3, rule=rule, fix="none")
    say(f"[gpu] graphs of several steps, {rule} {storage}, rows of two-step passes {rows}")
    with L.Domain(p, storage=storage, history_capacity=512) as g, \
            L.Domain(p, storage=storage, history_capacity=512) as e:
        if rows:
            L.lbm_set_steps_per_pass(g.h, 2, rows)
        assert g.blocks() == (0, 0, 0)
        L.lbm_set_profiling(e.h, 1)  # timed steps launch every kernel
        for n in (1, 2, 5, 37, 64, 3, 100):
            g.step(n)
            e.step(n)
            assert all(np.array_equal(a, b) for a, b in zip(g.moments(), e.moments())), n
            assert g.total_mass() == e.total_mass()
        state = L.lbm_get_state(g.h)
        g.step(33)
        want, hist = g.moments(), g.mass_history()
        g.step(5)
        L.lbm_set_state(g.h, state)
        g.step(33)
        assert all(np.array_equal(a, b) for a, b in zip(g.moments(), want))
        assert np.array_equal(g.mass_history(), hist)


class Captured:
    """What `work` enqueues on `stream`, as a graph."""

    def __init__(self, stream, work):
        self.H, self.s = hip(), stream
        for f in ("hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphInstantiate",
                  "hipGraphLaunch", "hipGraphDestroy", "hipGraphExecDestroy",
                  "hipStreamSynchronize"):
            getattr(self.H, f).argtypes = None
        assert self.H.hipStreamBeginCapture(self.s, C.c_int(1)) == 0  # thread local
        try:
            work()
        finally:
            self.g, self.x = C.c_void_p(), C.c_void_p()
            rc = self.H.hipStreamEndCapture(self.s, C.byref(self.g))
        assert rc == 0 and self.g
        assert self.H.hipGraphInstantiate(C.byref(self.x), self.g, None, None, C.c_size_t(0)) == 0

    def launch(self):
        assert self.H.hipGraphLaunch(self.x, self.s) == 0
        assert self.H.hipStreamSynchronize(self.s) == 0

    def close(self):
        self.H.hipGraphExecDestroy(self.x)
        self.H.hipGraphDestroy(self.g)


@pytest.fixture
def stream():
    H, s = hip(), C.c_void_p()
    H.hipStreamCreateWithFlags.argtypes = [C.POINTER(C.c_void_p), C.c_uint]
    H.hipStreamDestroy.argtypes = [C.c_void_p]
    assert H.hipStreamCreateWithFlags(C.byref(s), 1) == 0
    yield s
    H.hipStreamDestroy(s)


@pytest.mark.parametrize("storage", ["f64", "f16dev"])
@pytest.mark.parametrize("warm", [0, 9])
def test_domain_on_a_captured_stream(L, stream, storage, warm):
    p = cfg.cfg1("mls", "A")
    say(f"[gpu] captured steps after {warm} others, {storage}")
    with L.Domain(p, storage=storage, history_capacity=256, stream=stream.value) as a, \
            L.Domain(p, storage=storage, history_capacity=256) as b:
        assert a.blocks()[0] >= 2
        L.lbm_set_profiling(b.h, 1)
        if warm:
            a.step(warm)
            b.step(warm)
        L.lbm_sync(a.h)
        for n in (1, 6, 2 * a.blocks()[0] + 3):
            c = Captured(stream, lambda: L.lbm_step_async(a.h, n))
            b.step(n)
            try:
                for k in range(3):  # (nothing was recorded)
                    assert all(np.array_equal(x, y) for x, y in zip(a.moments(), b.moments())), n
                    c.launch()
            finally:
                c.close()
            a.step(n)
            b.step(n)
            assert all(np.array_equal(x, y) for x, y in zip(a.moments(), b.moments())), n
            assert np.array_equal(a.mass_history(), b.mass_history())


def test_batch_on_a_captured_stream(L, stream):
    ps = [cfg.batch_instance(k, seed=11, side_lo=40, side_hi=90) for k in range(3)]
    say("[gpu] captured steps of a batch")
    doms = [L.Domain(p, storage="f64", history_capacity=256) for p in ps]
    try:
        with L.Batch(storage="f64", eos="cs", max_instances=4, arena_bytes=1 << 26,
                     stream=stream.value) as b:
            slots = [b.add(p, 200, history_capacity=256) for p in ps]
            b.run(9)
            b.sync()
            assert b.blocks()[0] >= 2
            for d in doms:
                L.lbm_set_profiling(d.h, 1)
                d.step(9)
            c = Captured(stream, lambda: b.run(7))
            b.sync()
            try:
                for k in range(3):
                    c.launch()
                    b.run(9)  # blocks between the replays
                    for d, s in zip(doms, slots):
                        d.step(16)
                        assert b.status(s)[0] == d.t
                        assert all(np.array_equal(x, y) for x, y in zip(b.moments(s), d.moments()))
                        assert np.array_equal(b.mass_history(s), d.mass_history()), k
            finally:
                c.close()
    finally:
        for d in doms:
            d.close()

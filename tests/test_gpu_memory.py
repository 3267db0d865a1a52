"""Device memory of a domain and of a batch, in a process of its own whose
allocations are counted and fail one at a time.  A domain whose tables for
several steps per launch find no memory takes single steps, and the tables come
last, so that they take nothing those need; every other allocation that fails ends the call
with LBM_ENOMEM and gives back what it took.  A batch does without its tables
in the same way."""
import os
import subprocess
import sys

import numpy as np
import pytest

from lbm_inputs import configs as cfg

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("what", ["domain", "batch"])
def test_allocations_that_fail(what):
    r = subprocess.run([sys.executable, "-u", "-m", "tests.test_gpu_memory", what], cwd=ROOT,
                       timeout=100, capture_output=True, text=True)
    say(r.stdout[-3000:], r.stderr[-3000:])
    assert r.returncode == 0


def _single(L, p, storage, n):
    with L.Domain(p, storage=storage, history_capacity=64) as d:
        L.lbm_set_profiling(d.h, 1)
        d.step(n)
        return d.moments(), d.mass_history()


def _domain(S, L):
    for make, storage in ((lambda: cfg.cfg1("mls", "B"), "f64"),
                          (lambda: cfg.sloped_channel(16, fix="A", g0=1e-3), "f32dev")):
        p = make()
        moments, hist = _single(L, p, storage, 20)
        base = S.live
        S.start()
        L.Domain(p, storage=storage, history_capacity=64).close()
        calls, passed = S.calls, []
        assert S.live == base
        for k in range(calls):
            S.start(fail=k)
            try:
                d = L.Domain(p, storage=storage, history_capacity=64)
            except L.LbmError as e:
                assert e.code == L.LBM_ENOMEM, (k, e.code)
            else:
                with d:
                    passed.append(k)
                    S.start()
                    d.step(20)
                    assert all(np.array_equal(a, b) for a, b in zip(d.moments(), moments))
                    assert np.array_equal(d.mass_history(), hist)
            assert S.live == base, k
        say(f"{p.name} {storage}: {calls} allocations, created without number {passed}")
        # the tables, the last of them: nothing that single steps need comes after
        assert passed == [calls - 1]


def _batch(S, L):
    ps = [cfg.batch_instance(k, seed=11, side_lo=40, side_hi=90) for k in range(3)]
    alone = [_single(L, p, "f64", 40) for p in ps]
    base = S.live

    def run():
        with L.Batch(storage="f64", eos="cs", max_instances=4, arena_bytes=1 << 26) as b:
            slots = [b.add(p, 40, history_capacity=64) for p in ps]
            b.run(40)
            for s, (moments, hist) in zip(slots, alone):
                assert all(np.array_equal(x, y) for x, y in zip(b.moments(s), moments))
                assert np.array_equal(b.mass_history(s), hist)

    S.start()
    run()
    calls, passed = S.calls, []
    assert S.live == base
    for k in range(calls):
        S.start(fail=k)
        try:
            run()
            passed.append(k)
        except L.LbmError as e:
            assert e.code == L.LBM_ENOMEM, (k, e.code)
        assert S.live == base, k
    say(f"batch: {calls} allocations, ran without each of {passed}")
    assert len(passed) == 3              # the pool, the list of tiles, the arguments


if __name__ == "__main__":
    from tests._malloc_shim import Shim
    shim = Shim()
    from paper_1908_09235_amd import lbm
    {"domain": _domain, "batch": _batch}[sys.argv[1]](shim, lbm)
    say("done")

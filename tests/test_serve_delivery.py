"""CPU tests of when the request loop hands over a finished solve's results.

The loop runs on stand-ins for the solver, the batch and the copy to the host
that record what happens in order.  A finished result must not wait for other
requests to be set up or for an autotune, its moments (device memory that the
budget does not count) must be gone before anything new is allocated, at most
one solve's moments may exist at a time, and no failure may lose a result that
was finished before it.
"""
import types

import numpy as np
import pytest

from paper_2208_09267_amd import serve
from paper_2208_09267_amd import workloads as W


class _Solver:
    def __init__(self, loop, rid):
        self.loop, self.rid, self.time = loop, rid, 0

    def step(self, n):
        self.time += n

    def moments(self):
        self.loop.event("moments", self.rid)
        self.loop.held.add(self.rid)
        self.loop.most_held = max(self.loop.most_held, len(self.loop.held))
        return (self.rid,)

    def close(self):
        self.loop.event("close", self.rid)


class _Loop:
    """A Server whose device work only records its order."""

    def __init__(self, monkeypatch, fail_start=(), fail_step_at=None, **kw):
        self.events, self.held, self.most_held = [], set(), 0
        self.fail_start, self.fail_step_at, self.steps = fail_start, fail_step_at, 0
        loop = self

        class Batch:
            def __init__(self, solvers):
                self.solvers = solvers

            def update(self, solvers):
                self.solvers = solvers

            def autotune(self, trial):
                loop.event("autotune", None)
                return 256, 0, 0

            def set_tuning(self, *a):
                pass

            def step(self, n):
                if n == 0:
                    return
                loop.event("step", n)
                loop.steps += n
                if loop.fail_step_at is not None and loop.steps >= loop.fail_step_at:
                    raise RuntimeError("a launch failed")
                for s in self.solvers:
                    s.step(n)

            def close(self):
                pass

        stream = types.SimpleNamespace(synchronize=lambda: None)
        monkeypatch.setattr(serve.vanse, "Batch", Batch)
        monkeypatch.setattr(serve.torch.cuda, "current_stream", lambda: stream)
        monkeypatch.setattr(serve.torch.cuda, "current_device", lambda: 0)
        monkeypatch.setattr(serve.torch.cuda, "Stream", lambda *a: stream)
        self.logged = []
        self.server = serve.Server(log=lambda r: self.logged.append(r.rid), **kw)
        self.server._start = self._start
        self.server._to_host = self._to_host

    def event(self, what, which):
        self.events.append((what, which))

    def _start(self, rid, work, now):
        self.event("start", rid)
        if rid in self.fail_start:
            raise MemoryError("no memory for request %d" % rid)
        res = serve.Result(rid, work.name, arrival=now, steps=work.steps, cells=work.ncells)
        return serve._Active(rid, work, _Solver(self, rid), work.steps, res), res

    def _to_host(self, fields):
        self.event("deliver", fields[0])
        self.held.discard(fields[0])
        return tuple(np.zeros(1) for _ in range(3))

    def run(self, steps, edge=8):
        work = [W.Workload("r%d" % k, "D3Q19", (edge, edge, edge), 0.7, n, 0.75, 100.0, seed=k)
                for k, n in enumerate(steps)]
        return self.server.run([(0.0, w) for w in work], realtime=False)

    def index(self, what, which):
        return self.events.index((what, which))


def test_results_are_handed_over_before_other_requests_are_set_up(monkeypatch):
    loop = _Loop(monkeypatch, max_active=2, autotune=False)
    res = loop.run([20, 40, 60, 30])
    assert [r.rid for r in res] == [0, 1, 2, 3] and all(r.error is None for r in res)
    assert sorted(loop.logged) == [0, 1, 2, 3]
    for k, (what, rid) in enumerate(loop.events):
        if what == "start":  # nothing that finished is still waiting
            done = {r for w, r in loop.events[:k] if w == "moments"}
            assert done <= {r for w, r in loop.events[:k] if w == "deliver"}, rid


def test_results_are_handed_over_before_an_autotune(monkeypatch):
    loop = _Loop(monkeypatch, autotune=True)
    loop.run([40, 2000, 4000])  # each retirement leaves another size class
    for k, (what, _) in enumerate(loop.events):
        if what == "autotune":
            done = {r for w, r in loop.events[:k] if w == "moments"}
            assert done <= {r for w, r in loop.events[:k] if w == "deliver"}
    assert sum(w == "autotune" for w, _ in loop.events) >= 2


def test_one_solves_moments_at_a_time(monkeypatch):
    loop = _Loop(monkeypatch, autotune=False)
    loop.run([30, 30, 30, 30, 50])  # four retire at the same boundary
    assert loop.most_held == 1
    assert sorted(loop.logged) == [0, 1, 2, 3, 4]


def test_copies_run_beside_the_next_steps(monkeypatch):
    loop = _Loop(monkeypatch, autotune=False, chunk=8)
    loop.run([16, 100])  # nothing to admit: the copy comes after the next launches
    k = loop.index("moments", 0)
    after = [w for w, _ in loop.events[k:loop.index("deliver", 0)]]
    assert "step" in after


@pytest.mark.parametrize("kw,steps", [({"fail_start": (2,), "max_active": 2}, [20, 40, 60]),
                                      ({"fail_step_at": 25}, [20, 60])])
def test_a_failure_loses_no_finished_result(monkeypatch, kw, steps):
    fail = {k: kw.pop(k) for k in ("fail_start", "fail_step_at") if k in kw}
    loop = _Loop(monkeypatch, autotune=False, **fail, **kw)
    with pytest.raises((MemoryError, RuntimeError)):
        loop.run(steps)
    assert loop.logged == [0]

"""GPU tests of the calls whose answer the host waits for (diagnostics, the
checks of a new phi or force field, the mean mass of the 16-bit modes): they
share pinned result slots, poll for a while and then wait for the stream.

Different kinds of call in turn, on a stream with much work before them, and
from several threads with streams of their own must all see their own answer.
"""
import threading

import numpy as np
import pytest
import torch

from paper_2208_09267_amd import vanse
from paper_2208_09267_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(dims, dtype, seed, period=40.0):
    s = vanse.Solver("D3Q19", dims, 0.7, dtype)
    s.set_porosity(0.75, torch.from_numpy(W.fourier_eps(dims, seed=seed)).cuda(), period)
    s.init(None, torch.from_numpy(np.ascontiguousarray(W.taylor_green(dims, 0.02))).cuda())
    return s


def _flat(d):
    return [d[0]] + d[1] + d[2]


def test_answers_behind_milliseconds_of_work():
    dims = (128, 128, 64)
    s = _solver(dims, vanse.FP64, 1, 0.0)  # a static phi: stable over the many steps below
    pert = torch.from_numpy(W.fourier_eps(dims, seed=2)).cuda()
    bad = pert.clone()
    bad.view(-1)[12345] = float("nan")
    for k in range(3):
        s.step(300)  # about 20 ms: the poll of one ends, and the stream is waited for
        first = s.diagnostics()
        assert first == s.diagnostics()  # and of an idle stream, in the poll
        f = s.populations()
        assert abs(first[0] - float(f.sum())) <= 1e-12 * first[0]
        s.step(300)
        with pytest.raises(vanse.VanseError) as e:
            s.set_porosity(0.75, bad, 40.0)
        assert e.value.code == vanse.EINVAL
        s.step(300)
        s.set_porosity(0.75, pert)
    s.close()


def _talk(seed, rounds, out, barrier=None):
    """A sequence of every kind of call, with answers that differ per solver."""
    try:
        dims = (20 + seed, 18, 14)
        n = int(np.prod(dims))
        with torch.cuda.stream(torch.cuda.Stream()):
            a, b = _solver(dims, vanse.FP64, seed), _solver(dims, vanse.FP16_SHIFTED, seed)
            rng = np.random.default_rng(seed)
            F = torch.from_numpy(rng.uniform(-1e-5, 1e-5, (3, n))).cuda()
            wrong = F.clone()
            wrong[2, n - 1] = float("inf")
            log = []
            if barrier:
                barrier.wait()
            for k in range(rounds):
                phi = torch.full((n,), 0.05 + 0.001 * k + 0.0001 * seed, dtype=torch.float64, device="cuda")
                a.set_porosity(0.7, phi)
                a.set_force_field(F * (k + 1))
                a.step(2)
                log.append(_flat(a.diagnostics()))
                for call in (lambda: a.set_force_field(wrong), lambda: a.set_porosity(0.95, phi)):
                    try:  # reaches past 1: refused with the range it found
                        call()
                        log.append("accepted")
                    except vanse.VanseError as e:
                        log.append(str(e))
                b.init(torch.full((n,), 1.0 + 0.01 * k + 0.001 * seed, dtype=torch.float64, device="cuda"))
                b.step(1)
                log.append(_flat(b.diagnostics()))
            a.close()
            b.close()
        out[seed] = log
    except BaseException as e:  # reported by the test's thread
        out[seed] = e


def test_several_threads_see_their_own_answers():
    seeds, rounds = range(1, 9), 25
    want, got = {}, {}
    for seed in seeds:
        _talk(seed, rounds, want)
    barrier = threading.Barrier(len(seeds))
    threads = [threading.Thread(target=_talk, args=(seed, rounds, got, barrier)) for seed in seeds]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    for seed in seeds:
        assert not isinstance(want[seed], BaseException), want[seed]
        assert not isinstance(got[seed], BaseException), got[seed]
        assert got[seed] == want[seed], seed
        assert "accepted" not in got[seed] and len(want[seed]) == 4 * rounds
    assert want[1] != want[2]

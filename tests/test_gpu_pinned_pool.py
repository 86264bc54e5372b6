"""Transfers of objects that share pinned buffers: the first one of an object costs what
the later ones do, objects in several threads keep apart, and an object whose transfer
was refused or cut short leaves the others' right.
"""
import threading
import time

import numpy as np
import pytest

from paper_2510_18221_amd import workloads as wl

from gpu_util import need_gpu, say
from worldstate import assert_same_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


def cfg(seed, **kw):
    return wl.desc(**dict(dict(width=40, height=36, n_agents_init=150, capacity=400, window=5, n_scalars=8, n_actions=7,
                               e_init=150, seed=seed), **kw))


# an allocation of the buffer takes 15 - 60 us, a small transfer about 12 (and 20 by a copy):
# a first call of twice the later ones' time would have paid for one
@pytest.mark.parametrize("together", [False, True])
def test_first_transfer_does_not_allocate(eco, together):
    first, later, kept = [], [], []
    for i in range(21):
        w = eco.World(cfg(i))
        w.step(1)
        w.prepare(4)
        import torch
        torch.cuda.synchronize()
        t = [time.perf_counter()]
        for _ in range(4):
            w.read_sampled()
            t.append(time.perf_counter())
        first.append(t[1] - t[0])
        later.append(min(np.diff(t)[1:]))
        if together:
            kept.append(w)
        else:
            w.close()
    for w in kept:
        w.close()
    a, b = float(np.median(first)) * 1e6, float(np.median(later)) * 1e6
    say(f"first transfer {a:.1f} us, later {b:.1f} us")
    assert a < 2 * b + 8   # (8: what a first call costs beside the transfer)


def test_objects_in_threads(eco):
    """More threads than buffers, each with objects of its own: the results of one after another."""
    import torch
    steps, threads = 6, 10

    def work(i, out):
        s = torch.cuda.Stream()
        states = []
        for r in range(3):
            with eco.World([cfg(100 * i + r), cfg(100 * i + r, width=33, height=47)], stream=s) as w:
                for t in range(steps):
                    w.step_with_actions(wl.biased_actions(800, 7, i, t))
                    states += [w.read_state(0), w.read_state(1)]
                w.write_state(states[-2], 0)
                w.step(2)
                states += [w.read_state(0), w.read_state(1)]
                states.append(w.stats())
        out[i] = states

    alone, at_once = {}, {}
    for i in range(threads):
        work(i, alone)
    ts = [threading.Thread(target=work, args=(i, at_once)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in range(threads):
        for a, b in zip(alone[i], at_once[i]):
            if isinstance(a, dict):
                assert_same_state(a, b, f"thread {i}")
            else:
                assert a == b


def test_refused_calls_between(eco):
    a, b = eco.World(cfg(1)), eco.World(cfg(1))
    acts = np.zeros(400, np.uint8)
    acts[0] = 200   # a live slot's action that does not exist: refused after the flags were read
    for t in range(20):
        with pytest.raises(eco.EcoError):
            a.step_with_actions(acts)
        a.step(1)
        b.step(1)
        assert_same_state(a.read_state(), b.read_state(), f"step {t}")
    a.close()
    b.close()

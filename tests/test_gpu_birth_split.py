"""Births of a step at the numbers where the blocks that share a child change: with 256
compute units eight blocks a child up to 255 births (four with 32-wide layers), four up to
511, two up to 1,023, one from 1,024 on, counted over all worlds of an object.  Agents stand
four cells apart, so that every parent asked has its child and the number is exact.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import workloads as wl

from gpu_util import assert_stats_match, assert_weights_close, compare_world, need_gpu
from worldstate import empty_state

pytestmark = pytest.mark.gpu

W, H = 160, 120
N = (W // 4) * (H // 4)   # 1,200 agents a world
EDGES = [255, 256, 511, 512, 1023, 1024]


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


def cfg_of(wdtype, hidden, seed, n_actions=7):
    return wl.desc(width=W, height=H, n_agents_init=0, capacity=2 * N + 300, resource_density=0.1, regrow_prob=0.02,
                   mutation_sigma=0.05, window=3, n_scalars=4, hidden1=hidden, hidden2=hidden, n_actions=n_actions,
                   wdtype=wdtype, e_cost=0, e_eat=0, e_child=0, seed=seed)


def spaced(cfg, seed, parents=N):
    """Every agent on a cell of its own 4 x 4 block, in random slots; `parents` of them at the threshold.  A child
    (no energy) dies at its next step, before the claims."""
    rng = np.random.default_rng(seed)
    st = empty_state(W, H, cfg["capacity"], uid_next=N)
    slots = rng.choice(cfg["capacity"], N, replace=False)
    x, y = np.meshgrid(np.arange(0, W, 4), np.arange(0, H, 4))
    cells = (y * W + x).ravel().astype(np.int32)
    st["pos"][:] = 0
    st["alive"][slots], st["pos"][slots], st["occ"][cells] = 1, cells, slots
    st["uid"][slots] = np.arange(N)
    st["facing"][slots] = rng.integers(0, 4, N)
    st["energy"][slots] = 100
    st["energy"][rng.choice(slots, parents, replace=False)] = 200
    return st


def share(total, worlds):
    """Births of each world: uneven, none in the first of several."""
    if worlds == 1:
        return [total]
    return [0, total // 3, total - total // 3]


@pytest.mark.parametrize("births", EDGES)
@pytest.mark.parametrize("wdtype,hidden,worlds", [(wl.FP32, 32, 1), (wl.FP32, 64, 3), (wl.BF16, 64, 1), (wl.FP8, 128, 1),
                                                  (wl.FP8, 32, 3)])
def test_children_match_oracle(eco, births, wdtype, hidden, worlds):
    cfgs = [cfg_of(wdtype, hidden, 50 + i) for i in range(worlds)]
    gw, ows = eco.World(cfgs), [orc.OracleWorld(c) for c in cfgs]
    states = [spaced(c, [births, i]) for i, c in enumerate(cfgs)]
    for i, (ow, st) in enumerate(zip(ows, states)):
        ow.write_state(st)
        gw.write_state(st, i)
    rng = np.random.default_rng(births)
    for t in range(2):
        acts = [np.zeros(c["capacity"], np.uint8) for c in cfgs]
        for a, st, n in zip(acts, states, share(births, worlds)):
            a[rng.choice(np.flatnonzero(st["alive"]), n, replace=False)] = 5
        for ow, a in zip(ows, acts):
            ow.step(actions=a)
        gw.step_with_actions(np.concatenate(acts))
        stats = gw.stats()
        assert sum(s["births"] for s in stats) == births
        for i, (ow, n) in enumerate(zip(ows, share(births, worlds))):
            assert stats[i]["births"] == n
            gs = compare_world(gw, ow, f"world {i} step {t}", i, weights_slots=2)
            assert_stats_match(stats[i], ow.stats(), f"world {i} step {t}")
            children = np.flatnonzero((gs["alive"] == 1) & (gs["energy"] == 0))
            assert len(children) == n
            for s in np.concatenate([children[:1], children[:: max(1, n // 8)], children[-1:]]):
                for master in (True, False):
                    assert_weights_close(gw.read_weights(int(s), i, master=master), ow.weights(int(s), master=master),
                                         f"world {i} child {s} step {t}")
    gw.close()


@pytest.mark.parametrize("births", EDGES)
@pytest.mark.parametrize("worlds", [1, 3])
def test_records_inside_a_call(eco, births, worlds):
    """Four steps in one call and in four: records completed by the next step's launch and by the call's end.
    Every policy rests, so that the parents' cells behind stay free."""
    cfgs = [cfg_of(wl.FP32, 64, 60 + i, n_actions=5) for i in range(worlds)]
    a, b = eco.World(cfgs), eco.World(cfgs)
    rest = np.zeros(a.P, np.float32)
    rest[-5] = 60.0   # the first of the output biases
    rng = np.random.default_rng(births)
    for i, (c, n) in enumerate(zip(cfgs, share(births, worlds))):
        st = spaced(c, [births, i], parents=n)
        for w in (a, b):
            w.write_state(st, i)
        for s in np.flatnonzero(st["alive"]):
            m = rest.copy()
            m[rng.integers(0, a.P - 5, 4)] = rng.random(4).astype(np.float32)   # traits of their own
            for w in (a, b):
                w.write_weights(int(s), m, i)
    a.step(4)
    for _ in range(4):
        b.step(1)
    for i, n in enumerate(share(births, worlds)):
        for x, y in zip(a.stats_history(i, 4), b.stats_history(i, 4)):
            assert x["births"] == n and x["population"] == N + n
            for k, v in x.items():
                if k in ("trait_mean", "trait_var"):   # the children's sums in another order
                    assert abs(v - y[k]) <= 1e-12 * abs(y[k]), (i, k, v, y[k])
                else:
                    assert v == y[k], (i, k, v, y[k])
        sa, sb = a.read_state(i), b.read_state(i)
        for k in ("alive", "pos", "uid", "energy"):
            np.testing.assert_array_equal(sa[k] * sa["alive"], sb[k] * sb["alive"], err_msg=k)
        for s in np.flatnonzero(sa["alive"])[:: 200]:
            np.testing.assert_array_equal(a.read_weights(int(s), i), b.read_weights(int(s), i))
    a.close()
    b.close()

"""Births at the sizes where their launch changes shape: the number of births of a
step decides how many blocks share one child (eight, four, two, one), and the
records of steps inside one call are completed by the launch after the births.
Every child's weights are compared with the oracle's, every record with its.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import workloads as wl

from gpu_util import assert_stats_match, assert_weights_close, compare_world, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


def parents_world(n, wdtype=wl.FP32, hidden=32, **kw):
    """n agents at the reproduction threshold; a child is born with no energy and dies at its first step."""
    base = dict(width=160, height=120, n_agents_init=n, capacity=2 * n + 300, resource_density=0.1, regrow_prob=0.02,
                mutation_sigma=0.05, window=3, n_scalars=4, hidden1=hidden, hidden2=hidden, n_actions=7, wdtype=wdtype,
                e_init=200, e_cost=0, e_eat=0, e_child=0, seed=5)
    base.update(kw)
    return wl.desc(**base)


# births: one; below and above 128 (eight blocks a child, with 32-wide layers four), 256, 512 and 1,024 (one block)
@pytest.mark.parametrize("births", [1, 100, 200, 400, 900, 1500])
@pytest.mark.parametrize("wdtype,hidden", [(wl.FP32, 32), (wl.BF16, 64), (wl.FP8, 128)])
def test_children_match_oracle(eco, births, wdtype, hidden):
    n = 1700
    cfg = parents_world(n, wdtype, hidden)
    ow, gw = orc.OracleWorld(cfg), eco.World(cfg)
    rng = np.random.default_rng([births, wdtype])
    for t in range(2):
        before = gw.read_state()["uid"].max()
        acts = np.zeros(cfg["capacity"], np.uint8)
        acts[rng.choice(n, births, replace=False)] = 5
        ow.step(actions=acts)
        gw.step_with_actions(acts)
        gs = compare_world(gw, ow, f"{births} births step {t}", weights_slots=2)
        assert_stats_match(gw.stats()[0], ow.stats(), f"{births} births step {t}")
        children = np.flatnonzero((gs["alive"] == 1) & (gs["age"] == 0))
        assert 0 < len(children) <= births
        for s in children[:: max(1, len(children) // 12)]:
            for master in (True, False):
                assert_weights_close(gw.read_weights(int(s), master=master), ow.weights(int(s), master=master),
                                     f"child {s} step {t}")
    gw.close()


@pytest.mark.parametrize("worlds", [1, 3])
@pytest.mark.parametrize("side", [24, 150])   # 24: the single-block launch (one world), 150: the separate kernels
def test_records_inside_a_call(eco, worlds, side):
    """Seven steps in one call and in seven calls: the same records, births in every step."""
    cfgs = [parents_world(side * side // 6, width=side, height=side + 2 * i, seed=i) for i in range(worlds)]
    a, b = eco.World(cfgs), eco.World(cfgs)
    a.step(7)
    for _ in range(7):
        b.step(1)
    for w in range(worlds):
        ha, hb = a.stats_history(w, 7), b.stats_history(w, 7)
        assert all(h["births"] > 0 for h in ha)
        for x, y in zip(ha, hb):
            for k, v in x.items():
                if k in ("trait_mean", "trait_var"):   # the children's sums in another order
                    assert abs(v - y[k]) <= 1e-12 * abs(y[k]), (w, k, v, y[k])
                else:
                    assert v == y[k], (w, k, v, y[k])
    a.close()
    b.close()


# every agent claims at every step, so most empty cells have two to four claimants;
# grids one or two cells wide have the same cell on several sides
@pytest.mark.parametrize("w,h,n", [(1, 1, 1), (1, 9, 4), (9, 1, 4), (2, 2, 2), (2, 40, 30), (3, 3, 5), (64, 64, 1600),
                                   (150, 101, 6000)])
@pytest.mark.parametrize("ecology", [False, True])
@pytest.mark.parametrize("split", [False, True])
def test_contended_claims_match_oracle(eco, w, h, n, ecology, split):
    kw = dict(width=w, height=h, n_agents_init=n, capacity=w * h + 3, mutation_sigma=0.05,
              window=3 if min(w, h) > 2 else 1, n_scalars=8, hidden1=32, hidden2=32, wdtype=wl.BF16, e_cost=0, e_init=9000, e_repro=50, seed=w * h)
    if ecology:
        cfg = wl.ecology_desc(eco=dict(b_repro=1, w_child=1, w_init=5000, b_init=90), **kw)
    else:
        cfg = wl.desc(n_actions=7, resource_density=0.3, **kw)
    ow, gw = orc.OracleWorld(cfg), eco.World(cfg)
    if split:
        gw.set_flags(eco.RT_USE_GRAPH | eco.RT_SPLIT_STEP)
    rng = np.random.default_rng([w, h])
    for t in range(4):
        acts = np.where(rng.random(cfg["capacity"]) < 0.8, 7 if ecology else 5, rng.integers(0, 3, cfg["capacity"]))
        ow.step(actions=acts.astype(np.uint8))
        gw.step_with_actions(acts.astype(np.uint8))
        compare_world(gw, ow, f"{w} x {h} step {t}", weights_slots=3)
        st = gw.stats()[0]
        assert_stats_match(st, ow.stats(), f"{w} x {h} step {t}")
        if n > 1000 and t == 0:
            assert st["births"] > 400 and st["births_blocked_cell"] > 400
    gw.close()

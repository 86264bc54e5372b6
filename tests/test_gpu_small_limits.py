"""The single-block step (k_step_small) at its limits, against the separate kernels and
the oracle: the most slots and cells an object may have (include/eco.h names both), live
agents in either half of the slots and more of them than the block has threads, a width
that is not a multiple of four with a ragged last group of cells, and graphs of more than
one step, whose records the block beside it completes.  Each case first shows that its
object takes the single block.
"""
import os
import re

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import eco as eco_mod
from paper_2510_18221_amd import workloads as wl

from gpu_util import assert_stats_match, assert_weights_close, compare_world, need_gpu
from worldstate import assert_same_state

pytestmark = pytest.mark.gpu

with open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "eco.h")) as f:
    LIMITS = {k: int(v) for k, v in re.findall(r"#define ECO_SMALL_STEP_MAX_(SLOTS|CELLS) (\d+)u", f.read())}


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


def busy(**kw):
    """Births and deaths in every step: agents at the reproduction threshold, children born with no energy."""
    base = dict(width=64, height=64, n_agents_init=3400, capacity=8192, resource_density=0.3, regrow_prob=0.05,
                mutation_sigma=0.05, window=5, n_scalars=8, hidden1=32, hidden2=32, n_actions=7, e_init=200, e_cost=0,
                e_child=0, seed=41)
    base.update(kw)
    return wl.desc(**base)


def eco_world(**kw):
    e = dict(w_cost=1, age_shift=6, b_init=4, terrain_scale=12, sea_level=12, water_per_depth=3, **kw.pop("eco", {}))
    base = dict(width=64, height=64, n_agents_init=3000, capacity=8192, window=7, hidden1=32, hidden2=32,
                mutation_sigma=0.05, e_init=250, flags=eco_mod.DESC_ECOLOGY | eco_mod.DESC_TERRAIN)
    base.update(kw)
    return wl.ecology_desc(eco=e, **base)


COLOUR = eco_mod.DESC_COLOUR_VISION
CASES = {
    # every slot pass and cell group full, up to four agents a thread
    "limits": busy(),
    "limits_colour_attack": busy(flags=COLOUR, attack_enabled=1, e_child=40, wdtype=wl.BF16, seed=42),
    # the ecology with terrain, colours and strikes
    "eco_limits": eco_world(n_actions=9, attack_enabled=1, flags=eco_mod.DESC_ECOLOGY | eco_mod.DESC_TERRAIN | COLOUR,
                            eco=dict(attack_damage=50), seed=43),
    # 63 x 65 cells: the flow's path cell by cell, three cells in the last group
    "eco_odd": eco_world(width=63, height=65, n_agents_init=1500, capacity=4000, seed=44),
}


def spread(st, seed):
    """The same agents in random slots of the whole capacity."""
    cap = st["alive"].size
    old = np.flatnonzero(st["alive"])
    new = np.sort(np.random.default_rng(seed).choice(cap, old.size, replace=False))
    out = dict(st)
    for k, v in st.items():
        if isinstance(v, np.ndarray) and v.size == cap and k != "occ":
            out[k] = np.zeros_like(v)
            out[k][new] = v[old]
    assert st["occ"].size != cap
    out["occ"] = np.full_like(st["occ"], -1)
    out["occ"][out["pos"][new]] = new
    return out


def takes_single_block(eco, cfg):
    w = eco.World(cfg)
    w.set_flags(eco.RT_TIME_KERNELS)
    w.step(1)
    kt = w.kernel_times(reset=True)
    w.close()
    assert kt["move"][1] == 1
    apart = {kt[k][1] for k in ("birth_claim", "birth_scan", "birth_commit", "compact")}
    assert len(apart) == 1
    return apart == {0}


@pytest.mark.parametrize("name", sorted(CASES))
def test_matches_oracle(eco, name):
    cfg = CASES[name]
    assert takes_single_block(eco, cfg)
    ow, gw = orc.OracleWorld(cfg), eco.World(cfg)
    st = spread(ow.state(), cfg["seed"])
    ow.write_state(st)
    gw.write_state(st)
    births = 0
    for t in range(6):
        acts = wl.biased_actions(cfg["capacity"], cfg["n_actions"], 5, t, p_forward=0.3, p_eat=0.3,
                                 **({"p_attack": 0.05} if cfg.get("attack_enabled") else {}))
        ow.step(actions=acts)
        gw.step_with_actions(acts)
        gs = compare_world(gw, ow, f"{name} step {t}", weights_slots=3)
        stats = gw.stats()[0]
        assert_stats_match(stats, ow.stats(), f"{name} step {t}")
        births += stats["births"]
        for s in np.flatnonzero((gs["alive"] == 1) & (gs["age"] == 0))[-2:]:   # the step's last children
            assert_weights_close(gw.read_weights(int(s)), ow.weights(int(s)), f"{name} child {s} step {t}")
    assert births > 0
    gw.close()


# 40 steps: a graph of 32 and one of the rest; agents that live on, so that the counts stay
@pytest.mark.parametrize("name", sorted(CASES))
def test_equals_separate_kernels_over_graphs(eco, name):
    cfg = CASES[name]
    assert takes_single_block(eco, cfg)
    a, b, c = eco.World(cfg), eco.World(cfg), eco.World(cfg)
    b.set_flags(eco.RT_USE_GRAPH | eco.RT_SPLIT_STEP)
    c.set_flags(0)   # the single block, launch by launch
    st = spread(a.read_state(), cfg["seed"])
    live = np.flatnonzero(st["alive"])
    if cfg["capacity"] == LIMITS["SLOTS"]:
        assert live.size >= 3000 and (live >= LIMITS["SLOTS"] // 2).sum() > 1000
    for w in (a, b, c):
        w.write_state(st)
        for n in (40, 1, 2, 35):
            w.step(n)
    sa = a.read_state()
    for w, what in ((b, "separate kernels"), (c, "launch by launch")):
        assert_same_state(sa, w.read_state(), f"{name} against {what}")
        for x, y in zip(a.stats_history(0, 78), w.stats_history(0, 78)):
            for k, v in x.items():
                if k in ("trait_mean", "trait_var"):   # the tiles' sums in another order
                    assert abs(v - y[k]) <= 1e-12 * max(abs(v), abs(y[k])), (name, what, x["step"], k, v, y[k])
                else:
                    assert v == y[k], (name, what, x["step"], k, v, y[k])
        for s in np.flatnonzero(sa["alive"])[::400]:
            np.testing.assert_array_equal(a.read_weights(int(s)), w.read_weights(int(s)))
    assert sum(h["births"] for h in a.stats_history(0, 78)[1:]) > 0
    for w in (a, b, c):
        w.close()


# the line: the limits of the header, one cell and one slot past them, and a world well inside
@pytest.mark.parametrize("cells,slots,single", [(0, 0, True), (1, 0, False), (0, 1, False), (1 - LIMITS["CELLS"], 0, True)])
def test_objects_inside_the_limits_take_the_single_block(eco, cells, slots, single):
    cfg = wl.desc(width=LIMITS["CELLS"] + cells, height=1, n_agents_init=1, capacity=LIMITS["SLOTS"] + slots, window=1,
                  seed=1)
    assert takes_single_block(eco, cfg) == single

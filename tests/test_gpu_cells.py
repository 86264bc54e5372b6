"""The cell pass with one and with four cells per thread: grids around the line between
the two (131,072 cells, each world's rounded up to 64) and with ragged last groups and
tiles, against the oracle.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import workloads as wl

from gpu_util import assert_stats_match, compare_world, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


# 4,097 cells: past the single-block launch; 131,072 / 131,073: one and four cells per thread; 395 x 397: W % 4 = 3
@pytest.mark.parametrize("w,h", [(241, 17), (67, 99), (512, 256), (43691, 3), (395, 397)])
@pytest.mark.parametrize("kind", ["plain", "colour", "ecology", "ocean"])
def test_cells_match_oracle(eco, w, h, kind):
    flags = {"plain": 0, "colour": eco.DESC_COLOUR_VISION, "ecology": eco.DESC_ECOLOGY,
             "ocean": eco.DESC_ECOLOGY | eco.DESC_TERRAIN | eco.DESC_COLOUR_VISION}[kind]
    kw = dict(width=w, height=h, n_agents_init=900, capacity=2000, window=3, hidden1=32, hidden2=32, wdtype=wl.BF16,
              flags=flags, seed=w + h)
    if flags & eco.DESC_ECOLOGY:
        cfg = wl.ecology_desc(n_scalars=12 if flags & eco.DESC_TERRAIN else 8, attack_enabled=1, **kw)
        n_actions = 9
    else:
        cfg = wl.desc(n_actions=7, regrow_prob=0.05, resource_density=0.2, **kw)
        n_actions = 6
    ow, gw = orc.OracleWorld(cfg), eco.World(cfg)
    rng = np.random.default_rng([w, h])
    for t in range(3):
        acts = rng.integers(0, n_actions, cfg["capacity"]).astype(np.uint8)
        ow.step(actions=acts)
        gw.step_with_actions(acts)
        compare_world(gw, ow, f"{kind} {w} x {h} step {t}", weights_slots=2)
        assert_stats_match(gw.stats()[0], ow.stats(), f"{kind} {w} x {h} step {t}")
    gw.close()


def test_cells_of_uneven_worlds_match_oracle(eco):
    sides = [(300, 200), (9, 7), (250, 283)]   # 60,032 + 64 + 70,784 cells: one per thread
    cfgs = [wl.desc(width=w, height=h, n_agents_init=50, capacity=130, window=3, n_actions=7, hidden1=32, hidden2=32,
                    regrow_prob=0.05, seed=i) for i, (w, h) in enumerate(sides)]
    cfgs[1].update(n_agents_init=9)
    gw = eco.World(cfgs)
    ows = [orc.OracleWorld(c) for c in cfgs]
    gw.step(3)
    for i, ow in enumerate(ows):
        for _ in range(3):
            ow.step()
        compare_world(gw, ow, f"world {i}", i, weights_slots=2)
        assert_stats_match(gw.stats()[i], ow.stats(), f"world {i}")
    gw.close()

"""Host transfers: small arrays of a state go through the object's pinned buffer in one
launch, large ones by themselves.  A written state reads back exactly, and its
neighbours in the object are untouched, at odd sizes (tails below 16 bytes), at sizes
around the buffer's limits and with the ecology's 17 arrays.
"""
import numpy as np
import pytest

from paper_2510_18221_amd import workloads as wl

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


def random_state(eco, cfg, rng, ecology):
    """A consistent state: agents on distinct cells in random slots, every other field random."""
    cap, cells = cfg["capacity"], cfg["width"] * cfg["height"]
    n = min(cap, cells) // 2
    slots, pos = rng.choice(cap, n, replace=False), rng.choice(cells, n, replace=False).astype(np.int32)
    st = dict(step=int(rng.integers(0, 2 ** 40)), uid_next=int(rng.integers(0, 2 ** 50)),
              uid=rng.integers(0, 2 ** 60, cap).astype(np.uint64), parent_uid=rng.integers(0, 2 ** 60, cap).astype(np.uint64),
              pos=np.zeros(cap, np.int32), energy=rng.integers(1, 200, cap).astype(np.int32),
              age=rng.integers(0, 999, cap).astype(np.int32), occ=np.full(cells, -1, np.int32),
              facing=rng.integers(0, 4, cap).astype(np.uint8), alive=np.zeros(cap, np.uint8),
              action=rng.integers(0, 5, cap).astype(np.uint8), res=rng.integers(0, 2, cells).astype(np.uint8),
              wall=np.zeros(cells, np.uint8))
    st["alive"][slots], st["pos"][slots], st["occ"][pos] = 1, pos, slots
    if ecology:
        for k, m in (("water", cap), ("biomass", cap), ("hp", cap), ("cell_water", cells), ("cell_energy", cells),
                     ("cell_biomass", cells)):
            st[k] = rng.integers(1, 50, m).astype(np.int32)
    return st


# slots and cells of the written world: a few, odd, arrays around 256 KiB (65,536 int32),
# and together above the 1 MiB buffer
@pytest.mark.parametrize("cap,w,h", [(1, 3, 3), (37, 9, 7), (1001, 51, 49), (65536, 256, 256), (65537, 257, 256),
                                     (140001, 401, 399)])
@pytest.mark.parametrize("ecology", [False, True])
def test_written_state_reads_back(eco, cap, w, h, ecology):
    mk = wl.ecology_desc if ecology else wl.desc
    kw = dict(window=1, hidden1=32, hidden2=32)
    cfgs = [mk(width=13, height=11, n_agents_init=20, capacity=45, seed=1, **kw),
            mk(width=w, height=h, n_agents_init=1, capacity=cap, seed=2, **kw),
            mk(width=8, height=9, n_agents_init=30, capacity=33, seed=3, **kw)]
    world = eco.World(cfgs)
    before = [world.read_state_raw(i) for i in (0, 2)]
    st = random_state(eco, cfgs[1], np.random.default_rng([cap, ecology]), ecology)
    world.write_state(st, 1)
    got = world.read_state(1)
    for k, v in st.items():
        if isinstance(v, int):
            assert got[k] == v, k
        else:
            np.testing.assert_array_equal(got[k], v, err_msg=k)
    for i, b in zip((0, 2), before):
        np.testing.assert_array_equal(world.read_state_raw(i), b)
    stats = world.stats()
    assert [s["population"] for s in stats] == [20, int(st["alive"].sum()), 30]
    assert stats[1]["step"] == st["step"]
    world.close()


@pytest.mark.parametrize("worlds", [1, 3])
def test_actions_out_of_range(eco, worlds):
    """An action that does not exist is refused for a live slot, before anything moves, and ignored for a free one."""
    cfgs = [wl.desc(width=9, height=7, n_agents_init=5, capacity=11, window=3, n_actions=7, seed=i) for i in range(worlds)]
    a, b = eco.World(cfgs), eco.World(cfgs)
    acts = np.full(11 * worlds, 4, np.uint8)
    acts[11 * worlds - 1] = 255   # a free slot of the last world
    a.step_with_actions(acts)
    b.step_with_actions(np.full(11 * worlds, 4, np.uint8))
    for bad in (7, 255):
        acts[11 * worlds - 11] = bad   # a live slot of the last world
        with pytest.raises(Exception, match="action out of range"):
            a.step_with_actions(acts)
    for i in range(worlds):
        np.testing.assert_array_equal(a.read_state_raw(i), b.read_state_raw(i))
    assert a.stats() == b.stats()
    a.close()
    b.close()

"""Workloads of the world step whose speed is followed, through the package's public entry points.

A case is one object of one or more worlds and one pass of a program that owns it:

* kind "step": advance by `steps` whole steps, then look at the result: the last
  step's statistics, the live agents' fields by slot and the grid layers;
* kind "rollout": start the worlds again from their seeds (new weights, positions
  and resources), run an episode of `steps` steps, then look at the result;
* kind "evaluate": load a population checkpoint (state and per-agent weights are
  the caller's), take one step with the caller's actions and read what every
  policy would have done: its logits and sampled action.

The populations are stationary, so that a pass costs the same however often it is
repeated: no step cost, an eaten unit carries no energy and a child is born with
none, so that it dies at its first step.  `parents` is the share of the agents at the
reproduction threshold, and sets the rate of births and deaths (with seven actions
a seventh of them asks to reproduce in a step; with five all of them do).  The
ecology's worlds are held: no costs, no health damage, no births.  The episodes of
kind "rollout" run the full dynamics.

Sizes: the 64 x 64 world with 256 agents, the paper's table of grids (128^2 to 1024^2
with 1,092 / 4,213 / 16,345 / 63,198 live agents), the 65,536-agent world at the three
storage types, batches of uneven worlds with log-uniform sides, and the 15 x 15
window with 128-wide layers.
"""
import math
import os

import numpy as np
import torch

from paper_2510_18221_amd import eco
from paper_2510_18221_amd import workloads as wl

OPTIONS = {
    "plain": 0,
    "colour": eco.DESC_EVOLVE_TEMPERATURE | eco.DESC_COLOUR_VISION,
    "ecology": eco.DESC_ECOLOGY,
    # the paper's vision agent with attacks and the evolving temperature, in the ecology with terrain
    "ocean": eco.DESC_ECOLOGY | eco.DESC_TERRAIN | eco.DESC_COLOUR_VISION | eco.DESC_EVOLVE_TEMPERATURE,
}
HELD_ECOLOGY = dict(e_cost_move=0, w_cost=0, hp_overspend=0, age_shift=31, attack_damage=0)
DTYPES = {"f32": wl.FP32, "bf16": wl.BF16, "fp8": wl.FP8}


def _case(name=None, **kw):
    c = dict(kind="step", option="plain", dtype="f32", width=64, height=64, worlds=1, agents=256, capacity=4096,
             window=5, scalars=4, hidden=32, actions=5, parents=0.0, tuned=False, steps=100)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    big = dict(width=1024, height=1024, agents=65536, capacity=131072, window=11, scalars=8, hidden=64, actions=7)
    ocean = dict(option="ocean", window=7, scalars=12, hidden=64, actions=9, dtype="bf16")
    return [
        # the smallest call: one step of the small world, looked at after every step
        _case("small64_one_step", steps=1, parents=0.01),
        # the small world's 100 steps between two looks (a birth in most steps)
        _case("small64_100_steps", steps=100, parents=0.01),
        # the paper's Ocean runs at the smaller grid sizes, with the average population each holds
        _case("ocean128_bf16", width=128, height=128, agents=1092, capacity=8192, steps=100, **ocean),
        _case("ocean256_bf16", width=256, height=256, agents=4213, capacity=16384, steps=50, **ocean),
        # the resource-and-compass agent of the ecology at 512^2, FP8 storage
        _case("ecology512_fp8", option="ecology", width=512, height=512, agents=16345, capacity=32768, window=11,
              scalars=12, hidden=64, actions=8, dtype="fp8", steps=40),
        # the 65,536-agent world: FP32 with about one birth per hundred agents and step
        _case("world65k_f32_births", parents=0.1, tuned=True, steps=32, **big),
        # the same in BF16 where most agents can reproduce: births and deaths of a tenth of the population each step
        _case("turnover65k_bf16", parents=0.9, tuned=True, dtype="bf16", steps=20, **big),
        # FP8 storage, an uneven grid and an odd population
        _case("uneven61k_fp8", dtype="fp8", steps=40, parents=0.02,
              **dict(big, width=1100, height=939, agents=61003, capacity=100003)),
        # many independent worlds of uneven size in one object
        _case("batch24_bf16", worlds=24, width=512, height=64, agents=0, capacity=0, window=11, scalars=8, hidden=64,
              actions=7, dtype="bf16", parents=0.05, steps=20),
        # the wide agent: 15 x 15 window and 128-wide layers
        _case("wide32k_bf16", width=1024, height=1024, agents=32768, capacity=40960, window=15, scalars=8, hidden=128,
              actions=7, dtype="bf16", parents=0.05, steps=20),
        # short episodes from new seeds (parameter sweeps, evolution experiments)
        _case("rollout12_f32", kind="rollout", worlds=12, width=256, height=64, agents=0, capacity=0, window=11,
              scalars=8, hidden=64, actions=7, steps=32),
        # a checkpoint's policies evaluated from outside: state in, logits and actions out
        _case("evaluate777_f32", kind="evaluate", width=96, height=80, agents=777, capacity=777, window=11, scalars=8,
              hidden=64, actions=7, steps=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_WORK = 2.0e11    # bytes of a drawn case's pass at most (the largest listed case moves about 3e11)
MOST_MEMORY = 3.0e10  # bytes of a drawn case's weights


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["rollout", "evaluate", "evaluate"])
    dtype = rng.choice(sorted(DTYPES))
    if kind == "evaluate":
        w, h = rng.randint(40, 200), rng.randint(40, 200)
        n = _log_int(rng, 33, 1000)
        return _case(kind=kind, dtype=dtype, width=w, height=h, agents=n, capacity=n, window=rng.choice([1, 3, 5, 7, 11, 15]),
                     scalars=rng.choice([4, 8]), hidden=rng.choice([32, 64, 128]), actions=rng.choice([5, 7]), steps=1)
    if kind == "rollout":
        lo = rng.randint(32, 80)
        return _case(kind=kind, dtype=dtype, worlds=rng.randint(2, 16), width=rng.randint(lo + 1, 320), height=lo, agents=0,
                     capacity=0, window=rng.choice([5, 7, 11]), scalars=8, hidden=rng.choice([32, 64]), actions=7,
                     steps=rng.randint(10, 60))
    option = rng.choice(["plain", "plain", "plain", "ecology", "ocean", "colour"])
    eco_world = option in ("ecology", "ocean")
    scalars = rng.choice([8, 12]) if eco_world else rng.choice([4, 8])
    actions = {"ecology": 8, "ocean": 9}.get(option) or rng.choice([5, 7])
    hidden = rng.choice([32, 64, 64, 128])
    window = rng.choice([3, 5, 7, 7, 9, 11, 11, 15])
    parents = 0.0 if eco_world else rng.choice([0.0, 0.01, 0.05, 0.3])
    steps = rng.choice([1, 10, 20, 40, 100])
    if not eco_world and rng.random() < 0.25:
        lo = rng.randint(32, 96)
        c = _case(option=option, dtype=dtype, worlds=rng.randint(2, 32), width=rng.randint(lo + 1, 512), height=lo, agents=0,
                  capacity=0, window=window, scalars=scalars, hidden=hidden, actions=actions, parents=parents, steps=steps)
    else:
        w, h = _log_int(rng, 48, 1200), _log_int(rng, 48, 1200)
        n = max(32, int(w * h * rng.uniform(0.02, 0.09)))
        c = _case(option=option, dtype=dtype, width=w, height=h, agents=n, capacity=int(n * rng.uniform(1.125, 2.0)) + 8,
                  window=window, scalars=scalars, hidden=hidden, actions=actions, parents=parents, steps=steps)
    while work(c)["bytes"] > MOST_WORK or _memory(c) > MOST_MEMORY:   # fewer steps, then a smaller world
        if c["steps"] > 10:
            c["steps"] = c["steps"] // 2
        else:
            c["width"] = max(48, c["width"] * 3 // 4)
            if c["worlds"] == 1:
                c["agents"] = c["agents"] * 3 // 4
                c["capacity"] = c["capacity"] * 3 // 4 + 8
            else:
                c["worlds"] = max(2, c["worlds"] * 3 // 4)
    return c


def _worlds(case):
    """(width, height, agents, capacity) of each world of the object."""
    if case["worlds"] == 1:
        return [(case["width"], case["height"], case["agents"], case["capacity"])]
    out = []   # sides log-uniform between the case's two, 6.25% occupancy
    for side in wl.batch_sides(case["worlds"], lo=case["height"], hi=case["width"]):
        n = int(round(0.0625 * side * side))
        out.append((side, side, n, (int(1.125 * n) + 63) // 64 * 64))
    return out


def _descs(case, seed):
    flags = OPTIONS[case["option"]]
    out = []
    for i, (w, h, n, cap) in enumerate(_worlds(case)):
        kw = dict(width=w, height=h, n_agents_init=n, capacity=cap, window=case["window"], n_scalars=case["scalars"],
                  hidden1=case["hidden"], hidden2=case["hidden"], n_actions=case["actions"], mutation_sigma=0.01,
                  wdtype=DTYPES[case["dtype"]], flags=flags, seed=seed * 1000 + i)
        if flags & eco.DESC_ECOLOGY:
            out.append(wl.ecology_desc(eco=HELD_ECOLOGY, e_init=230, e_cost=0, e_repro=1 << 30,
                                       attack_enabled=1 if case["actions"] == 9 else 0, **kw))
        elif case["kind"] == "rollout":   # the full dynamics, births from the first steps on
            out.append(wl.desc(resource_density=0.3, regrow_prob=0.02, e_init=190, **kw))
        else:
            out.append(wl.desc(resource_density=0.05, regrow_prob=0.01, e_init=100, e_cost=0, e_eat=0, e_child=0, **kw))
    return out


def _spread_energies(case, world, seed):
    """The agents' energies: a share `parents` of them at the reproduction threshold, the others below."""
    rng = np.random.default_rng([seed, 7])
    for i in range(world.n_worlds):
        st = world.read_state(i)
        n = st["energy"].size
        above = rng.random(n) < case["parents"]
        st["energy"] = np.where(above, rng.integers(200, 300, n), rng.integers(1, 200, n)).astype(np.int32)
        world.write_state(st, i)


def _population(case, seed):
    """The checkpoint of kind "evaluate": every slot alive, grid, energies, ages, facings, weights and actions."""
    rng = np.random.default_rng([seed, 11])
    W, H, n = case["width"], case["height"], case["agents"]
    cells, S, h, A = W * H, case["window"], case["hidden"], case["actions"]
    D = 4 * S * S + case["scalars"]
    pos = rng.choice(cells, n, replace=False).astype(np.int32)
    occ = np.full(cells, -1, np.int32)
    occ[pos] = np.arange(n, dtype=np.int32)
    st = dict(step=int(rng.integers(0, 1000)), uid_next=n, uid=np.arange(n, dtype=np.uint64),
              parent_uid=np.full(n, 2 ** 64 - 1, np.uint64), pos=pos, energy=rng.integers(1, 200, n).astype(np.int32),
              age=rng.integers(0, 1500, n).astype(np.int32), occ=occ, facing=rng.integers(0, 4, n).astype(np.uint8),
              alive=np.ones(n, np.uint8), action=np.zeros(n, np.uint8),
              res=(rng.random(cells) < 0.1).astype(np.uint8), wall=np.zeros(cells, np.uint8))
    sizes = [(h, D), (h,), (h, h), (h,), (A, h), (A,)]
    layers = [(rng.standard_normal((n,) + s, dtype=np.float32) * np.float32(1 / math.sqrt(s[-1]))) for s in sizes]
    actions = rng.integers(0, 5, n).astype(np.uint8)
    return st, layers, actions


def _restore(world, seed):
    """The same object started from another seed."""
    world.reset(np.arange(world.n_worlds, dtype=np.uint64) + np.uint64(seed * 1000))


def prepare(case, seed):
    case = dict(case)
    world = eco.World(_descs(case, seed))
    if case["tuned"]:   # the launch shape this package's tuner has kept for the 65,536-agent world
        world.autotune(cache=os.path.join(os.path.dirname(eco.__file__), "launch_cache.jsonl"))
    state = dict(case=case, world=world, seed=seed)
    if case["kind"] == "evaluate":
        world.set_flags(eco.RT_KEEP_LOGITS)
        st, layers, actions = _population(case, seed)
        for j in range(case["agents"]):
            world.write_weights(j, np.concatenate([x[j].ravel() for x in layers]))
        state.update(checkpoint=st, actions=actions)
    else:
        if case["kind"] == "step" and not OPTIONS[case["option"]] & eco.DESC_ECOLOGY:
            _spread_energies(case, world, seed)
        world.prepare(case["steps"])
    torch.cuda.synchronize()
    return state


AGENT_FIELDS = ("uid", "parent_uid", "pos", "energy", "age", "facing", "action", "water", "biomass", "hp")
GRID_FIELDS = ("occ", "res", "cell_water", "cell_energy", "cell_biomass")


def _look(world):
    """Every world's statistics of the last step, its live agents and its grid layers."""
    stats = world.stats()
    out = {"stats." + k: np.array([s[k] for s in stats]) for k in stats[0]}
    states = [world.read_state(i) for i in range(world.n_worlds)]
    out["alive"] = np.concatenate([s["alive"] for s in states])
    out["clock"] = np.array([[s["step"], s["uid_next"]] for s in states])
    for k in AGENT_FIELDS:   # the fields of free slots are unspecified: zero here
        if k in states[0]:
            out[k] = np.concatenate([s[k] * s["alive"] for s in states])
    for k in GRID_FIELDS:
        if k in states[0]:
            out[k] = np.concatenate([s[k] for s in states]) if len(states) > 1 else states[0][k]
    return out


def run(state):
    case, world = state["case"], state["world"]
    if case["kind"] == "evaluate":
        world.write_state(state["checkpoint"])
        world.step_with_actions(state["actions"])
        return dict(_look(world), logits=world.read_logits(), sampled=world.read_sampled())
    if case["kind"] == "rollout":
        _restore(world, state["seed"])
    world.step(case["steps"])
    return _look(world)


def _params(case):
    D = 4 * case["window"] ** 2 + case["scalars"]
    h, A = case["hidden"], case["actions"]
    nw, nb = h * D + h * h + A * h, 2 * h + A
    per_agent = {"f32": 4 * (nw + nb), "bf16": 2 * (nw + nb), "fp8": nw + 8 * nb}[case["dtype"]]
    return nw, nw + nb, per_agent


def _memory(case):
    _, P, per_agent = _params(case)
    return sum(c for _, _, _, c in _worlds(case)) * (per_agent + (0 if case["dtype"] == "f32" else 4 * P))


def work(case):
    """Per step every live agent's weights once and its fields in and out, every cell's layers, and for a birth the
    parent's master in, the child's master and storage copy out; the weights written once more by a rollout."""
    nw, P, per_agent = _params(case)
    sizes = _worlds(case)
    n = sum(s[2] for s in sizes)
    cells = sum(s[0] * s[1] for s in sizes)
    slots = sum(s[3] for s in sizes)
    ecology = case["option"] in ("ecology", "ocean")
    births = 0.0 if ecology else case["parents"] * n * 0.9 * (1 if case["actions"] == 5 else 1 / 7)
    birth = 8 * P + (0 if case["dtype"] == "f32" else per_agent)
    one = n * (per_agent + 40) + cells * (20 if ecology else 3) + births * birth
    look = slots * (43 if ecology else 31) + cells * (18 if ecology else 6)
    total = case["steps"] * one + look
    if case["kind"] == "rollout":
        total += n * (birth - 4 * P) + 8 * cells
    if case["kind"] == "evaluate":
        total += look + 4 * n * case["actions"]
    return {"bytes": float(total), "flops": float(2 * case["steps"] * n * nw)}


def _observations(case, st):
    """The policies' inputs in 64 bits: the S x S window rotated so that the agent faces its top row, four channels
    a cell (agent, resource, wall, the occupant's energy bin), then the scalar sensors."""
    W, H, S = case["width"], case["height"], case["window"]
    R = S // 2
    grid = np.zeros((H, W, 4))
    occ = st["occ"].reshape(H, W)
    grid[..., 0] = occ >= 0
    grid[..., 1] = st["res"].reshape(H, W)
    energy = st["energy"].astype(np.int64)
    bins = np.minimum(8 * energy // 200, 7)
    grid[..., 3] = np.where(occ >= 0, bins[np.maximum(occ, 0)], 0)
    rows = []
    for j in range(case["agents"]):
        y, x = divmod(int(st["pos"][j]), W)
        patch = grid[np.ix_(np.arange(y - R, y + R + 1) % H, np.arange(x - R, x + R + 1) % W)]
        scalars = [energy[j] / 256.0, min(int(st["age"][j]), 1024) / 1024.0, grid[y, x, 1], float(energy[j] >= 200)]
        if case["scalars"] == 8:
            scalars += [float(st["facing"][j] == k) for k in range(4)]
        rows.append(np.concatenate([np.rot90(patch, k=int(st["facing"][j])).ravel(), scalars]))
    return np.stack(rows)


def _stored(case, m, bias):
    """The values that a storage type keeps of the FP32 parameters m [agents, rows, columns] (biases: FP32 with FP8)."""
    t = torch.from_numpy(np.ascontiguousarray(m))
    if case["dtype"] == "bf16":
        t = t.bfloat16()
    elif case["dtype"] == "fp8" and not bias:
        top = t.abs().amax(-1, keepdim=True)
        scale = torch.where(top > 0, top / 448.0, torch.ones_like(top))
        return ((t / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double() * scale.double()).numpy()
    return t.double().numpy()


def exact(case, seed):
    if case["kind"] != "evaluate":
        return None   # the state is whole numbers; the trait moments need every mutated weight
    st, layers, _ = _population(case, seed)
    x = _observations(case, st)[..., None]
    for i in range(0, 6, 2):
        x = _stored(case, layers[i], False) @ x + _stored(case, layers[i + 1], True)[..., None]
        if i < 4:
            x = np.maximum(x, 0.0)
    square = sum((v.astype(np.float64) ** 2).reshape(case["agents"], -1).sum(1) for v in layers)
    return {"logits": x[..., 0], "stats.energy_total": np.array([float(st["energy"].sum())]),
            "stats.trait_mean": np.array([square.mean()]), "stats.trait_var": np.array([square.var()])}

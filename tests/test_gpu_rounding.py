"""Written weights round to BF16 as the oracle rounds them: every exponent, ties to both
sides, the smallest and the largest floats (those that overflow included)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import workloads as wl

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


@pytest.mark.parametrize("window,scalars", [(3, 4), (3, 8), (15, 8)])   # an even and an odd number of inputs' quads
def test_written_bf16_weights_are_rounded_exactly(eco, window, scalars):
    gw = eco.World([wl.desc(width=16, height=16, n_agents_init=2, capacity=3, window=window, n_scalars=scalars, n_actions=7,
                            hidden1=32, hidden2=32, wdtype=wl.BF16, seed=1)])
    rng = np.random.default_rng([window, scalars])
    low = np.array([0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF], np.uint32)   # the half that is rounded away
    bits = rng.integers(0, 0x7F80, gw.P).astype(np.uint32) << 16 | rng.choice(low, gw.P)
    bits[:12] = np.concatenate([0x7F7F0000 | low, low]).astype(np.uint32)   # next to the largest and to zero
    m = (bits | rng.integers(0, 2, gw.P).astype(np.uint32) << 31).view(np.float32)
    m = m[rng.permutation(gw.P)]
    gw.write_weights(1, m)
    want = (np.array([orc.bf16_rne(float(x)) for x in m], np.uint32) << 16).view(np.float32).astype(np.float64)
    np.testing.assert_array_equal(gw.read_weights(1, master=True), m.astype(np.float64))
    np.testing.assert_array_equal(gw.read_weights(1), want)
    gw.close()

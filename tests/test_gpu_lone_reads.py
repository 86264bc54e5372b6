"""Reads of one array (sampled actions, logits, an agent's weights): through a pinned buffer
up to 16 KiB, above that by a copy.  Both sides of the line return the same values, and
neither takes longer than a copy of the same bytes.
"""
import ctypes
import time

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2510_18221_amd import workloads as wl

from gpu_util import LOGIT_TOL, assert_weights_close, logit_err, need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eco():
    need_gpu()
    from paper_2510_18221_amd import eco as m
    m.lib()
    return m


# bytes of the sampled actions: slots; of the logits: 32 a slot; of the weights: 6,656 and 18,944
@pytest.mark.parametrize("slots", [64, 511, 512, 513, 16383, 16384, 16385, 40000])
@pytest.mark.parametrize("window", [1, 5])
def test_values(eco, slots, window):
    cfg = wl.desc(width=32, height=32, n_agents_init=60, capacity=slots, window=window, seed=slots)
    ow, gw = orc.OracleWorld(cfg), eco.World([dict(cfg, seed=1, n_agents_init=3), cfg])   # the second world of the object
    gw.set_flags(eco.RT_KEEP_LOGITS)
    logits, sampled = ow.step(want_logits=True, want_sampled=True)
    gw.step(1)
    live = np.zeros(slots, bool)
    live[:60] = True
    got = gw.read_logits(1)
    assert logit_err(got[live], logits[live]).max() <= LOGIT_TOL and np.isnan(got[~live]).all()
    s = gw.read_sampled(1)
    assert (s[~live] == 255).all() and (s[live] < 5).all()
    assert (s[live] != sampled[live]).sum() <= 1   # (a logit's last bits can turn a draw that lies on an edge)
    for slot in (0, 59):
        for master in (False, True):
            assert_weights_close(gw.read_weights(slot, 1, master=master), ow.weights(slot, master=master), f"slot {slot}")
    gw.close()


@pytest.mark.parametrize("slots", [4096, 16384, 16448, 65536, 262144])
def test_no_longer_than_a_copy(eco, slots):
    import torch
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    w = eco.World([wl.desc(width=8, height=8, n_agents_init=4, capacity=slots, window=3)])
    src = torch.empty(slots, dtype=torch.uint8, device="cuda")
    out = np.empty(slots, np.uint8)
    p, n, stream = out.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(slots), torch.cuda.current_stream().cuda_stream
    read, copy = [], []
    for _ in range(400):
        a = time.perf_counter()
        assert eco.lib().eco_world_read_sampled(w._h, 0, p, slots) == 0
        b = time.perf_counter()
        assert hip.hipMemcpyAsync(p, ctypes.c_void_p(src.data_ptr()), n, 2, ctypes.c_void_p(stream)) == 0   # 2: to the host
        assert hip.hipStreamSynchronize(ctypes.c_void_p(stream)) == 0
        c = time.perf_counter()
        read.append(b - a)
        copy.append(c - b)
    w.close()
    r, c = float(np.median(read)) * 1e6, float(np.median(copy)) * 1e6
    say(f"{slots} bytes: read {r:.1f} us, copy {c:.1f} us")
    assert r <= 1.1 * c


def slots_world(eco, wdtype, window=3, hidden=32):
    return eco.World([wl.desc(width=16, height=16, n_agents_init=3, capacity=40, window=window, hidden1=hidden, hidden2=hidden,
                              wdtype=wdtype, seed=1)])


@pytest.mark.parametrize("wdtype", [wl.FP32, wl.BF16, wl.FP8])
def test_slots_that_had_no_weights(eco, wdtype):
    """Zeros until weights are written, also after a reset; written ones as they are, zeros among them."""
    w = slots_world(eco, wdtype)
    rng = np.random.default_rng(wdtype)
    for _ in range(2):
        for slot in (3, 4, 38, 39):
            for master in (False, True):
                assert not w.read_weights(slot, master=master).any()
        m = rng.integers(-8, 9, w.P).astype(np.float32) / 8
        for first in (0, 16, 300, w.P):   # leading zeros: fewer and more than the 16 bytes that a read looks at; all
            m[:first] = 0
            for slot in (3, 38):
                w.write_weights(slot, m)
                np.testing.assert_array_equal(w.read_weights(slot, master=True), m.astype(np.float64))
                if wdtype != wl.FP8:
                    np.testing.assert_array_equal(w.read_weights(slot), m.astype(np.float64))
                else:
                    assert (w.read_weights(slot) != 0).any() == (m != 0).any()
        w.write_weights(38, rng.standard_normal(w.P).astype(np.float32))
        w.reset()
    w.close()


def test_child_takes_no_longer_than_a_founder(eco):
    w = slots_world(eco, wl.FP32, window=5)
    w.write_weights(20, np.ones(w.P, np.float32))
    t = {0: [], 20: []}
    for _ in range(400):
        for slot in t:
            a = time.perf_counter()
            w.read_weights(slot)
            t[slot].append(time.perf_counter() - a)
    w.close()
    founder, child = (float(np.median(v)) * 1e6 for v in t.values())
    say(f"weights of 18,944 bytes: founder {founder:.1f} us, child {child:.1f} us")
    assert child <= 1.12 * founder

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

"""Steps of an object whose stream is being captured: one and two steps, which are launched
kernel by kernel otherwise, do there what more steps do (they stay graphs), so that the
number of steps decides nothing about what the capture holds."""
import ctypes

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


@pytest.mark.parametrize("side", [40, 100])   # the single block, the separate kernels
def test_few_steps_do_what_many_do(eco, side):
    import torch
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    stream = torch.cuda.Stream()
    s = ctypes.c_void_p(stream.cuda_stream)
    seen = {}
    for n in (1, 2, 3, 33, 34, 64):
        w = eco.World([wl.desc(width=side, height=side, n_agents_init=150, capacity=400, e_init=150, seed=1)], stream=stream)
        torch.cuda.synchronize()
        graph, nodes = ctypes.c_void_p(), ctypes.c_size_t(0)
        assert hip.hipStreamBeginCapture(s, 1) == 0   # 1: thread-local
        try:
            w.step(n)
            refused = False
        except eco.EcoError:
            refused = True
        ended = hip.hipStreamEndCapture(s, ctypes.byref(graph))
        if graph.value:
            assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
            hip.hipGraphDestroy(graph)
        hip.hipGetLastError()
        torch.cuda.synchronize()
        if not refused:
            step = w.stats()[0]["step"]
            assert step in (0, n)
            seen[n] = (False, ended, nodes.value, step == n)
            w.step(2)
            assert w.stats()[0]["step"] == step + 2
        else:
            seen[n] = (True, ended, nodes.value)
        w.close()
    assert len(set(seen.values())) == 1, seen

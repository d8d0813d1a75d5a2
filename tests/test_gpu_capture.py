"""Steps captured into a HIP graph by the caller: a graph of an even number of steps leaves the state in
the buffer it found it in, whatever form the steps take, so that replays advance it and eager steps
may come between them.  Every replay is checked against a simulation that takes the same steps eagerly."""
import ctypes

import numpy as np
import pytest

from devmem import hip
from paper_1705_10045_amd import inputs as I
from paper_1705_10045_amd import lbm

pytestmark = pytest.mark.gpu

THREAD_LOCAL = 1     # hipStreamCaptureModeThreadLocal
HEADER = 48          # bytes of a checkpoint before the populations (it holds the step count)


class Graph:
    """What `record` enqueues on `stream`, replayed on call."""

    def __init__(self, stream, record):
        h = hip()
        graph, self.exec, self.stream = ctypes.c_void_p(), ctypes.c_void_p(), stream
        assert h.hipStreamBeginCapture(stream, THREAD_LOCAL) == 0
        try:
            record()
        finally:
            assert h.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
        assert h.hipGraphInstantiate(ctypes.byref(self.exec), graph, None, None, ctypes.c_size_t(0)) == 0
        assert h.hipGraphDestroy(graph) == 0

    def __call__(self):
        assert hip().hipGraphLaunch(self.exec, self.stream) == 0

    def close(self):
        assert hip().hipGraphExecDestroy(self.exec) == 0


def _state(sim):
    return sim.checkpoint()[HEADER:]


def _slab(ny, nx):
    n = max(nx, ny)
    c = I.slab_2d(n=n, width=n // 3)
    return 9, c["params"], c["rho0"][:, :ny, :nx].copy(), c["u0"][:, :, :ny, :nx].copy(), c["T0"][:, :ny, :nx].copy()


def _drop(shape):
    c = I.droplet_3d(shape=shape, radius=5.0)
    return c["Q"], c["params"], c["rho0"], c["u0"], c["T0"]


@pytest.mark.parametrize("steps", [2, 10, 34])
@pytest.mark.parametrize("name,args,storage", [("row 1000", _slab(1, 1000), 8), ("plane 128x96", _slab(96, 128), 8),
                                               ("plane 128x96", _slab(96, 128), 4), ("plane 400x300", _slab(300, 400), 4),
                                               ("box 33x20x12", _drop((12, 20, 33)), 4),
                                               ("box 64^3", _drop((64, 64, 64)), 8)])
def test_replays_of_an_even_number_of_steps_advance_the_state(name, args, storage, steps):
    print("captured steps: %s %dB, %d per graph" % (name, storage, steps), flush=True)
    h, stream = hip(), ctypes.c_void_p()
    assert h.hipStreamCreateWithFlags(ctypes.byref(stream), 1) == 0
    with lbm.Sim(*args, storage_bytes=storage, stream=stream.value) as a, \
            lbm.Sim(*args, storage_bytes=storage) as b:
        a.step(2)            # the kernels are loaded before the capture
        b.step(2)
        graph = Graph(stream, lambda: a.step_async(steps))
        for between in (0, 2, 12, 0, 4):
            graph()
            a.step(between)
            b.step(steps + between)
            same = _state(a) == _state(b)
            assert same, between
        graph.close()
    assert h.hipStreamDestroy(stream) == 0

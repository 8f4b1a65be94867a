"""Steps of the field producer in one call against calls of one step: only a
call's last step writes the velocity, and the x-transformed advection term that
the next step starts from lives beside it, so neither the grouping of steps nor
a read-back in between may change a bit."""
import numpy as np
import pytest
import torch

from paper_2607_17836_amd import ns2d, synth

pytestmark = pytest.mark.gpu


# every size with kernels of its own (one and two waves a transform, the fused
# column step up to 1024, the four transforms side by side up to 512)
@pytest.mark.parametrize("n", [64, 128, 256, 512, 1024, 2048])
def test_steps_in_one_call_equal_single_steps(n):
    w0 = synth.random_vorticity(n, min(n / 10, 20), 23, omega_rms=3.0)
    a, b = (ns2d.Ns2d(n, 1e-4, 1e-3) for _ in range(2))
    for _ in range(2):   # a second vorticity starts afresh
        a.set_vorticity(w0)
        b.set_vorticity(w0)
        a.step(1)
        a.step(4)
        for _ in range(5):
            b.step(1)
            b.get_fields()
        for p, q in zip(a.get_fields(), b.get_fields()):
            assert np.array_equal(p, q)
        assert a.steps == b.steps == 5
    a.close()
    b.close()


# a step captured once and replayed goes on from where the last one ended
@pytest.mark.parametrize("n", [64, 256, 512, 1024])
def test_captured_step_replays(n):
    w0 = synth.random_vorticity(n, min(n / 10, 20), 23, omega_rms=3.0)
    stream = torch.cuda.Stream()
    a = ns2d.Ns2d(n, 1e-4, 1e-3, stream=stream.cuda_stream)
    b = ns2d.Ns2d(n, 1e-4, 1e-3)
    for s in (a, b):
        s.set_vorticity(w0)
        s.step(2)
        s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(1)
    for _ in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        b.step(1)
        for p, q in zip(a.get_fields(), b.get_fields()):
            assert np.array_equal(p, q)
    a.close()
    b.close()

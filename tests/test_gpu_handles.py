"""What making and destroying handles, and reading, may not do to the streams of
the same program."""
import gc

import numpy as np
import pytest
import torch

import oracle
from paper_1208_2080_amd import binding
from paper_1208_2080_amd import workloads as wl

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

K2 = wl.critical_coupling(2)


def test_destroy_does_not_wait():
    """The last handle is destroyed while its stream still sweeps."""
    gc.collect()
    stream = torch.cuda.Stream()
    lat = binding.Lattice(4096, 2, K2, seed=1, obs_capacity=4, stream=stream)
    lat.sweep(1)
    lat.measure(0, 1)
    torch.cuda.synchronize()
    lat.sweep(600)           # tens of milliseconds
    lat.close(sync=False)
    busy = not stream.query()
    torch.cuda.synchronize()
    assert busy


def test_destroy_while_another_stream_is_captured():
    """In a capture of the strictest mode the last handle goes, and the graph is
    whole."""
    gc.collect()
    x = torch.zeros(64, device="cuda")
    lat = binding.Lattice(24, 2, K2, seed=1, obs_capacity=4)
    lat.sweep(2)
    rows = lat.measure(0, 2)
    assert np.array_equal(rows, oracle.OracleLattice(24, 2, K2, 1).run(2))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="global"):
        x += 1
        lat.close(sync=False)
        x += 1
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 6.0
    again = binding.Lattice(24, 2, K2, seed=1, obs_capacity=4)
    again.sweep(2)
    assert np.array_equal(again.measure(0, 2), rows)
    again.close()


def test_sweep_by_steps_on_a_stream_under_capture_is_refused():
    """The call fails before it has touched the stream, so the capture goes on."""
    stream = torch.cuda.Stream()
    lat = binding.Lattice(200, 2, K2, seed=2, obs_capacity=4, stream=stream)
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        x += 1
        with pytest.raises(binding.SwError) as e:
            lat.sweep(1)
        x += 1
    assert e.value.code == binding.SW_EHIP and lat.sweeps_done == 0
    for _ in range(2):
        graph.replay()
    lat.sweep(3)
    torch.cuda.synchronize()
    assert float(x[0]) == 4.0
    assert np.array_equal(lat.measure(0, 3), oracle.OracleLattice(200, 2, K2, 2).run(3))
    lat.close()

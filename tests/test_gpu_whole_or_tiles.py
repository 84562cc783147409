"""Lattices that are swept whole by some calls and by tiles by others (the
default height, L = 97 ... 128): what a call leaves for the next one, bit for bit
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_2080_amd import binding
from paper_1208_2080_amd import workloads as wl

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

Q = 3
K = wl.critical_coupling(Q)


def same_labels(lat, out, when):
    bx, by = lat.bonds()
    assert np.array_equal(bx, oracle.pack_bonds(out["bx"])) and np.array_equal(by, oracle.pack_bonds(out["by"])), when
    assert np.array_equal(lat.labels(), out["labels"]), when


@pytest.mark.parametrize("L", [97, 128])
def test_labels_follow_the_sweeps_that_ran(L):
    """A sweep that the caller captures runs whole when its graph is replayed, not
    when it is recorded, and the calls between go by tiles: the labels read are
    those of the last sweep that ran, and a read does not change the next one."""
    print(f"case L={L}", flush=True)
    stream = torch.cuda.Stream()
    lat = binding.Lattice(L, Q, K, seed=9, obs_capacity=512, stream=stream)
    ref = oracle.OracleLattice(L, Q, K, 9)

    def sweep(n):
        lat.sweep(n)
        for _ in range(n):
            out = ref.sweep()
        return out

    def replay():
        with torch.cuda.stream(stream):
            graph.replay()
        return ref.sweep()

    out = sweep(150)
    same_labels(lat, out, "before the capture")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lat.sweep(1)
    same_labels(lat, out, "recorded, not run")
    same_labels(lat, replay(), "first replay")
    same_labels(lat, replay(), "second replay")
    out = sweep(120)
    same_labels(lat, out, "after the replays")
    out = replay()
    same_labels(lat, out, "replay after a call by tiles")
    same_labels(lat, out, "the same labels again")
    out = sweep(1)
    same_labels(lat, out, "one sweep")
    assert np.array_equal(lat.spins(), ref.s)
    lat.close()


@pytest.mark.parametrize("tile_rows", [0, binding.SW_TILE_WHOLE])
def test_labels_of_a_capture_that_never_ran(tile_rows):
    """No sweep has run since the start (or a load): there are no labels."""
    L = 40
    stream = torch.cuda.Stream()
    lat = binding.Lattice(L, Q, K, seed=4, obs_capacity=8, stream=stream, tile_rows=tile_rows)
    ref = oracle.OracleLattice(L, Q, K, 4)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lat.sweep(1)
    with pytest.raises(binding.SwError) as e:
        lat.labels()
    assert e.value.code == binding.SW_ESTATE
    with torch.cuda.stream(stream):
        graph.replay()
    out = ref.sweep()
    same_labels(lat, out, "after a replay")
    lat.load_spins(ref.s, 1)
    with pytest.raises(binding.SwError) as e:
        lat.labels()
    assert e.value.code == binding.SW_ESTATE
    lat.sweep(1)
    same_labels(lat, ref.sweep(), "after a load")
    lat.close()


def test_labels_after_group_sweeps_and_replays():
    """A group sweeps its lattices by tiles, a captured call of one of them whole."""
    stream = torch.cuda.Stream()
    Ls = [33, 100]
    lats = [binding.Lattice(L, Q, K, seed=L, obs_capacity=64, stream=stream) for L in Ls]
    refs = [oracle.OracleLattice(L, Q, K, L) for L in Ls]
    group = binding.Group(2, sum(binding.tile_count(L, Q) for L in Ls), stream=stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for lat in lats:
            lat.sweep(1)
    for step in range(3):
        group.sweep(lats, [2, 1])
        for lat, ref, n in zip(lats, refs, (2, 1)):
            for _ in range(n):
                out = ref.sweep()
            same_labels(lat, out, f"group, step {step}, L={lat.L}")
        with torch.cuda.stream(stream):
            graph.replay()
        for lat, ref in zip(lats, refs):
            same_labels(lat, ref.sweep(), f"replay, step {step}, L={lat.L}")
    group.close()
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("L", [64, 97, 128, 200])
def test_two_threads_on_one_stream(L):
    """Two threads with a lattice each sweep on one stream in calls of many
    sweeps: no call takes up what the other thread enqueues meanwhile."""
    import threading

    stream = torch.cuda.Stream()
    lats = [binding.Lattice(L, Q, K, seed=s, obs_capacity=8, stream=stream) for s in (1, 2)]
    errors = []
    start = threading.Barrier(2)

    def use(lat):
        try:
            start.wait(60)
            for n in (120, 3, 150, 101, 1):
                lat.sweep(n)
        except BaseException as e:   # reported by the test's thread
            errors.append(e)

    threads = [threading.Thread(target=use, args=(lat,)) for lat in lats]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for lat, seed in zip(lats, (1, 2)):
        ref = oracle.OracleLattice(L, Q, K, seed)
        rows = ref.run(375)
        assert np.array_equal(lat.measure(370, 5), rows[370:]), seed
        assert np.array_equal(lat.spins(), ref.s), seed
        lat.close()


def test_sweeps_while_another_stream_is_captured():
    """A call on one stream, of any number of sweeps, while this thread captures
    another in the strictest mode."""
    for L in (64, 117, 200):
        stream = torch.cuda.Stream()
        lat = binding.Lattice(L, Q, K, seed=3, obs_capacity=8, stream=stream)
        x = torch.zeros(64, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode="global"):
            x += 1
            lat.sweep(150)
            x += 1
        graph.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == 2.0
        ref = oracle.OracleLattice(L, Q, K, 3)
        rows = ref.run(150)
        assert np.array_equal(lat.measure(143, 7), rows[143:])
        assert np.array_equal(lat.spins(), ref.s)
        lat.close()


@pytest.mark.parametrize("L,n,null_stream,by_tiles", [
    (96, 120, False, False), (97, 99, False, False), (97, 100, False, True), (128, 150, False, True),
    (128, 5, False, False), (96, 3, True, False), (97, 3, True, True), (128, 1, True, True)])
def test_profiled_sweeps_take_the_way_of_plain_ones(L, n, null_stream, by_tiles):
    """By tiles every phase has its time; whole, one kernel has it all."""
    stream = torch.cuda.default_stream() if null_stream else torch.cuda.Stream()
    lat = binding.Lattice(L, Q, K, seed=6, obs_capacity=8, stream=stream)
    ms = lat.sweep_profiled(n)
    assert 0 < ms[4] <= ms[0]
    assert (ms[1:4] > 0).all() if by_tiles else (ms[1:4] == 0).all(), ms
    ref = oracle.OracleLattice(L, Q, K, 6)
    for _ in range(n):
        out = ref.sweep()
    assert np.array_equal(lat.spins(), ref.s)
    same_labels(lat, out, "profiled")
    assert np.array_equal(lat.measure(n - 1, 1)[0], out["obs"])
    lat.close()


@pytest.mark.parametrize("L,tile_rows", [(2, 0), (3, 0), (63, 0), (96, 0), (97, 0), (128, 0), (65, binding.SW_TILE_WHOLE)])
def test_labels_read_with_and_without_a_pinned_buffer(L, tile_rows):
    """Labels left by the whole kernel and by tiles, by more readers at once than
    there are buffers."""
    import threading

    stream = torch.cuda.Stream()
    group = binding.Group(6, 6 * binding.tile_count(L, Q), stream=stream)
    lats = [binding.Lattice(L, Q, K, seed=s, obs_capacity=8, stream=stream, tile_rows=tile_rows) for s in range(6)]
    refs = [oracle.OracleLattice(L, Q, K, s) for s in range(6)]
    for n in (1, 120):
        for lat in lats:
            lat.sweep(n)
        outs = []
        for ref in refs:
            for _ in range(n):
                out = ref.sweep()
            outs.append(out["labels"])
        if n == 120:
            group.sweep(lats[:3], [1] * 3)
            outs[:3] = [ref.sweep()["labels"] for ref in refs[:3]]
        got = {}
        threads = [threading.Thread(target=lambda i=i: got.update({i: [lats[i].labels() for _ in range(4)]}))
                   for i in range(6)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for i in range(6):
            assert all(np.array_equal(g, outs[i]) for g in got[i]), (n, i)
    group.close()
    for lat in lats:
        lat.close()

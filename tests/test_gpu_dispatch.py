"""GPU parity at the edges of the rules that pick a kernel: sizes on both sides
of each line, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_2080_amd import binding
from paper_1208_2080_amd import workloads as wl

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)


def check(L, q, K=None, seed=7, calls=(1, 2), tile_rows=0, random_start=True):
    """Sweeps in calls of the given lengths; spins, labels and bonds after each
    call, every row at the end."""
    K = wl.critical_coupling(q) if K is None else K
    print(f"case L={L} q={q} K={K} calls={calls} ty={tile_rows}", flush=True)
    n = sum(calls)
    lat = binding.Lattice(L, q, K, seed=seed, random_start=random_start, obs_capacity=max(2, n), tile_rows=tile_rows)
    ref = oracle.OracleLattice(L, q, K, seed, random_start=random_start)
    rows = []
    for c in calls:
        lat.sweep(c)
        for _ in range(c):
            out = ref.sweep()
            rows.append(out["obs"])
        assert np.array_equal(lat.spins(), ref.s), "spins"
        bx, by = lat.bonds()
        assert np.array_equal(bx, oracle.pack_bonds(out["bx"])), "+x bonds"
        assert np.array_equal(by, oracle.pack_bonds(out["by"])), "+y bonds"
        assert np.array_equal(lat.labels(), out["labels"]), "labels"
    assert np.array_equal(lat.measure(0, n), np.array(rows)), "rows"
    lat.close()


@pytest.mark.parametrize("L", [200, 1024, 1025, 2048, 2049])
def test_waves_per_tile(L):
    """Sixteen, eight or four waves a tile, by the number of tiles: 256 tiles and
    289 (the labelling's line), 1024 and 1089 (the flip's)."""
    check(L, 2)


@pytest.mark.parametrize("L", [200, 1024, 1025])
def test_waves_per_tile_xy(L):
    print(f"case XY L={L}", flush=True)
    lat = binding.XYLattice(L, wl.K_KT_XY, seed=5, obs_capacity=4)
    ref = oracle.XYOracleLattice(L, wl.K_KT_XY, 5)
    for c in (1, 2):
        lat.sweep(c)
        for _ in range(c):
            out = ref.sweep()
        assert np.array_equal(lat.angles(), ref.a)
        assert np.array_equal(lat.labels(), out["labels"])
    lat.close()


@pytest.mark.parametrize("tile_rows", [0, 64])
def test_sweep_counters_of_a_mixed_batch(tile_rows):
    """Replicas swept whole and by tiles advance their own counters over calls
    of sweep_all and sweep, whatever the order."""
    reps = [dict(L=L, q=q, K=wl.critical_coupling(q), seed=50 + i, random_start=True)
            for i, (L, q) in enumerate([(64, 2), (300, 3), (100, 2), (129, 2), (33, 4)])]
    print(f"case mixed batch ty={tile_rows}", flush=True)
    b = binding.Batch(reps, obs_capacity=64, tile_rows=tile_rows)
    b.sweep_all(1)
    b.sweep_all(18)
    each = [3, 0, 5, 2, 1]
    b.sweep(each)
    b.sweep_all(2)
    for r, rep in enumerate(reps):
        ref = oracle.OracleLattice(rep["L"], rep["q"], rep["K"], rep["seed"], random_start=True)
        n = 21 + each[r]
        rows = ref.run(n)
        assert b.sweeps_done(r) == n
        assert np.array_equal(b.measure(r, 0, n), rows), f"rows of replica {r}"
        assert np.array_equal(b.spins(r), ref.s), f"spins of replica {r}"
    b.close()


@pytest.mark.parametrize("L,q", [(2, 2), (16, 3), (17, 2), (48, 2), (49, 8), (63, 9), (64, 17), (65, 2), (113, 4),
                                 (127, 16), (128, 255)])
def test_whole_lattice_strips(L, q):
    """One to eight rows a strip, one and two passes of columns, full and partial
    strips and passes, every way the states are counted; the rows of the first
    sweep of a call, of later ones and of the last."""
    check(L, q, calls=(1, 2, 9), tile_rows=binding.SW_TILE_WHOLE)


@pytest.mark.parametrize("K", [0.0, float("inf")])
@pytest.mark.parametrize("L", [5, 64, 128])
def test_whole_lattice_extreme_couplings(L, K):
    """No bond at all, and one cluster holding every equal bond (the longest
    chains and the fullest queues, from a cold start too)."""
    check(L, 2, K=K, calls=(2, 3), tile_rows=binding.SW_TILE_WHOLE)
    check(L, 2, K=K, calls=(2,), tile_rows=binding.SW_TILE_WHOLE, random_start=False)


@pytest.mark.parametrize("L,reps,tile_rows", [(2, 1, 64), (63, 2, 64), (65, 1, 32), (200, 1, 128), (512, 4, 64),
                                              (513, 4, 64)])
def test_cluster_sums_of_few_and_many_tiles(L, reps, tile_rows):
    """Sums of |C|^2 and |C|^4 with sixteen waves a tile (up to 256 tiles) and
    with four (324), ragged tiles, runs that end at a tile's edge, K = inf (one
    cluster over all tiles: the largest sizes) next to K_c."""
    Ks = [float("inf"), wl.critical_coupling(2), 0.0, 0.8]
    rep = [dict(L=L, q=2, K=Ks[i], seed=3 + i, random_start=i != 0, cluster_sums=True) for i in range(reps)]
    print(f"case cluster sums L={L} reps={reps} ty={tile_rows}", flush=True)
    b = binding.Batch(rep, obs_capacity=8, tile_rows=tile_rows)
    b.sweep_all(3)
    for i, r in enumerate(rep):
        ref = oracle.OracleLattice(L, 2, r["K"], r["seed"], random_start=r["random_start"])
        want = []
        for _ in range(3):
            sizes = np.unique(ref.sweep()["labels"], return_counts=True)[1]
            want.append([sum(int(c) ** 2 for c in sizes), sum(int(c) ** 4 for c in sizes)])
        assert b.cluster_sums(i, 0, 3).tolist() == want, f"replica {i}"
    b.close()


@pytest.mark.parametrize("L,q,tile_rows", [(129, 2, 64), (193, 3, 64), (257, 9, 64), (191, 4, 32), (321, 5, 128),
                                           (1023, 2, 64), (1027, 16, 64), (1153, 2, 64), (130, 2, 32), (192, 13, 128)])
def test_full_and_ragged_strips(L, q, tile_rows):
    """Full strips of odd lattices (pairs that cross rows' starts and tiles'
    edges) and of even ones, ragged tiles beside them, at every tile height and
    number of waves, every way the states are counted."""
    check(L, q, calls=(1, 3), tile_rows=tile_rows)


@pytest.mark.parametrize("K", [0.0, float("inf")])
@pytest.mark.parametrize("L", [128, 193, 1025])
def test_extreme_couplings_by_tiles(L, K):
    check(L, 2, K=K, calls=(2,), tile_rows=64)
    check(L, 3, K=K, calls=(2,), tile_rows=64, random_start=False)


@pytest.mark.parametrize("q", [2, 3, 4, 5, 8, 9, 16, 17, 255])
def test_state_counts_by_subsets(q):
    """The counts of a lattice loaded with every state in known numbers, full and
    partial words at the right edge."""
    for L in (130, 197):
        rng = np.random.default_rng(q)
        spins = rng.choice(q, size=(L, L), p=np.arange(1, q + 1) / (q * (q + 1) / 2)).astype(np.uint8)
        lat = binding.Lattice(L, q, 0.0, seed=1, obs_capacity=8, tile_rows=64)
        ref = oracle.OracleLattice(L, q, 0.0, 1, spins=spins, sweep=5)
        lat.load_spins(spins, 5)
        lat.sweep(3)
        print(f"case counts q={q} L={L}", flush=True)
        assert np.array_equal(lat.measure(5, 3), ref.run(3))
        lat.close()


@pytest.mark.parametrize("K", [0.0, 1e-30, 0.3, 50.0, 1e300, float("inf")])
@pytest.mark.parametrize("L", [65, 130])
def test_xy_bond_estimates(L, K):
    """Bonds of the XY sweep over the whole range of couplings (the estimates
    under- and overflow at its ends): bonds, labels and angles as the oracle's."""
    print(f"case XY L={L} K={K}", flush=True)
    for start in (True, False):
        lat = binding.XYLattice(L, K, seed=21, random_start=start, obs_capacity=4)
        ref = oracle.XYOracleLattice(L, K, 21, random_start=start)
        for _ in range(3):
            lat.sweep(1)
            out = ref.sweep()
            bx, by = lat.bonds()
            assert np.array_equal(bx, oracle.pack_bonds(out["bx"]))
            assert np.array_equal(by, oracle.pack_bonds(out["by"]))
            assert np.array_equal(lat.labels(), out["labels"])
            assert np.array_equal(lat.angles(), ref.a)
        lat.close()


@pytest.mark.parametrize("Ls", [[64] * 3, [128, 17], [64, 200], [2, 3, 500, 128]])
def test_batches_of_small_lattices(Ls):
    """Lattices that fit LDS alone (swept whole) and beside one that does not
    (swept by tiles with it, or whole in a call that sweeps only them or sweeps
    them further), with calls of both kinds in turn."""
    reps = [dict(L=L, q=2 + i, K=wl.critical_coupling(2 + i), seed=80 + i, random_start=True) for i, L in enumerate(Ls)]
    print(f"case small batch {Ls}", flush=True)
    b = binding.Batch(reps, obs_capacity=64)
    counts = np.zeros(len(Ls), dtype=int)
    small = [2 if L <= 128 else 0 for L in Ls]
    more = [6 if L <= 128 else 3 for L in Ls]
    fewer = [1 if L <= 128 else 4 for L in Ls]
    for each in (None, small, more, fewer, None, small, None):
        if each is None:
            b.sweep_all(2)
            each = [2] * len(Ls)
        else:
            b.sweep(each)
        counts += each
    for r, rep in enumerate(reps):
        ref = oracle.OracleLattice(rep["L"], rep["q"], rep["K"], rep["seed"], random_start=True)
        rows = ref.run(int(counts[r]))
        assert np.array_equal(b.measure(r, 0, int(counts[r])), rows), f"rows of replica {r}"
        assert np.array_equal(b.spins(r), ref.s), f"spins of replica {r}"
    b.close()


def test_reads_small_and_large_from_several_threads():
    """Reads that fit a pinned buffer and reads that do not, more readers at once
    than there are buffers, and after every handle (and buffer) was given back."""
    import threading

    def use(i, L, n, errors):
        try:
            lat = binding.Lattice(L, 2, 0.88, seed=i, obs_capacity=n + 1, stream=torch.cuda.Stream())
            ref = oracle.OracleLattice(L, 2, 0.88, i)
            rows = ref.run(n)
            for _ in range(3):
                if lat.sweeps_done == 0:
                    lat.sweep(n)
                assert np.array_equal(lat.measure(0, n), rows)
                assert np.array_equal(lat.measure(n // 2, 1), rows[n // 2:n // 2 + 1])
                assert lat.measure(0, 0).shape == (0, 4)
                assert np.array_equal(lat.spins(), ref.s)
            lat.close()
        except BaseException as e:   # reported by the test's thread
            errors.append((L, n, e))

    for _ in range(2):
        errors = []
        jobs = [(1, 7, 3), (2, 33, 5), (3, 362, 2), (4, 363, 2), (5, 400, 2), (6, 16, 2800), (7, 9, 40)]
        threads = [threading.Thread(target=use, args=(*j, errors)) for j in jobs]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors


@pytest.mark.parametrize("L,q,f,tile_rows,random_start", [
    (1472, 2, 1.0, 0, True), (1473, 2, 1.0, 0, True), (1600, 2, 1.1, 0, False), (1537, 4, 1.05, 0, True),
    (1056, 3, 1.0, 32, True), (1088, 3, 1.0, 32, True), (2944, 2, 1.05, 128, False), (3200, 2, 1.0, 0, True)])
def test_merges_that_climb_both_chains(L, q, f, tile_rows, random_start):
    """Tile counts on both sides of the lower line (529 and 576, 561 and 578),
    from random and from ordered starts."""
    check(L, q, K=f * wl.critical_coupling(q), tile_rows=tile_rows, calls=(1, 3), random_start=random_start)


@pytest.mark.parametrize("L", [10240, 10241])
def test_merges_agree_across_the_upper_line(L):
    """The same sweeps with 64-row tiles (25600 of them at L = 10240, the line)
    and with 32-row tiles, twice as many."""
    print(f"case L={L}", flush=True)
    got = []
    for ty in (64, 32):
        lat = binding.Lattice(L, 2, wl.critical_coupling(2), seed=3, obs_capacity=16, tile_rows=ty)
        lat.sweep(8)
        got.append((lat.measure(0, 8), lat.spins()))
        lat.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("L,K,tile_rows,calls", [(2112, 0.0, 64, (1, 1)), (2112, float("inf"), 64, (2,)),
                                                 (2100, None, 0, (1, 2)), (1090, None, 32, (3,))])
def test_cluster_sums_by_four_waves(L, K, tile_rows, calls):
    """The flip's own cluster sums above 1024 tiles (four waves a tile): sites
    alone, one cluster over all tiles, K_c with ragged tiles; the sums of every
    sweep whether it is the last of a call or not."""
    print(f"case cluster sums L={L} K={K} ty={tile_rows} calls={calls}", flush=True)
    K = wl.critical_coupling(2) if K is None else K
    ref = oracle.OracleLattice(L, 2, K, 11, random_start=False)
    b = binding.Batch([dict(L=L, q=2, K=K, seed=11, random_start=False, cluster_sums=True)], obs_capacity=8,
                      tile_rows=tile_rows)
    want = []
    for n in calls:
        b.sweep_all(n)
        for _ in range(n):
            sizes = np.unique(ref.sweep()["labels"], return_counts=True)[1]
            want.append([sum(int(c) ** 2 for c in sizes), sum(int(c) ** 4 for c in sizes)])
    assert b.cluster_sums(0, 0, sum(calls)).tolist() == want
    b.close()


@pytest.mark.parametrize("L,f", [(704, 1.0), (705, 1.0), (705, 0.99), (640, 1.1), (1001, 1.1)])
def test_merges_of_spanning_clusters(L, f):
    """Both sides of the lower line (121 and 144 tiles) and of the coupling."""
    check(L, 3, K=f * wl.critical_coupling(3), calls=(2, 2), random_start=f <= 1.0)


@pytest.mark.parametrize("L,K", [(705, 1.03), (705, 1.05), (1001, 2.0), (1500, float("inf"))])
def test_merges_of_spanning_clusters_xy(L, K):
    print(f"case XY L={L} K={K}", flush=True)
    cold = K > 1.5
    lat = binding.XYLattice(L, K, seed=5, random_start=not cold, obs_capacity=4)
    ref = oracle.XYOracleLattice(L, K, 5, random_start=not cold)
    for c in (1, 2):
        lat.sweep(c)
        for _ in range(c):
            out = ref.sweep()
        assert np.array_equal(lat.angles(), ref.a)
        assert np.array_equal(lat.labels(), out["labels"])
    lat.close()


@pytest.mark.parametrize("L", [96, 97, 117, 128])
@pytest.mark.parametrize("null_stream", [False, True])
def test_lattices_that_fit_lds_whole_or_by_tiles(L, null_stream):
    """Both sides of the line for plain lattices (L = 96) and of the number of
    sweeps from which the captured steps are made (100): calls of one lattice go
    from the whole kernel to the tiles, and a call that the caller captures goes
    back to one launch."""
    q, K = 3, wl.critical_coupling(3)
    print(f"case L={L} null_stream={null_stream}", flush=True)
    stream = torch.cuda.default_stream() if null_stream else torch.cuda.Stream()
    lat = binding.Lattice(L, q, K, seed=5, obs_capacity=256, stream=stream)
    ref = oracle.OracleLattice(L, q, K, 5)
    rows = []
    for n in (1, 99, 100, 1, 3):
        lat.sweep(n)
        for _ in range(n):
            out = ref.sweep()
            rows.append(out["obs"])
        assert np.array_equal(lat.spins(), ref.s), f"spins after {n}"
        assert np.array_equal(lat.labels(), out["labels"]), f"labels after {n}"
        bx, by = lat.bonds()
        assert np.array_equal(bx, oracle.pack_bonds(out["bx"])) and np.array_equal(by, oracle.pack_bonds(out["by"]))
    assert np.array_equal(lat.measure(0, 204), np.array(rows))
    if not null_stream:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            lat.sweep(1)
        for _ in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
            ref.sweep()
            assert np.array_equal(lat.spins(), ref.s), "spins after a replay"
    lat.close()


def sums_of(labels):
    sizes = np.unique(labels, return_counts=True)[1]
    return [sum(int(c) ** 2 for c in sizes), sum(int(c) ** 4 for c in sizes)]


# (L, q, with cluster sums): large and small lattices, with the sums and without
MIXED = [(200, 2, True), (200, 2, False), (64, 3, False), (97, 2, True), (300, 4, False), (33, 2, True)]


def test_batch_with_cluster_sums_in_some_replicas():
    """One flip for all of them: those without the sums leave it early."""
    reps = [dict(L=L, q=q, K=wl.critical_coupling(q), seed=20 + i, random_start=True, cluster_sums=cs)
            for i, (L, q, cs) in enumerate(MIXED)]
    print("case mixed cluster sums, batch", flush=True)
    b = binding.Batch(reps, obs_capacity=16)
    b.sweep_all(2)
    b.sweep([i % 3 for i in range(len(reps))])
    b.sweep_all(1)
    for i, r in enumerate(reps):
        n = 3 + i % 3
        ref = oracle.OracleLattice(r["L"], r["q"], r["K"], r["seed"], random_start=True)
        outs = [ref.sweep() for _ in range(n)]
        assert np.array_equal(b.measure(i, 0, n), np.array([o["obs"] for o in outs])), i
        assert np.array_equal(b.spins(i), ref.s), i
        if r["cluster_sums"]:
            assert b.cluster_sums(i, 0, n).tolist() == [sums_of(o["labels"]) for o in outs], i
        else:
            with pytest.raises(binding.SwError):
                b.cluster_sums(i, 0, n)
    b.close()


def test_group_with_cluster_sums_in_some_lattices():
    print("case mixed cluster sums, group", flush=True)
    lats = [binding.Lattice(L, q, wl.critical_coupling(q), seed=20 + i, obs_capacity=16, cluster_sums=cs)
            for i, (L, q, cs) in enumerate(MIXED)]
    refs = [oracle.OracleLattice(L, q, wl.critical_coupling(q), 20 + i) for i, (L, q, cs) in enumerate(MIXED)]
    group = binding.Group(len(lats), sum(binding.tile_count(L, q) for L, q, _ in MIXED))
    outs = [[] for _ in lats]
    for each in ([2] * 6, [0, 1, 1, 3, 1, 2], [1, 0, 2, 0, 1, 1]):
        group.sweep(lats, each)
        for i, n in enumerate(each):
            outs[i] += [refs[i].sweep() for _ in range(n)]
    for i, (lat, (L, q, cs)) in enumerate(zip(lats, MIXED)):
        n = len(outs[i])
        assert np.array_equal(lat.measure(0, n), np.array([o["obs"] for o in outs[i]])), i
        assert np.array_equal(lat.spins(), refs[i].s) and np.array_equal(lat.labels(), outs[i][-1]["labels"]), i
        if cs:
            assert lat.cluster_sums(0, n).tolist() == [sums_of(o["labels"]) for o in outs[i]], i
    group.close()
    for lat in lats:
        lat.close()


# launch_merge picks the hooks that climb both chains from 144 tiles on (and up to
# 25600, at a coupling where clusters span the lattice); the flip takes sixteen
# waves a tile up to 256 tiles, eight up to 1024, four above.
@pytest.mark.parametrize("L,tile_rows,tiles", [(512, 32, 128), (513, 32, 153), (1024, 128, 128), (1025, 128, 153),
                                               (704, 64, 121), (705, 64, 144)])
def test_lower_line_of_the_two_chain_merge(L, tile_rows, tiles):
    """Both sides of 144 tiles at every tile height."""
    assert binding.tile_count(L, 2, tile_rows) == tiles
    for f in (1.0, 1.3):
        check(L, 2, K=f * wl.critical_coupling(2), tile_rows=tile_rows, calls=(1, 2), random_start=f == 1.0)


@pytest.mark.parametrize("K", [2.19, 2.2, 3.0])
def test_merges_far_above_the_transition(K):
    """Both sides of K = 2.2, from where the hooks climb one chain again."""
    check(900, 3, K=K, calls=(2, 2))
    check(900, 3, K=K, calls=(2,), random_start=False)

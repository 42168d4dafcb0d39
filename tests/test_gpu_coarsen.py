"""gosh_coarsen_device (Alg. 4 on the GPU: degree sort, marking rounds, CSR rebuild) against
the oracle and against gosh_coarsen: the hierarchy is unique, so everything is compared
bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

import graphgen
import paper_2008_12336_amd as G
from oracle import gosh_oracle as O
from tests.test_coarsen import _ring_lattice, assert_same_hierarchy
from tests.util import (DENY_NARROW, DENY_RADIX, DENY_STAGING, DENY_TABLE, SEAM_DENY, SEAM_RADIX_FROM, SEAM_WEIGHT_BITS,
                        SEAM_WIDE_SUMS, csr_from_pairs, seam)

pytestmark = pytest.mark.gpu


def device_hierarchy(n, xadj, adj, offsets64, **kw):
    xt = torch.from_numpy(np.asarray(xadj, dtype=np.int64 if offsets64 else np.int32))
    at = torch.from_numpy(np.asarray(adj, dtype=np.int32))
    return G.gosh_coarsen_device(n, xt, at, **kw)


CASES = {
    "er1024": lambda: (1024, graphgen.er_gnm(1024, 8192, 1)),
    "rmat4096": lambda: (4096, graphgen.rmat(12, 1 << 15, 2)),
    "cl5000": lambda: (5000, graphgen.chung_lu(5000, 40000, 3)),
    "rmat65536": lambda: (1 << 16, graphgen.rmat(16, 1 << 19, 5)),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("offsets64", [False, True])
def test_device_hierarchy_matches_oracle(name, offsets64):
    n, edges = CASES[name]()
    c = graphgen.to_csr(n, edges)
    xadj, adj = c.xadj.numpy(), c.adj.numpy()
    for kw in (dict(threshold=100, min_shrink=1.0), dict(threshold=50, min_shrink=0.8),
               dict(threshold=10, min_shrink=1.0, max_levels=3)):
        graphs, maps, mults = O.coarsen(xadj, adj, **kw)
        h = device_hierarchy(n, xadj, adj, offsets64, **kw)
        assert_same_hierarchy(h, graphs, maps, mults)
        assert h.levels >= 2
        h.free()


def test_device_tiny_and_degenerate():
    rng = np.random.default_rng(11)
    for n in (2, 3, 7, 33, 64, 65):
        for m in (0, 1, n, 4 * n):
            pairs = [(int(a), int(b)) for a, b in rng.integers(0, n, size=(m, 2))]
            xadj, adj = csr_from_pairs(n, pairs)
            graphs, maps, mults = O.coarsen(xadj, adj, threshold=1, min_shrink=1.0)
            h = device_hierarchy(n, xadj, adj, False, threshold=1, min_shrink=1.0)
            assert_same_hierarchy(h, graphs, maps, mults)
            h.free()
    # a clique collapses into one vertex: every entry falls inside the cluster
    pairs = [(i, j) for i in range(6) for j in range(i)]
    xadj, adj = csr_from_pairs(6, pairs)
    h = device_hierarchy(6, xadj, adj, True, threshold=1)
    n1, x1, a1 = h.graph(1)
    assert n1 == 1 and a1.size == 0 and list(x1) == [0, 0]
    h.free()


def test_device_large_matches_host():
    # 2^20 vertices, hub rows far longer than a wavefront: beyond what the oracle does fast
    n = 1 << 20
    c = graphgen.to_csr(n, graphgen.chung_lu(n, 1 << 23, 4), offsets64=True)
    hh = G.gosh_coarsen(n, c.xadj, c.adj, threshold=100, min_shrink=0.8)
    hd = G.gosh_coarsen_device(n, c.xadj, c.adj, threshold=100, min_shrink=0.8)
    assert hh.levels == hd.levels
    for i in range(hh.levels):
        nh, xh, ah = hh.graph(i)
        nd, xd, ad = hd.graph(i)
        assert nh == nd and np.array_equal(xh, xd) and np.array_equal(ah, ad)
        if i > 0:
            assert np.array_equal(hh.mult(i), hd.mult(i))
            assert int(hd.mult(i).sum()) <= c.adj.numel()
        if i + 1 < hh.levels:
            assert np.array_equal(hh.map(i), hd.map(i))
    hh.free()
    hd.free()


@pytest.mark.parametrize("name", ["path", "ring3", "uniform", "mixed"])
def test_device_marking_with_long_dependency_chains(name):
    """Graphs whose marking is one long chain (the rounds stall and the host sweep takes
    over) or many short ones (resolved by the rounds) still give the sequential result."""
    if name == "path":
        n = 30000
        xadj, adj = csr_from_pairs(n, [(i, i + 1) for i in range(n - 1)])
    elif name == "ring3":
        n = 20000
        xadj, adj = _ring_lattice(n, 3)
    elif name == "uniform":
        n = 60000
        c = graphgen.to_csr(n, graphgen.er_gnm(n, 4 * n, 11))
        xadj, adj = c.xadj.numpy(), c.adj.numpy()
    else:
        n = 50000
        path = [(i, i + 1) for i in range(30000)]
        c = graphgen.chung_lu(n, 120000, 12)
        xadj, adj = csr_from_pairs(n, path + [tuple(e) for e in c.tolist()])
    graphs, maps, mults = O.coarsen(xadj, adj, threshold=n // 2, min_shrink=1.0, max_levels=2)
    h = device_hierarchy(n, xadj, adj, False, threshold=n // 2, min_shrink=1.0, max_levels=2)
    assert_same_hierarchy(h, graphs, maps, mults)
    h.free()


def test_device_isolated_vertices_and_no_progress():
    # only isolated vertices: nothing merges, the hierarchy keeps the one level and no map
    xadj, adj = csr_from_pairs(10, [])
    h = device_hierarchy(10, xadj, adj, False, threshold=1)
    assert h.levels == 1
    h.free()
    # a star plus isolated vertices: one merge level, then no progress
    xadj, adj = csr_from_pairs(12, [(0, i) for i in range(1, 6)])
    graphs, maps, mults = O.coarsen(xadj, adj, threshold=1, min_shrink=1.0)
    h = device_hierarchy(12, xadj, adj, True, threshold=1, min_shrink=1.0)
    assert_same_hierarchy(h, graphs, maps, mults)
    h.free()


def test_release_device_keeps_everything_readable():
    n = 4096
    c = graphgen.to_csr(n, graphgen.rmat(12, 1 << 15, 2))
    xadj, adj = c.xadj.numpy(), c.adj.numpy()
    graphs, maps, mults = O.coarsen(xadj, adj, threshold=100, min_shrink=1.0)
    h = G.gosh_coarsen_device(n, c.xadj, c.adj, threshold=100, min_shrink=1.0)
    h.trim_scratch()  # the levels stay on the device
    h.trim_scratch()
    assert np.array_equal(h.map(0), maps[0])
    h.release_device()
    assert_same_hierarchy(h, graphs, maps, mults)
    # training from the released (host) copies still works and agrees with the oracle's shapes
    M0 = torch.zeros(n, 16, dtype=torch.float32, device="cuda:0")
    stats = G.gosh_embed(h, M0, 3, 12, 0.3, 0.05, 1, flags=G.GOSH_FLAG_SEQUENTIAL)
    torch.cuda.synchronize()
    assert [s["n"] for s in stats] == [g[0].size - 1 for g in graphs]
    assert bool(torch.isfinite(M0).all())
    h.release_device()  # idempotent
    h.free()


def test_device_rejects_malformed_graphs():
    xadj, adj = csr_from_pairs(300, [(i, i + 1) for i in range(299)])
    bad_adj = adj.copy()
    bad_adj[7] = 300  # neighbour id out of range
    with pytest.raises(G.GoshError, match="neighbour"):
        device_hierarchy(300, xadj, bad_adj, False, threshold=10)
    bad_x = xadj.copy()
    bad_x[5] = bad_x[6] + 1  # offsets decrease
    with pytest.raises(G.GoshError, match="xadj"):
        device_hierarchy(300, bad_x, adj, False, threshold=10)
    # the device is still usable afterwards
    h = device_hierarchy(300, xadj, adj, False, threshold=10)
    assert h.levels >= 2
    h.free()


def test_entries_are_not_read_where_the_offsets_are_wrong():
    """A device-resident graph whose nnz is more than its offsets end at, by far more than the memory there is:
    refused for its offsets, before anybody looks at so many entries."""
    xadj, adj = csr_from_pairs(300, [(i, i + 1) for i in range(299)])
    xd, ad = torch.from_numpy(xadj).to("cuda:0"), torch.from_numpy(adj).to("cuda:0")
    for nnz in (adj.size + 1, 1 << 36):
        g, out = G.csr_view(300, xd, ad), C.c_void_p()
        g.nnz = nnz
        assert G.lib().gosh_coarsen_device(C.byref(g), 10, 1.0, 64, 0, C.byref(out)) == -1
        assert "xadj" in G.gosh_last_error() and not out.value
    G.gosh_coarsen_device(300, xd, ad, threshold=10).free()


@pytest.mark.parametrize("offsets64", [False, True])
def test_device_resident_input_graph(offsets64):
    """G_0 given as device tensors is used in place (no upload), gives the same hierarchy,
    and its host copy appears on request."""
    n = 4096
    c = graphgen.to_csr(n, graphgen.rmat(12, 1 << 15, 2), offsets64=offsets64)
    xadj, adj = c.xadj.numpy(), c.adj.numpy()
    graphs, maps, mults = O.coarsen(xadj, adj, threshold=100, min_shrink=0.8)
    xd, ad = c.xadj.to("cuda:0"), c.adj.to("cuda:0")
    h = G.gosh_coarsen_device(n, xd, ad, threshold=100, min_shrink=0.8)
    # train first (nothing has been downloaded yet), then read everything back
    want, _, _, _ = O.embed(xadj, adj, 16, 3, 12, 0.3, 0.05, 4, threshold=100, min_shrink=0.8)
    M0 = torch.zeros(n, 16, dtype=torch.float32, device="cuda:0")
    assert h.shape(0) == (n, adj.size) and h.shape(1)[0] == graphs[1][0].size - 1
    stats = G.gosh_embed(h, M0, 3, 12, 0.3, 0.05, 4, flags=G.GOSH_FLAG_SEQUENTIAL)
    torch.cuda.synchronize()
    assert all(s["upload_ms"] < 5.0 for s in stats)
    err = np.abs(M0.cpu().numpy() - want).max() / np.abs(want).max()
    assert err <= 1e-5
    assert_same_hierarchy(h, graphs, maps, mults)
    n0, x0, a0 = h.graph(0)
    assert x0.dtype == (np.int64 if offsets64 else np.int32)
    h.release_device()  # the caller's device tensors stay the caller's
    assert_same_hierarchy(h, graphs, maps, mults)
    h.free()
    assert torch.equal(xd.cpu(), c.xadj) and torch.equal(ad.cpu(), c.adj)
    with pytest.raises(TypeError):
        G.gosh_coarsen_device(n, xd, c.adj, threshold=100)
    with pytest.raises(TypeError):
        G.gosh_coarsen(n, xd, ad, threshold=100)
    # the C entry points that read the graph on the host refuse device memory themselves
    gd = G.csr_view(n, xd, ad)
    out = C.c_void_p()
    assert G.lib().gosh_coarsen(C.byref(gd), 100, 1.0, 64, 0, C.byref(out)) == -1
    assert "host graph" in G.gosh_last_error()
    assert G.lib().gosh_csr_validate(C.byref(gd)) == -1


from hypothesis import given, settings, strategies as st  # noqa: E402

_graphs = st.integers(min_value=2, max_value=90).flatmap(
    lambda n: st.tuples(st.just(n), st.lists(
        st.tuples(st.integers(0, n - 1), st.integers(0, n - 1)), min_size=0, max_size=6 * n)))


@settings(max_examples=60, deadline=None)
@given(_graphs, st.booleans())
def test_device_random_tiny_graphs_match_oracle(g, offsets64):
    n, pairs = g
    xadj, adj = csr_from_pairs(n, pairs)
    graphs, maps, mults = O.coarsen(xadj, adj, threshold=1, min_shrink=1.0)
    h = device_hierarchy(n, xadj, adj, offsets64, threshold=1, min_shrink=1.0)
    assert_same_hierarchy(h, graphs, maps, mults)
    h.free()


def hub_graph(hubs, edges_of, seed):
    """Hubs with leaves of degree one and two: a leaf joins its hub, and a leaf of two hubs
    leaves an entry between them, so coarse row a merges about edges_of[a] + leaves entries."""
    rng = np.random.default_rng(seed)
    pairs, nxt = set(), hubs
    for a, e in enumerate(edges_of):
        pairs |= {(min(a, int(b)), max(a, int(b))) for b in rng.integers(0, hubs, e) if b != a}
        for _ in range(12):
            pairs.add((a, nxt))
            if rng.random() < 0.7:
                pairs.add((int(rng.integers(0, hubs)), nxt))
            nxt += 1
    return graphgen.to_csr(nxt, torch.tensor(sorted(pairs), dtype=torch.int64))


def assert_equals_host(csr, levels=None, **kw):
    n = csr.xadj.numel() - 1
    h = G.gosh_coarsen_device(n, csr.xadj, csr.adj, **kw)
    ref = G.gosh_coarsen(n, csr.xadj, csr.adj, **kw)
    assert h.levels == ref.levels >= (levels or 2)
    for i in range(h.levels):
        if i + 1 < h.levels:
            assert np.array_equal(h.map(i), ref.map(i))
        for got, want in zip(h.graph(i), ref.graph(i)):
            assert np.array_equal(got, want)
        if i:
            assert np.array_equal(h.mult(i), ref.mult(i))
    h.free()


@pytest.mark.parametrize("wide_sums", [0, 1])
@pytest.mark.parametrize("lengths", [range(20, 44), [*range(140, 250, 2), 1024], [2000, 2040, 2100, 9000, 17000, 40000]])
def test_coarse_rows_of_every_way_of_merging(lengths, wide_sums):
    """Rows that a wavefront sorts (among few columns those of up to 512 entries, of up to 2,400 among
    120,000), then bitmaps, from 32,768 on counters, level by level with growing multiplicities, against
    gosh_coarsen."""
    lengths = list(lengths)
    hubs = max(64, 3 * max(lengths))
    edges = [lengths[a] if a < len(lengths) else 3 for a in range(hubs)]
    with seam(SEAM_WIDE_SUMS, wide_sums):
        assert_equals_host(hub_graph(hubs, edges, 5), 3, threshold=4, min_shrink=1.0)


def test_blocks_of_freed_hierarchies_are_reused_bounded_and_given_back():
    n = 1 << 18
    csr = graphgen.to_csr(n, graphgen.rmat(18, 1 << 22, 7)).to("cuda:0")
    run = lambda: G.gosh_coarsen_device(n, csr.xadj, csr.adj, threshold=500, min_shrink=0.9)
    free_bytes = lambda: torch.cuda.mem_get_info()[0]
    h = run()
    h.trim_scratch()
    h.free()
    trim = lambda: G.lib().gosh_hierarchy_trim_scratch(None)
    assert trim() == 0
    slack = 16 << 20
    start, total = torch.cuda.mem_get_info()
    run().free()
    kept = start - free_bytes()
    assert 0 < kept <= total // 64 + slack
    for _ in range(3):
        run().free()
    assert abs(start - free_bytes() - kept) <= slack  # the same blocks again
    assert trim() == 0
    assert start - free_bytes() <= slack


def test_hierarchies_built_and_freed_by_two_threads():
    import threading

    graphs = [graphgen.to_csr(1 << 15, graphgen.rmat(15, 1 << 18, s)) for s in (1, 2)]
    refs = [G.gosh_coarsen(1 << 15, c.xadj, c.adj, threshold=50, min_shrink=0.9) for c in graphs]
    failures = []

    def work(c, ref):
        try:
            for _ in range(6):
                h = G.gosh_coarsen_device(1 << 15, c.xadj, c.adj, threshold=50, min_shrink=0.9)
                assert h.levels == ref.levels
                for i in range(h.levels - 1):
                    assert np.array_equal(h.map(i), ref.map(i))
                    assert np.array_equal(h.mult(i + 1), ref.mult(i + 1))
                h.free()
        except BaseException as e:
            failures.append(e)

    threads = [threading.Thread(target=work, args=a) for a in zip(graphs, refs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures


def test_coarsening_without_pinned_staging():
    """Copies between pageable memory and the device go through pinned slots only because that is
    faster: a graph of 11 MB and a map of 5 MB move without them too."""
    n = 1_250_000
    csr = graphgen.to_csr(n, graphgen.er_gnm(n, 1_400_000, 3))
    ref = G.gosh_coarsen(n, csr.xadj, csr.adj, threshold=1000, min_shrink=0.9, max_levels=2)
    with seam(SEAM_DENY, DENY_STAGING):
        h = G.gosh_coarsen_device(n, csr.xadj, csr.adj, threshold=1000, min_shrink=0.9, max_levels=2)
        assert np.array_equal(h.map(0), ref.map(0))
        for got, want in zip(h.graph(1), ref.graph(1)):
            assert np.array_equal(got, want)
    h.free()


def test_matrix_placement_counts_kept_blocks_as_free():
    """gosh_matrix_place asks how much memory is free: blocks kept from freed hierarchies are."""
    n = 1 << 18
    csr = graphgen.to_csr(n, graphgen.rmat(18, 1 << 22, 7)).to("cuda:0")
    kept = G.lib()._ZN4gosh10block_keptEv
    kept.restype, kept.argtypes = C.c_size_t, []
    G.gosh_coarsen_device(n, csr.xadj, csr.adj, threshold=500, min_shrink=0.9).free()
    assert kept() > 0
    with pytest.raises(G.GoshError, match="no room for an arena"):
        G.gosh_matrix_place((1 << 31) - 2, 512)
    assert kept() == 0


def wide_graph(hubs, lengths, seed):
    """hub_graph for many hubs: the rows of the first ones reach over all of them."""
    rng = np.random.default_rng(seed)
    leaves = hubs + np.arange(3 * hubs)
    second = leaves[rng.random(3 * hubs) < 0.7]
    u = np.concatenate((np.repeat(np.arange(len(lengths)), lengths), np.arange(hubs), np.repeat(np.arange(hubs), 3),
                        rng.integers(0, hubs, second.size)))
    v = np.concatenate((rng.integers(0, hubs, sum(lengths)), (np.arange(hubs) + 1) % hubs, leaves, second))
    n = 4 * hubs
    key = np.unique((np.minimum(u, v) * n + np.maximum(u, v))[u != v])
    return graphgen.to_csr(n, torch.from_numpy(np.stack((key // n, key % n), 1)))


@pytest.fixture(scope="module")
def long_rows():
    """300,000 columns, two pieces of 2^18, and rows on both sides of their border; the longest
    coarse row has 226,000 entries, four slices of 2^16."""
    return wide_graph(300_000, [2040, 2060, 9000, 36000, 39000, 70000, 200_000, 420_000], 5)


# SEAM_RADIX_FROM, SEAM_DENY
WAYS = {"ranked and counted": (0, 0), "by radix": (1, 0), "no memory to sort": (1, DENY_RADIX),
        "no memory to count": (0, DENY_TABLE)}


@pytest.mark.parametrize("wide_sums", [0, 1])
@pytest.mark.parametrize("way", sorted(WAYS))
def test_long_rows_over_several_pieces(long_rows, way, wide_sums):
    """Every way of merging long rows, with 32-bit sums and with the 64-bit ones of graphs of 2^32
    entries and more (other LDS sizes, exchanges and atomics)."""
    with seam(SEAM_RADIX_FROM, WAYS[way][0]), seam(SEAM_DENY, WAYS[way][1]), seam(SEAM_WIDE_SUMS, wide_sums):
        assert_equals_host(long_rows, 4, threshold=4, min_shrink=1.0)


def test_rebuild_of_wide_graphs_costs_no_more_than_sorting_their_entries():
    """Twenty vertices of four million neighbours among seven million coarse ones: reading their rows
    once per range of columns took three times a sort of all entries."""
    n, dev = 32_000_000, "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    draw = lambda hi, m: torch.randint(0, hi, (m,), generator=g, device=dev)
    u, v = torch.cat((draw(20, 80_000_000), draw(n, 64_000_000))), draw(n, 144_000_000)
    u, v = u[u != v], v[u != v]
    key = torch.unique(torch.cat((u * n + v, v * n + u)))
    del u, v
    adj = (key % n).to(torch.int32)
    xadj = torch.searchsorted(key, torch.arange(n + 1, device=dev) * n)
    key = key[torch.randperm(key.numel(), generator=g, device=dev, dtype=torch.int64)]
    sort_ms = []
    for _ in range(2):  # the first one also gets its memory
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        torch.sort(key)
        b.record()
        torch.cuda.synchronize()
        sort_ms.append(a.elapsed_time(b))
    del key
    torch.cuda.empty_cache()
    build_ms = []
    for _ in range(2):
        h = G.gosh_coarsen_device(n, xadj, adj, threshold=10_000, min_shrink=0.8, max_levels=2)
        assert h.shape(1)[0] > 6_000_000
        build_ms.append(h.times(0)["build_ms"])
        h.free()
    print(f"[wide] rebuild {min(build_ms):.1f} ms, sort of its {adj.numel()} entries {min(sort_ms):.1f} ms")
    assert min(build_ms) <= 1.25 * min(sort_ms)


@pytest.mark.parametrize("n,per_vertex", [(8191, 3), (8192, 3), (8195, 600), (65_535, 2), (65_541, 4), (65_536, 300),
                                          ((1 << 20) - 1, 2), ((1 << 20) + 3, 3)])
def test_marking_with_few_lanes_per_vertex(n, per_vertex):
    """The marking kernels give a vertex 4, 8, 16 or 64 lanes by the vertices of a level, more where its
    rows are long: both sides of each border, vertices that do not fill the last wavefront, rows
    of many turns."""
    edges = graphgen.chung_lu(n, per_vertex * n, 11)
    assert_equals_host(graphgen.to_csr(n, edges), threshold=500, min_shrink=0.9)


@pytest.mark.parametrize("weight_bits,wide_sums,radix_from", [(1, 0, 0), (3, 0, 0), (3, 1, 0), (2, 0, 1)])
@pytest.mark.parametrize("lengths", [[*range(120, 140), *range(1000, 1040, 3)], [2040, 2050, 4090, 4100, 9000, 40000]])
def test_weights_beside_and_apart_from_their_columns(lengths, weight_bits, wide_sums, radix_from):
    """Multiplicities that fit the bits a column leaves, and such as do not, up to none: the seam takes the
    bits away that graphs of 2^28 clusters lack.  Rows of the sorting networks (up to 512 entries, and 2,048),
    of the bitmap, the counters and the radix sort."""
    hubs = max(64, 3 * max(lengths))
    edges = [lengths[a] if a < len(lengths) else 3 for a in range(hubs)]
    with seam(SEAM_WIDE_SUMS, wide_sums), seam(SEAM_WEIGHT_BITS, weight_bits), seam(SEAM_RADIX_FROM, radix_from):
        assert_equals_host(hub_graph(hubs, edges, 5), 3, threshold=4, min_shrink=1.0)


NETWORKS = [16, 32, 64, 128, 256, 512, 1024, 2048, 4096]  # the longest row of each sorting network


@pytest.fixture(scope="module")
def bordered():
    """Rows of the lengths around every network's longest, at both levels of a rebuild, without weights and
    with: 240,000 hubs in a ring, each with a leaf, and vertices tied to some of them, all of which are centres
    of stars of three in the finest graph.  So many columns leave even rows of 4,096 entries to the networks."""
    hubs, rng = 240_000, np.random.default_rng(5)
    wanted = [(level, b + o) for b in NETWORKS for o in (-1, 0, 1) for level in (0, 1)]
    apart = iter(np.split(rng.permutation(hubs), np.cumsum([w for _, w in wanted])))
    hub = len(wanted) + np.arange(hubs)
    n1 = len(wanted) + 2 * hubs
    ends, twice_ends = [(hub, hub + hubs), (hub, np.roll(hub, 1)), (hub, np.roll(hub, 2))], []
    for s, (level, w) in enumerate(wanted):
        twice = max(1, w // 16)  # entries that name a column once more
        x = w - 3 * twice if level else w - 6 - 3 * twice
        to, me = hub[next(apart)[:x]], np.full(x, s)
        ends.append((me, to))
        if level:  # through a leaf of the coarse level; some entries have a weight of their own
            leaves = n1 + np.arange(twice)
            n1 += twice
            ends += [(me[:twice], leaves), (leaves, to[:twice])]
        twice_ends.append((me[:twice], to[-twice:]))
    stars, leaves = np.repeat(np.arange(n1), 3), np.arange(n1, 4 * n1)
    u2, v2 = (np.concatenate(e) for e in zip(*twice_ends))
    more = 4 * n1 + np.arange(u2.size)  # leaves of a star that are tied to another, too
    u, v = (np.concatenate((*e, *rest)) for e, rest in zip(zip(*ends), ((stars, u2, v2), (leaves, more, more))))
    n = 4 * n1 + u2.size
    key = np.unique(np.minimum(u, v) * n + np.maximum(u, v))
    return graphgen.to_csr(n, torch.from_numpy(np.stack((key // n, key % n), 1)))


@pytest.mark.parametrize("wide_sums", [0, 1])
@pytest.mark.parametrize("weight_bits", [0, 1])
def test_rows_around_the_longest_of_every_network(bordered, weight_bits, wide_sums):
    """Weights that all lie beside their columns (0: the 14 bits that are left) and such as do not."""
    n = bordered.xadj.numel() - 1
    ref = G.gosh_coarsen(n, bordered.xadj, bordered.adj, threshold=4, min_shrink=1.0, max_levels=3)
    for i in range(2):
        lengths = np.bincount(ref.map(i), weights=np.diff(ref.graph(i)[1])).astype(int)
        assert {b + o for b in NETWORKS for o in (-1, 0, 1)} <= set(lengths), i
        assert ref.shape(i + 1)[0] > 14 << 14 and ref.mult(i + 1).max() > 1
    with seam(SEAM_WEIGHT_BITS, weight_bits), seam(SEAM_WIDE_SUMS, wide_sums):
        assert_equals_host(bordered, 3, threshold=4, min_shrink=1.0, max_levels=3)


@pytest.mark.parametrize("n,linked,m", [
    (30_000, 30_000, 20_000),   # rows of one entry and without: more than a tile's tables hold
    (16_003, 9_003, 36_011),    # tiles of some hundred rows, the last one spans thousands without entries
    ((1 << 19) + 5, (1 << 19) + 5, 900_000)])  # clusters looked up in three bytes per vertex
def test_rows_of_a_tile(n, linked, m):
    """The tables by which the gather and the copy of the merged rows find the row of an entry."""
    assert_equals_host(graphgen.to_csr(n, graphgen.er_gnm(linked, m, 3)), threshold=10, min_shrink=1.0)


def test_clusters_are_looked_up_in_the_map_where_there_is_no_room_for_a_narrower_one():
    n = (1 << 19) + 5
    with seam(SEAM_DENY, DENY_NARROW):
        assert_equals_host(graphgen.to_csr(n, graphgen.er_gnm(n, 900_000, 3)), threshold=10, min_shrink=1.0, max_levels=3)


def test_more_undecided_vertices_than_a_wavefront_holds():
    """Two random permutations, and a vertex of a hundred neighbours that lifts the mean degree above the four of
    all others: nearly every vertex is undecided at first."""
    n = 1_200_007
    g = torch.Generator().manual_seed(3)
    ids = torch.arange(n)
    ends = [torch.cat((ids, ids, torch.zeros(100, dtype=torch.int64))),
            torch.cat([torch.randperm(n, generator=g) for _ in range(2)] + [torch.arange(1000, 1100)])]
    lo, hi = torch.minimum(*ends), torch.maximum(*ends)
    key = torch.unique((lo * n + hi)[lo < hi])
    assert_equals_host(graphgen.to_csr(n, torch.stack((key // n, key % n), 1)), threshold=n // 2, min_shrink=1.0, max_levels=2)

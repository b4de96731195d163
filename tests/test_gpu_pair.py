"""GPU parity of the pair path (deep graphs of low degree: per-source queues of
a level's vertices) against the oracle, and where a graph is found deep."""
import numpy as np
import pytest

import graphgen as gg
import paper_2401_02472_amd as bcm
from tests.gpu_checks import batched, check_bc, oracle_bc, oracle_bc_ext, plain, run_mode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    bcm.load_library()


def _auto(G, src):
    return run_mode(G, src, bcm.BC_MODE_AUTO)


def _deg16():
    """A long chain of vertices of exactly 16 arcs (8 parallel arcs to each
    neighbour) with self-loops' worth of room left, and pendant paths."""
    n, h = 21000, 60
    a = [(i, i + 1) for i in range(h) for _ in range(8)]
    b = [(h + 1 + i, h + 2 + i) for i in range(n - h - 2)]
    b += [(0, n - 1), (h, h + 1)]
    p = np.array(a + b)
    return gg.csr_from_edges(n, p[:, 0], p[:, 1], dedup=False)


def _island_grid():
    """A road-like grid beside isolated vertices and a short second component."""
    g = gg.grid_road(150, 150, seed=3)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    keep = src < g.col_idx
    u = np.concatenate([src[keep], [g.n + 10, g.n + 11, g.n + 11]])
    v = np.concatenate([g.col_idx[keep], [g.n + 11, g.n + 12, g.n + 13]])
    return gg.csr_from_edges(g.n + 20, u, v)


@pytest.mark.parametrize("g,k", [
    (gg.grid_road(150, 150, seed=1), 1), (gg.grid_road(150, 150, seed=1), 2),
    (gg.grid_road(300, 211, 0.05, 0.0, seed=2), 16), (gg.grid_road(160, 131, seed=5), 64),
    (gg.grid_road(160, 131, seed=5), 65), (gg.grid_road(160, 131, seed=5), 200),
    (_island_grid(), 70), (_deg16(), 40),
], ids=["k1", "k2", "deep16", "k64", "k65", "k200", "islands", "deg16"])
def test_parity(g, k):
    src = gg.sample_sources(g, k, seed=7)
    if g.n == 150 * 150 + 20:  # duplicates, an isolated source, the second component
        src[:6] = [5, 5, g.n - 20, g.n - 9, g.n - 8, g.n - 1]
    want = oracle_bc(g, src)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        first = batched(G, src)           # found deep on the way (or by what follows)
        check_bc(first, want)
        check_bc(plain(G, src[:2]), oracle_bc(g, src[:2]))
        got = batched(G, src)             # pairs from the first level on
        check_bc(got, want)
        assert np.array_equal(got, batched(G, src))
        check_bc(_auto(G, src[:1]), oracle_bc(g, src[:1]))
        check_bc(_auto(G, src[:3]), oracle_bc(g, src[:3]))
        # the loops that a caller names stay themselves
        host = batched(G, src, level_loop=bcm.BC_LOOP_HOST)
        assert np.array_equal(host, batched(G, src, level_loop=bcm.BC_LOOP_GRAPH))
        check_bc(host, want)


def test_profiled_run_counts_the_pairs():
    """Work counters of a profiled run: every reached (vertex, source) pair once
    per pass (the sources themselves in the forward pass only)."""
    g = gg.grid_road(160, 140, seed=8)
    src = gg.sample_sources(g, 20, seed=9)
    want = oracle_bc(g, src)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        batched(G, src)
        _, dist, _ = G.run_detail(src, bcm.make_options(bcm.BC_MODE_BATCHED))
        reached = int((dist >= 0).sum())
        G.profile_enable(True)
        G.profile_read(reset=True)
        check_bc(batched(G, src), want)
        p = G.profile_read(reset=True)
        assert p["forward"]["owners"] == reached
        assert p["reverse"]["owners"] == reached - src.size
        # each DAG arc once per pass, but for the arcs out of the sources
        first = sum(int((dist[i][g.col_idx[g.row_ptr[s]:g.row_ptr[s + 1]]] == 1).sum())
                    for i, s in enumerate(src))
        assert p["reverse"]["hits"] == p["forward"]["hits"] - first


@pytest.mark.parametrize("case", ["rounds", "range", "grow"])
def test_profiled_run_of_several_rounds(case):
    """The counters hold every round of a call: rounds of unequal size, sources
    run again with exponents, sources run again with room for more levels."""
    if case == "rounds":  # 3.4 MB of scratch per source, 4 GB per round
        g = gg.grid_road(400, 400, seed=10)
        src = np.tile(gg.sample_sources(g, 13, seed=11), 100)
    elif case == "range":
        g = gg.grid_full(600, 600)
        src = np.array([0, 599, 180300, 359999], np.int32)
    else:
        g = gg.path(21000)
        src = np.array([0, 20999, 10000, 3], np.int32)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        plain(G, src[:1])  # found deep; the pair path has not run yet
        G.profile_enable(True)
        G.profile_read(reset=True)
        batched(G, src)
        p = G.profile_read(reset=True)
        pairs = src.size * g.n  # the graphs are connected but for a few vertices
        assert p["forward"]["vertices"] == 0, "not the pair path"
        if case == "rounds":
            _, dist, _ = G.run_detail(src[:13], bcm.make_options(bcm.BC_MODE_BATCHED))
            pairs = 100 * int((dist >= 0).sum())
            assert p["forward"]["owners"] == pairs
            assert p["reverse"]["owners"] == pairs - src.size
        else:
            # a round that is given up counts what it did: one without
            # exponents, five with 1024 << i of the path's 21,000 levels
            tries = 2 if case == "range" else 6
            assert pairs <= p["forward"]["owners"] <= tries * pairs
            assert pairs - src.size <= p["reverse"]["owners"] <= tries * pairs
            assert p["forward"]["owners"] <= p["forward"]["arcs"] + 2 * src.size
            batched(G, src)  # one round
            p = G.profile_read(reset=True)
            assert p["forward"]["owners"] == pairs
            assert p["reverse"]["owners"] == pairs - src.size


def test_few_sources_past_a_group_share_the_round():
    """22.0 MB per source: a round's 4 GB hold 194 sources of this graph, 24
    groups of eight and two more, so 193 are one round.  A launch per level: a
    second round would add at least half as many as the deepest source takes,
    a source reaching at least half as far as any other."""
    g = gg.grid_road(1024, 1024, 0.05, 0.001, seed=2)
    src = gg.sample_sources(g, 193, seed=102)
    launches = {}
    with bcm.Graph(g.n, g.row_ptr, g.col_idx, bcm.BC_GRAPH_TRUST_SYMMETRIC) as G:
        batched(G, src)  # the depth is known from here on
        G.profile_enable(True)
        for m in (192, 193):
            G.profile_read(reset=True)
            got = batched(G, src[:m])
            p = G.profile_read(reset=True)
            assert p["forward"]["vertices"] == 0, "not the pair path"
            launches[m] = p["forward"]["launches"]
    assert launches[192] <= launches[193] < 1.25 * launches[192]
    check_bc(got, oracle_bc(g, src))


def test_counts_beyond_double_range():
    """A lattice whose counts pass double's range: found on the way, run again
    with exponents, and with them from the start in later calls."""
    g = gg.grid_full(600, 600)
    src = np.array([0, 599, 180300, 359999] + list(range(7, 340000, 28000)), np.int32)
    want = oracle_bc_ext(g, src)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        check_bc(batched(G, src), want)
        check_bc(batched(G, src), want)
        check_bc(_auto(G, src), want)
        # sources whose counts fit give the same with exponents as without
    small = np.array([180300, 180301], np.int32)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        plain(G, small[:1])
        a = _auto(G, small)
        check_bc(a, oracle_bc(g, small))
        _auto(G, src)
        assert np.array_equal(a, _auto(G, small))


@pytest.mark.parametrize("rows,cols,short,k,ext", [
    (700, 701, 0.001, 2, False),    # wide levels, few sources: a launch per level
    (1150, 1147, 0.001, 3, False),  # past the vertices whose visited bits fit LDS
    (1150, 1147, 0.0, 2, True),     # ... and counts past double's range
], ids=["wide", "large", "large-ext"])
def test_launch_per_level(rows, cols, short, k, ext):
    g = gg.grid_road(rows, cols, 0.0 if ext else 0.05, short, seed=12)
    src = gg.sample_sources(g, k, seed=13)
    if ext:
        src[0] = 0
    want = oracle_bc_ext(g, src) if ext else oracle_bc(g, src)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        for _ in range(3):
            got = batched(G, src)
            check_bc(got, want)
        assert np.array_equal(got, batched(G, src))


@pytest.mark.parametrize("g,k", [
    (gg.grid_road(150, 150, seed=1), 1), (gg.grid_road(150, 150, seed=1), 3),
    (gg.grid_road(150, 150, seed=1), 20), (gg.grid_road(400, 400, seed=10), 1300),
    (_island_grid(), 3), (gg.grid_full(600, 600), 9),
], ids=["k1", "k3", "k20", "rounds", "islands", "range"])
def test_a_call_gives_the_same_bits_whatever_ran_before(g, k):
    """The first call on a graph, one after calls with other sources, and one
    on a graph that ran something else first (the rounds of the 1,300 sources
    follow the depth seen)."""
    src = gg.sample_sources(g, min(k, 13), seed=21)
    src = np.tile(src, -(-k // src.size))[:k]
    if g.n == 600 * 600:
        src[0] = 0  # (counts past double's range)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        first = _auto(G, src)
        _auto(G, gg.sample_sources(g, 40, seed=22))
        G.single_source(180300 % g.n)  # (the lattice's middle: its counts fit double)
        assert np.array_equal(first, _auto(G, src))
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        _auto(G, src[:1])
        plain(G, src[1:2])
        assert np.array_equal(first, _auto(G, src))


def test_more_levels_than_the_first_estimate_and_trim():
    g = gg.path(21000)
    src = np.array([0, 20999, 10000, 3], np.int32)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        for _ in range(2):
            check_bc(batched(G, src), oracle_bc(g, src))
        assert 0 < G.workspace_held()
        G.trim_workspaces()
        assert G.workspace_held() == 0
        check_bc(_auto(G, src), oracle_bc(g, src))


def test_rounds_of_sources():
    """More sources than a round's scratch holds (3.4 MB each of 4 GB)."""
    g = gg.grid_road(400, 400, seed=10)
    ten = gg.sample_sources(g, 13, seed=11)
    src = np.tile(ten, 100)
    want = 100.0 * oracle_bc(g, ten)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        check_bc(batched(G, ten), oracle_bc(g, ten))
        check_bc(batched(G, src), want)


class _LittleMemory:
    """All of the device's memory but `leave` bytes taken (0: but for less than
    16 MB, whatever the free size reported)."""

    def __init__(self, leave):
        self.leave = leave

    def __enter__(self):
        import torch
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free, _ = torch.cuda.mem_get_info()
        leave = self.leave or 64 << 20
        self.blocks = [torch.empty(free - leave, dtype=torch.uint8, device="cuda")]
        try:
            while not self.leave and len(self.blocks) < 64:
                self.blocks.append(torch.empty(16 << 20, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass

    def __exit__(self, *exc):
        import torch
        self.blocks.clear()
        torch.cuda.empty_cache()


def test_fewer_sources_at_a_time_where_memory_is_short():
    g = gg.grid_road(1000, 1000, seed=23)
    some = gg.sample_sources(g, 10, seed=24)
    src = np.tile(some, 15)  # 3 GB or more of scratch at once
    want = 15.0 * oracle_bc(g, some)
    import torch
    out = torch.empty(g.n, dtype=torch.float64, device="cuda")
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        with _LittleMemory(1 << 30):
            G.run_async(src, out)
        check_bc(out.cpu().numpy(), want)
        G.run_async(src, out)
        check_bc(out.cpu().numpy(), want)


def test_another_path_where_memory_has_no_room_for_the_queues():
    g = gg.grid_road(1000, 1000, seed=23)
    src = gg.sample_sources(g, 2, seed=25)
    import torch
    out = torch.empty(g.n, dtype=torch.float64, device="cuda")
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        plain(G, src)  # its workspace is pooled (and given back to the call below)
        with _LittleMemory(0):
            G.run_async(src, out)
        check_bc(out.cpu().numpy(), oracle_bc(g, src))


def _caterpillar():
    """A deep tree of 23,230 vertices (one path between any two: counts of 1, so
    the host loop keeps its narrow rows): 505 vertices in a row, three children
    each, fourteen leaves to each of those."""
    spine = np.arange(505)
    kids = 505 + np.arange(3 * 505)
    leaves = 4 * 505 + np.arange(42 * 505)
    u = np.concatenate([spine[:-1], np.repeat(spine, 3), np.repeat(kids, 14)])
    v = np.concatenate([spine[1:], kids, leaves])
    return gg.csr_from_edges(46 * 505, u, v)


def test_admission_covers_every_call_on_a_deep_graph():
    """bc_workspace_bytes against the workspaces that the calls leave pooled: the
    host loop's for requests (the call of the server), the queues and the vertex
    order for a call of its own."""
    import torch
    g = _caterpillar()
    src = np.array([0], np.int32)
    want = oracle_bc(g, src)
    opt = bcm.make_options(bcm.BC_MODE_BATCHED, concurrency=1)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        plain(G, src)
        G.trim_workspaces()
        out = torch.empty(g.n, dtype=torch.float64, device="cuda")
        G.run_multi([src], [out])
        check_bc(out.cpu().numpy(), want)
        assert 0 < G.workspace_held() <= G.workspace_bytes(1, opt)
        G.trim_workspaces()
        check_bc(batched(G, src), want)
        order = 28 * g.n + 4 * g.nnz
        assert order < G.workspace_held() <= G.workspace_bytes(1, opt)
        G.trim_workspaces()
        assert G.workspace_held() == 0
        check_bc(batched(G, src), want)  # the vertex order built again


@pytest.mark.parametrize("g", [gg.rmat(11, 9, seed=26), gg.grid_road(150, 147, seed=27)],
                         ids=["small", "deep"])
def test_autotune_times_the_loop_its_settings_belong_to(g):
    """A small graph's own calls take a workgroup per source and a deep graph's
    take queues, which read none of the tuned settings: the tuner times the host
    loop there, and the calls stay as they were."""
    src = gg.sample_sources(g, 100, seed=28)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        before = _auto(G, src)
        G.profile_enable(True)
        G.profile_read(reset=True)
        assert not G.autotune(src)["cached"]
        p = G.profile_read(reset=True)
        assert p["fused"]["launches"] == 0 and p["forward"]["vertices"] > 0
        assert np.array_equal(before, _auto(G, src))
        p = G.profile_read(reset=True)
        if g.n <= 20415:
            assert p["fused"]["launches"] == 1
        else:
            assert p["forward"]["launches"] > 0 and p["forward"]["vertices"] == 0
        G.profile_enable(False)
        check_bc(before, oracle_bc(g, src))


@pytest.mark.parametrize("tail,deep", [(44, False), (45, True)])
def test_where_a_graph_is_deep(tail, deep):
    """A tree of fifteen children per vertex and four levels with a path at its
    root: 4 + tail levels from a leaf, of which three of the four searches at
    creation start."""
    n = 54241
    kids = np.arange(1, n)
    ends = n + np.arange(tail)
    g = gg.csr_from_edges(n + tail, np.concatenate([(kids - 1) // 15, [0], ends[:-1]]),
                          np.concatenate([kids, ends[:1], ends[1:]]))
    src = gg.sample_sources(g, 20, seed=29)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        G.profile_enable(True)
        check_bc(_auto(G, src), oracle_bc(g, src))
        p = G.profile_read(reset=True)
        as_queues = (p["fused"]["launches"] == 0 and p["forward"]["vertices"] == 0
                     and p["forward"]["launches"] > 0)
        assert as_queues == deep

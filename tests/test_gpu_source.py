"""GPU parity of the device-resident level loop (one workgroup per source)
where its kernel can go wrong: the largest graph whose values fit LDS and the
first that does not, the degree classes' edges (8 / 9, 64 / 65, 512 / 513
arcs), arcs that lead back many levels in directed graphs, several sources per
workgroup, several launches per call, and requests that share a call."""
import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2401_02472_amd as bcm
from tests.gpu_checks import batched, check_bc, check_sigma, oracle_bc, run_mode
from tests.test_gpu_pair import _LittleMemory

pytestmark = pytest.mark.gpu

MAX_N = 20415  # (160 KB - 512) / 8 - 1 values


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    bcm.load_library()


def _hubs(degrees, leaves):
    """A cycle of hubs, hub i with degrees[i] arcs (2 of them along the cycle),
    the rest to shared leaves chosen in turn."""
    h = len(degrees)
    pairs, at = [(i, (i + 1) % h) for i in range(h)], 0
    for i, d in enumerate(degrees):
        for _ in range(d - 2):
            pairs.append((i, h + at % leaves))
            at += 1
    p = np.array(pairs)
    return gg.csr_from_edges(h + leaves, p[:, 0], p[:, 1])


def _device(G, src):
    return batched(G, src, level_loop=bcm.BC_LOOP_DEVICE)


@pytest.mark.parametrize("g", [
    _hubs([7, 8, 9, 10, 63, 64, 65, 66, 511, 512, 513, 514, 1025, 3, 4, 5], 1500),
    _hubs([64, 65, 66, 67, 68, 127, 128, 129, 255, 256, 257], 300),
    gg.path(3), gg.star(2), gg.complete(70), gg.cycle(700),
    gg.erdos_renyi(MAX_N, 6, seed=1), gg.erdos_renyi(MAX_N + 1, 6, seed=1),
], ids=["hubs", "hubs16", "path3", "edge", "K70", "cycle", "largest", "too-large"])
def test_classes_and_size_limit(g):
    src = gg.sample_sources(g, min(g.n, 40), seed=2)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        got = _device(G, src)
        check_bc(got, oracle_bc(g, src))
        assert np.array_equal(got, _device(G, src))
        opt = bcm.make_options(bcm.BC_MODE_BATCHED, level_loop=bcm.BC_LOOP_DEVICE)
        _, dist, sigma = G.run_detail(src[:3], opt)
        for i in range(min(3, src.size)):
            od, osg, _, _ = oracle.single_source(g.row_ptr, g.col_idx, int(src[i]), with_delta=False)
            assert np.array_equal(dist[i], od)
            check_sigma(sigma[i], osg)
        # the measured run is another instance of the kernel
        G.profile_enable(True)
        assert np.array_equal(got, _device(G, src))
        G.profile_enable(False)


def test_directed_arcs_back_to_early_levels():
    """A long directed path whose vertices also point back to vertices of every
    earlier level (and of every residue of the level), joined to a dense part."""
    n = 60
    pairs = [(i, i + 1) for i in range(n - 1)]
    pairs += [(i, j) for i in range(n) for j in range(i) if (i * 7 + j) % 3 == 0]
    rng = np.random.default_rng(4)
    pairs += [(int(a), int(b)) for a, b in rng.integers(0, 400, (3000, 2)) if a != b]
    g = gg.directed(400, pairs, "back-arcs")
    src = np.arange(0, 400, 3, dtype=np.int32)
    want, st = oracle.bc(g.row_ptr, g.col_idx, src, directed=True)
    assert st == oracle.OK
    with bcm.Graph(g.n, g.row_ptr, g.col_idx, flags=bcm.BC_GRAPH_DIRECTED) as G:
        check_bc(_device(G, src), want)
        check_bc(_device(G, src[:1]), oracle.bc(g.row_ptr, g.col_idx, src[:1], directed=True)[0])


@pytest.mark.parametrize("k", [1, 512, 513, 1300])
def test_several_sources_per_workgroup(k):
    g = gg.rmat(11, 8, seed=5)
    src = gg.sample_sources(g, k, seed=6)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        got = _device(G, src)
        check_bc(got, oracle_bc(g, src))
        assert np.array_equal(got, _device(G, src))


def test_requests_over_several_launches_equal_alone():
    """More units than a launch's scratch holds (512 MB at 0.7 MB each): small
    requests before and after a large one whose units two launches share."""
    import torch
    g = gg.erdos_renyi(20000, 5, seed=7)
    sizes = [1] * 380 + [700] + [0] + [2] * 120
    reqs = [gg.sample_sources(g, k, seed=100 + i) if k else np.zeros(0, np.int32)
            for i, k in enumerate(sizes)]
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        outs = [torch.full((g.n,), -1.0, dtype=torch.float64, device="cuda") for _ in reqs]
        G.run_multi(reqs, outs)
        torch.cuda.synchronize()
        for i in (0, 200, 379, 380, 381, 382, len(reqs) - 1):
            alone = torch.full((g.n,), -1.0, dtype=torch.float64, device="cuda")
            G.run_multi([reqs[i]], [alone])
            got = outs[i].cpu().numpy()
            assert np.array_equal(got, alone.cpu().numpy()), f"request {i}"
            check_bc(got, oracle_bc(g, reqs[i]) if sizes[i] else np.zeros(g.n))


def test_workspaces_are_reported_and_trimmed():
    g = gg.rmat(12, 8, seed=8)
    src = gg.sample_sources(g, 100, seed=9)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        opt = bcm.make_options(bcm.BC_MODE_BATCHED, level_loop=bcm.BC_LOOP_DEVICE)
        want = _device(G, src)
        assert 0 < G.workspace_held() <= G.workspace_bytes(100, opt)
        G.trim_workspaces()
        assert G.workspace_held() == 0
        assert np.array_equal(want, _device(G, src))


@pytest.mark.parametrize("g,k,device", [
    (gg.erdos_renyi(10000, 100, seed=31), 40, False),   # few levels, many arcs
    (gg.erdos_renyi(10000, 100, seed=31), 300, True),   # ... but five batches
    (gg.rmat(12, 8, seed=32), 64, True),
    (gg.erdos_renyi(MAX_N, 4, seed=33), 64, True),
], ids=["dense", "dense-many", "rmat", "sparse"])
def test_the_loop_that_a_call_takes(g, k, device):
    src = gg.sample_sources(g, k, seed=34)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        G.profile_enable(True)
        got = batched(G, src)
        p = G.profile_read(reset=True)
        assert (p["fused"]["launches"] > 0) == device
        check_bc(got, oracle_bc(g, src))


def _back_arcs(n):
    """A directed graph of n vertices: a path of 70 levels whose vertices also
    point back, a dense part, and a sparse rest."""
    pairs = [(i, i + 1) for i in range(69)]
    pairs += [(i, j) for i in range(70) for j in range(i) if (i * 7 + j) % 3 == 0]
    rng = np.random.default_rng(n)
    pairs += [(int(a), int(b)) for a, b in rng.integers(0, 400, (3000, 2)) if a != b]
    pairs += [(int(a), int(b)) for a, b in rng.integers(0, n, (2 * n, 2)) if a != b]
    return gg.directed(n, pairs, "back-arcs")


@pytest.mark.parametrize("g,k", [
    (gg.erdos_renyi(MAX_N + 1, 4, seed=35), 70),          # the first past the LDS
    (gg.erdos_renyi(20448, 3, seed=36), 600),             # 639 whole words of bits
    (gg.erdos_renyi(20447, 3, seed=36), 600), (gg.erdos_renyi(20449, 3, seed=36), 1),
    (_hubs([7, 8, 9, 10, 63, 64, 65, 66, 511, 512, 513, 514, 1025, 3, 4, 5] + [3] * 9000, 22000), 40),
    (gg.rmat(15, 5, seed=37), 300),
    (gg.erdos_renyi(131072, 2, seed=38), 20),             # the largest ...
    (_back_arcs(30011), 90), (_back_arcs(20416), 600),
], ids=["first", "words", "words-1", "words+1", "hubs", "rmat", "largest", "back", "back-many"])
def test_values_in_memory(g, k):
    """Graphs whose values do not fit LDS: a bit per vertex there instead."""
    directed = g.name == "back-arcs"
    src = gg.sample_sources(g, min(k, 50), seed=39)
    src = np.tile(src, -(-k // src.size))[:k]
    want, st = oracle.bc(g.row_ptr, g.col_idx, src, directed=directed)
    assert st == oracle.OK
    with bcm.Graph(g.n, g.row_ptr, g.col_idx, bcm.BC_GRAPH_DIRECTED if directed else 0) as G:
        got = _device(G, src)
        check_bc(got, want)
        assert np.array_equal(got, _device(G, src))
        opt = bcm.make_options(bcm.BC_MODE_BATCHED, level_loop=bcm.BC_LOOP_DEVICE)
        few = src[:3]
        _, dist, sigma = G.run_detail(few, opt)
        for i in range(few.size):
            od, osg, _, _ = oracle.single_source(g.row_ptr, g.col_idx, int(few[i]),
                                                 with_delta=False, directed=directed)
            assert np.array_equal(dist[i], od)
            check_sigma(sigma[i], osg)
        G.profile_enable(True)
        G.profile_read(reset=True)
        assert np.array_equal(got, _device(G, src))
        p = G.profile_read(reset=True)
        assert p["fused"]["launches"] == 1, "not the device-resident loop"
        G.profile_enable(False)
        assert 0 < G.workspace_held() <= G.workspace_bytes(k, opt)


def test_graph_beyond_the_values_in_memory():
    g = gg.erdos_renyi(131073, 2, seed=38)
    src = gg.sample_sources(g, 20, seed=39)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        G.profile_enable(True)
        check_bc(_device(G, src), oracle_bc(g, src))
        assert G.profile_read(reset=True)["fused"]["launches"] == 0


def test_thousands_of_sources_past_the_lds_limit():
    """Exact-BC-like calls: one launch of a workgroup per source, not batches."""
    g = gg.erdos_renyi(21000, 4, seed=40)
    some = gg.sample_sources(g, 64, seed=41)
    src = np.tile(some, 16)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        G.profile_enable(True)
        got = run_mode(G, src, bcm.BC_MODE_AUTO)
        assert G.profile_read(reset=True)["fused"]["launches"] == 1
        check_bc(got, 16.0 * oracle_bc(g, some))


def test_requests_and_graphs_past_the_lds_limit():
    """Requests equal the ones alone and graphs that join a call their own runs,
    with the values in LDS and in memory, undirected and directed."""
    import torch
    g = gg.erdos_renyi(25001, 4, seed=42)
    reqs = [gg.sample_sources(g, k, seed=43 + k) for k in (1, 8, 64, 5, 300, 1)]
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        outs = [torch.full((g.n,), -1.0, dtype=torch.float64, device="cuda") for _ in reqs]
        G.run_multi(reqs, outs)
        for r, o in zip(reqs, outs):
            alone = torch.full((g.n,), -1.0, dtype=torch.float64, device="cuda")
            G.run_multi([r], [alone])
            assert torch.equal(o, alone)
            check_bc(o.cpu().numpy(), oracle_bc(g, r))
    gs = [gg.rmat(11, 8, seed=44), g, _back_arcs(22222), gg.directed(50, [(i, i + 1) for i in range(49)], "p"),
          gg.erdos_renyi(60000, 3, seed=45)]
    dirs = [False, False, True, True, False]
    Gs = [bcm.Graph(x.n, x.row_ptr, x.col_idx, bcm.BC_GRAPH_DIRECTED if d else 0)
          for x, d in zip(gs, dirs)]
    srcs = [gg.sample_sources(x, min(40, x.n - 1), seed=46) for x in gs]
    outs = [torch.full((x.n,), -1.0, dtype=torch.float64, device="cuda") for x in gs]
    loops = bcm.bc_run_graphs(Gs, srcs, outs)
    assert all(lp == bcm.BC_LOOP_DEVICE for lp in loops)
    for x, d, G, s, o, lp in zip(gs, dirs, Gs, srcs, outs, loops):
        own = batched(G, s, level_loop=lp, batch_width=64)
        assert np.array_equal(o.cpu().numpy(), own)
        check_bc(own, oracle.bc(x.row_ptr, x.col_idx, s, directed=d)[0])
        G.close()


def test_the_host_loop_where_the_scratch_does_not_fit():
    g = gg.erdos_renyi(50000, 4, seed=47)  # 512 units of 2.2 MB
    some = gg.sample_sources(g, 50, seed=48)
    src = np.tile(some, 11)
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        with _LittleMemory(640 << 20):
            got = run_mode(G, src, bcm.BC_MODE_AUTO)
        check_bc(got, 11.0 * oracle_bc(g, some))

"""Draws and subgraphs at the edges of their kernels' shapes, bit for bit against the oracle:
numbers of items around a subtile (16), a tile (4096) and a bitmap tile (32,768), weights
concentrated at the ends of tiles, probabilities at an address that is 8- but not 16-byte
aligned, rows around the 64 entries that a wavefront reads in one step and the 1024 that it reads
at once, draws around the counts from which marks are bytes and every edge is looked at,
indices written over the probabilities, and scratch at an odd address."""
import numpy as np
import pytest

import gen
from oracle import sampling as OS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_27209_amd as E
    return E


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 255, 4095, 4096, 4097, 8192, 32768, 32769])
def test_draw_at_tile_edges(n, shift):
    E = _gpu()
    g = gen.path_graph(n)
    rng = np.random.default_rng(n)
    P = rng.random(n) ** 8  # a few items carry most of the weight
    P[rng.random(n) < 0.3] = 0.0
    P[-1] = P[0] = 1.0
    P[15::16] = 0.0
    if n > 4096:
        P[4095] = P[4096] = 5.0
    P /= P.sum()
    G = E.Graph(g.rowptr, g.col, g.w)
    buf = torch.zeros(n + 1, dtype=torch.float64, device="cuda")
    prob = buf[shift:shift + n]
    prob.copy_(torch.from_numpy(P))
    got = G.draw("nodes", prob, 3000, seed=7).cpu().numpy()
    np.testing.assert_array_equal(got, OS.draw(P, 3000, 7))


def _hub_graph(n, degree):
    """Node 0 joined to 1 .. degree, and a path through all nodes."""
    u = np.concatenate([np.zeros(degree, np.int64), np.arange(n - 1)])
    v = np.concatenate([np.arange(1, degree + 1), np.arange(1, n)])
    return gen.from_edges(n, u, v)


@pytest.mark.parametrize("n,degree", [(70, 64), (600, 511), (600, 512), (600, 513), (5000, 4999),
                                      (32768, 1100), (32769, 32768), (131072, 1500)])
@pytest.mark.parametrize("items", ["nodes", "edges"])
def test_subgraph_at_row_and_tile_edges(n, degree, items):
    E = _gpu()
    g = _hub_graph(n, degree)
    G = E.Graph(g.rowptr, g.col, g.w)
    rng = np.random.default_rng(n + degree)
    N = n if items == "nodes" else g.m
    idx = np.concatenate([rng.integers(0, N, max(2, N // 2)), [0, N - 1, 0]])
    got = G.subgraph(items, torch.from_numpy(idx).cuda())
    want = (OS.node_subgraph if items == "nodes" else OS.edge_subgraph)(g, idx)
    for k in ("nodes", "edges", "u", "v"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])


def test_subgraph_scratch_at_an_odd_address():
    E = _gpu()
    from paper_2609_27209_amd import _abi
    g = _hub_graph(300, 200)
    G = E.Graph(g.rowptr, g.col, g.w)
    nb = _abi.erc_subgraph_scratch_bytes(G.handle)
    G._scratches["subgraph"] = torch.empty(nb + 4, dtype=torch.uint8, device="cuda")[4:]
    idx = np.arange(0, 300, 3)
    got = G.subgraph("nodes", torch.from_numpy(idx).cuda())
    want = OS.node_subgraph(g, idx)
    np.testing.assert_array_equal(got["edges"].cpu().numpy(), want["edges"])


def _random_graph(n, m, seed):
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    return gen.from_edges(n, u[u != v], v[u != v])


@pytest.mark.parametrize("n,m,count", [
    # marks by bits up to 65,536 draws, by bytes above; every edge from n / 16 node draws on
    (1000, 5000, 65536), (1000, 5000, 65537), (1000, 32768, 70000), (40000, 33000, 65537),
    (20000, 65536, 1249), (20000, 65536, 1250), (20000, 65700, 1251), (33, 400, 1), (33, 400, 2), (2, 1, 1),
    # more than 64 items per draw keep the bits
    (5000000, 4300000, 66000), (5000000, 4300000, 79000)])
@pytest.mark.parametrize("items", ["nodes", "edges"])
def test_subgraph_of_many_draws(n, m, count, items):
    E = _gpu()
    g = _random_graph(n, m, n + m) if n > 2 else gen.path_graph(2)
    G = E.Graph(g.rowptr, g.col, g.w)
    rng = np.random.default_rng(count)
    N = n if items == "nodes" else g.m
    # half of the draws fall on a tenth of the items
    idx = np.where(rng.random(count) < 0.5, rng.integers(0, N, count), rng.integers(0, N // 10 + 1, count))
    idx[-1] = N - 1
    got = G.subgraph(items, torch.from_numpy(idx).cuda())
    want = (OS.node_subgraph if items == "nodes" else OS.edge_subgraph)(g, idx)
    for k in ("nodes", "edges", "u", "v"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])


@pytest.mark.parametrize("bad", [-1, 1000])
def test_bad_index_among_many_draws(bad):
    E = _gpu()
    from paper_2609_27209_amd import _abi
    g = _random_graph(1000, 5000, 3)
    G = E.Graph(g.rowptr, g.col, g.w)
    idx = torch.arange(70000, dtype=torch.int64, device="cuda") % 1000
    idx[12345] = bad
    with pytest.raises(_abi.ErcError) as ei:
        G.subgraph("nodes", idx)
    assert ei.value.status == _abi.ERC_E_INVALID_ARG


@pytest.mark.parametrize("n,draws,at", [(5000, 5000, 0), (5000, 300, 100), (70000, 69000, 1000), (70000, 32768, 0)])
def test_indices_in_place_of_probabilities(n, draws, at):
    E = _gpu()
    from paper_2609_27209_amd import _abi
    rng = np.random.default_rng(n)
    P = rng.random(n)
    P /= P.sum()
    G = E.Graph(*(lambda g: (g.rowptr, g.col, g.w))(gen.path_graph(n)))
    buf = torch.from_numpy(P).cuda()
    sc = torch.empty(_abi.erc_draw_scratch_bytes(G.handle, _abi.ERC_NODES), dtype=torch.uint8, device="cuda")
    _abi.erc_draw(G.handle, _abi.ERC_NODES, buf.data_ptr(), draws, 9, sc.data_ptr(), sc.numel(),
                  buf.data_ptr() + 8 * at, torch.cuda.current_stream().cuda_stream)
    got = buf.view(torch.int64)[at:at + draws].cpu().numpy()
    np.testing.assert_array_equal(got, OS.draw(P, draws, 9))
    rest = np.concatenate([np.arange(at), np.arange(at + draws, n)])
    np.testing.assert_array_equal(buf.cpu().numpy()[rest], P[rest])


@pytest.mark.parametrize("degree", [63, 64, 65, 1022, 1023, 1024, 1025, 2047, 2048, 2049, 3073])
def test_long_rows_of_kept_nodes(degree):
    """The hub's row and as many of its neighbours as the draws that look at rows allow."""
    E = _gpu()
    n = 64 * degree
    g = _hub_graph(n, degree)
    G = E.Graph(g.rowptr, g.col, g.w)
    rng = np.random.default_rng(degree)
    # fewer than n / 16 draws: the hub, its first and last neighbours, and most of the others
    kept = np.concatenate([[0, 1, degree, degree - 1], 1 + rng.permutation(degree)[:max(0, n // 16 - 5)]])
    assert kept.size < n // 16 and np.unique(kept).size > 0.9 * degree
    idx = rng.permutation(kept)
    got = G.subgraph("nodes", torch.from_numpy(idx).cuda())
    want = OS.node_subgraph(g, idx)
    for k in ("nodes", "edges", "u", "v"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])

"""Draws and subgraphs at the edges of their kernels' shapes, bit for bit against the oracle:
numbers of items around a subtile (16), a tile (4096) and a bitmap tile (32,768), weights
concentrated at the ends of tiles, probabilities at an address that is 8- but not 16-byte
aligned, rows around the 512 entries that a wavefront reads at once, and scratch at an odd
address."""
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

"""The copies that erc_create makes: every array of the graph buffer arrives whole.

Small arrays go up together, from a buffer that also holds the gaps between them, and large
ones by themselves, so a buffer must never span the place of a large one.  Whether one could
depends on where the arrays end: the sizes here put the borders of the buffers (1 MB) and of
the large arrays (512 KB) before, between and behind every pair of neighbouring arrays.  The
plan check builds the copies on the host and compares them with the arrays, byte for byte.
On the GPU a lost array shows in the operator and the solve (the SpMM's row list above all).
"""
import numpy as np
import pytest

import gen
from oracle import erc as OE
from oracle import graph as OG

torch = pytest.importorskip("torch")


def _tree(n, chords, weighted, seed):
    """A random recursive tree with `chords` more edges."""
    rng = np.random.default_rng(seed)
    v = np.arange(1, n)
    u = (rng.random(n - 1) * v).astype(np.int64)
    a, b = rng.integers(0, n, chords), rng.integers(0, n, chords)
    u, v = np.concatenate([u, a[a != b]]), np.concatenate([v, b[a != b]])
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32) if weighted else None
    return gen.from_edges(n, u, v, w)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("weighted", [False, True])
def test_copies_bring_every_array(dtype, weighted):
    import paper_2609_27209_amd as E
    from paper_2609_27209_amd import _abi
    # 32,769 to 43,700 nodes: the row list is large, its neighbours are small
    shapes = [(n, c) for n in (32768, 32769, 33000, 36000, 40000, 43000, 43690, 43700, 65535, 65536, 66000)
              for c in (0, 5000, 20000, 40000)]
    shapes += [(n, c) for n in (1, 2, 500, 2000, 8000, 16384, 21000, 30000) for c in (0, 3 * n, 9 * n)]
    for n, c in shapes:
        g = _tree(n, c, weighted, n + c)
        d, keep = E._desc(g.rowptr, g.col, g.w, dtype)
        _abi.erc_debug_check_plan(d)
        del keep


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [33000, 43000])
def test_operator_and_solve_on_weighted_trees(n, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_27209_amd as E
    g = _tree(n, 0, True, n)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    delta = 0.5
    X = np.random.default_rng(n).standard_normal((n, 16)).astype(np.float32 if dtype == "f32" else np.float64)
    Y = G.debug_spmm(delta, torch.from_numpy(X)).cpu().numpy().astype(np.float64)
    L = OG.laplacian(g)
    X = X.astype(np.float64)
    scale = abs(L) @ np.abs(X) + delta * np.abs(X)
    eps = 2.0 ** -24 if dtype == "f32" else 2.0 ** -53
    # each output is a sum of deg + 1 terms in the working precision
    assert np.all(np.abs(Y - OE.laplacian_apply(L, delta, X)) <= 4 * eps * (np.diff(g.rowptr)[:, None] + 2) * scale)
    tol, bar = (1e-6, 1e-4) if dtype == "f32" else (1e-10, 1e-9)
    R, info = G.resistance(4, 4, delta, tol, 10000, 3)
    ref, _ = OE.resistance(g, 4, 4, delta, tol, 10000, 3, dtype)
    assert info["cols_unconverged"] == 0 and info["breakdowns"] == 0
    assert np.max(np.abs(R.cpu().numpy() - ref) / ref) <= bar


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_positions_for_long_rows_only_where_there_are_any(dtype):
    """Two bytes per entry, which only rows of more than 128 entries read."""
    import paper_2609_27209_amd as E
    from paper_2609_27209_amd import _abi
    n, k = 3000, 127
    ring = np.arange(n)
    size = []
    for at in (0, 1):  # node 0 with 2 + 126 and with 2 + 127 entries, as many entries in all
        u = np.concatenate([ring, np.full(k - 1 + at, 0), np.arange(1, 2 - at)])
        v = np.concatenate([(ring + 1) % n, 100 + np.arange(k - 1 + at), 1000 + np.arange(1, 2 - at)])
        g = gen.from_edges(n, u, v)
        assert g.nnz == 2 * (n + k) and np.diff(g.rowptr).max() == 128 + at
        d, keep = E._desc(g.rowptr, g.col, g.w, dtype)
        size.append(_abi.erc_graph_bytes(d))
        del keep
    assert size[1] - size[0] == -(-2 * g.nnz // 256) * 256

"""Row sums of R (p_u) and of kappa (node probabilities), four rows per wavefront.

Rows of 0, 1, 15 to 17 and 63 to 65 entries, of 255 to 257 (above 256 a whole wavefront takes
the row) and of 1023 to 1025, mixed within a wavefront's four; node counts around a wavefront's four
rows, a block's 16 and the 32,768 rows from which runs of rows go to one XCD.

Tolerance: a row of d entries is a sum of d terms of a few roundings each, in any order within
(d + 8) 2^-53 times the sum of their magnitudes; p and the node weights round once more, and
the node probabilities divide by a total within (n + d) 2^-53 of its own.
"""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_27209_amd as E
    return E


def _graph(n, degrees, weighted, seed):
    """Hubs of the given degrees among the first nodes, then pairs; ids shuffled, the rest isolated."""
    rng = np.random.default_rng(seed)
    us, vs = [], []
    h = len(degrees)
    for i, d in enumerate(degrees):
        us.append(np.full(d, i))
        vs.append(h + rng.choice(n - h, d, replace=False))
    if n >= 32000:
        k = np.arange(h, n - n // 8)
        us.append(k)
        vs.append(h + (k - h + 1 + rng.integers(0, n - h - 2, k.size)) % (n - h))
    u, v = np.concatenate(us), np.concatenate(vs)
    keep = u != v
    perm = rng.permutation(n)
    u, v = perm[u[keep]], perm[v[keep]]
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32) if weighted else None
    return gen.from_edges(n, u, v, w)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,degrees", [(2, [1]), (3, [2]), (4, [2]), (5, [1, 2]), (15, [7]), (16, [14]), (17, [15, 1]),
                                       (33, [15, 16, 17]), (150, [63, 64, 65, 1]), (700, [255, 256, 257]),
                                       (2500, [1023, 1024, 1025, 257, 256]), (32767, [300, 20000]),
                                       (32768, [257]), (32769, [256]), (34833, [4000])])
def test_row_sums(n, degrees, weighted):
    E = _gpu()
    g = _graph(n, degrees, weighted, n)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype="f64")
    eu, ev = (x.cpu().numpy() for x in G.edge_endpoints())
    rng = np.random.default_rng(1)
    R = rng.uniform(0.1, 1.0, eu.size)
    deg = np.diff(g.rowptr)
    rows = np.repeat(np.arange(n), deg)
    wt = np.ones(rows.size) if g.w is None else np.asarray(g.w, dtype=np.float64)
    lo, hi = np.minimum(rows, g.col), np.maximum(rows, g.col)
    eid = np.searchsorted(eu.astype(np.int64) * n + ev, lo.astype(np.int64) * n + hi)
    s = np.bincount(rows, weights=wt * R[eid], minlength=n)
    p, _ = G.curvature(torch.from_numpy(R).cuda())
    assert np.all(np.abs(p.cpu().numpy() - (1 - 0.5 * s)) <= 2.0 ** -53 * ((deg + 8) * s + 2))
    kappa = rng.uniform(-3.0, 2.0, eu.size)
    eta = 1e-3
    pn, _ = G.sampling_probs(torch.from_numpy(kappa).cuda(), eta)
    t = (kappa - kappa.min()) / (kappa.max() - kappa.min() + eta)
    c = np.bincount(rows, weights=t[eid], minlength=n)
    want = c / c.sum() if c.sum() > 0 else None
    pn = pn.cpu().numpy()
    if want is not None:
        assert np.all(np.abs(pn - want) <= 2.0 ** -53 * (2 * deg + n + deg.max() + 24) * want)
        assert np.all(pn[deg == 0] == 0)

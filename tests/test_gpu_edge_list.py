"""The per-edge kernels over the edge list, at edge counts around a wavefront (64) and a block
(256) and at every block width: R against the squared row differences of the same solve's Z
(erc_debug_solve_block) in fp64, and kappa against Eq. 2 on the same R.

Tolerance: R_e sums at most 256 fp64 squares whose terms are exact to one rounding, so two
summation orders differ by at most 256 x 2^-52 relative; kappa adds a few roundings to
2 (p_u + p_v) / R_e, relative to 2 (|p_u| + |p_v|) / R_e."""
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


@pytest.mark.parametrize("dtype,k", [("f32", 9), ("f32", 32), ("f32", 64), ("f32", 128), ("f32", 256),
                                     ("f64", 5), ("f64", 16), ("f64", 32), ("f64", 64), ("f64", 128)])
@pytest.mark.parametrize("m", [1, 3, 63, 64, 65, 255, 256, 257, 700])
def test_edge_distances_and_curvature(m, dtype, k):
    E = _gpu()
    rng = np.random.default_rng(m)
    n = max(3, m // 3 + 2)
    pairs = set()
    while len(pairs) < m:
        a, b = sorted(rng.integers(0, n, 2))
        if a != b:
            pairs.add((int(a), int(b)))
        if len(pairs) == n * (n - 1) // 2:
            n += 1
    u, v = np.array(sorted(pairs)).T
    g = gen.from_edges(n, u, v)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    args = dict(delta=1e-3, tol=1e-4, seed=11)
    Z, _, _ = G.debug_solve_block(k, k, args["delta"], args["tol"], args["seed"], 0, k)
    R, _ = G.resistance(k, k, **args)
    z = Z.cpu().numpy().astype(np.float64)
    eu, ev = (x.cpu().numpy() for x in G.edge_endpoints())
    np.testing.assert_array_equal(eu, u)
    np.testing.assert_array_equal(ev, v)
    want = ((z[eu] - z[ev]) ** 2).sum(1)
    R = R.cpu().numpy()
    np.testing.assert_allclose(R, want, rtol=256 * 2.0 ** -52, atol=0)
    # accumulation: twice the same columns
    R2 = torch.from_numpy(R).cuda().clone()
    G.resistance(k, k, out=R2, accumulate=True, **args)
    np.testing.assert_allclose(R2.cpu().numpy(), 2 * R, rtol=4 * 2.0 ** -52, atol=0)
    p, kappa = (x.cpu().numpy() for x in G.curvature(torch.from_numpy(R).cuda()))
    scale = 2 * (np.abs(p[eu]) + np.abs(p[ev])) / R
    assert np.max(np.abs(kappa - 2 * (p[eu] + p[ev]) / R) / scale) <= 8 * 2.0 ** -52

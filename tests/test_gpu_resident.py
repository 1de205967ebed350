"""The resident CG (one workgroup per column, small graphs) against the block kernels.

With profile=True (ERC_PROFILE_SPMM) a solve runs the block kernels whatever the graph's
size, so both paths solve the same right-hand sides.  The sizes sit at the edges of the
resident plan: one and two rows, a row more or less than a slice (64), than a workgroup (512
and 1024 threads) and than the largest fp32 and fp64 forms, rows of kResHeavy (128) entries
and one more, rows of several chunks, isolated rows, and q inside and outside the LDS.

Tolerance: the bars of the parity tests against the oracle, 1e-9 (fp64) and 1e-4 (fp32)
relative on R; the two paths' rounding differs in the order of row sums, in fp32 also in their
precision (fours added in fp64) and in beta (the reduced r.r against its expansion).  Plain CG in fp64 has to give the same solutions:
rows of up to 32 entries are summed in one order by both and beta has one form, and graphs with
longer rows take the block kernels.  R then differs only in the grouping of its 21 columns'
sum of squares, two orders of which are within 2 x 21 x 2^-53 of each other.
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


def _ring(n, weighted, seed, extra=3.0, isolated=0):
    """A ring on n - isolated nodes with extra * n random chords, ids shuffled."""
    rng = np.random.default_rng(seed)
    k = n - isolated
    u = np.arange(k)
    v = (u + 1) % k
    a, b = rng.integers(0, k, int(extra * k)), rng.integers(0, k, int(extra * k))
    u, v = np.concatenate([u, a]), np.concatenate([v, b])
    perm = rng.permutation(n)
    keep = u != v
    u, v = perm[u[keep]], perm[v[keep]]
    w = rng.uniform(0.5, 2.0, u.size).astype(np.float32) if weighted else None
    return gen.from_edges(n, u, v, w)


def _hubs(n, degrees, weighted, seed):
    """A sparse ring plus hubs of the given extra degrees."""
    rng = np.random.default_rng(seed)
    us, vs = [np.arange(n)], [(np.arange(n) + 1) % n]
    for h, d in enumerate(degrees):
        t = rng.choice(n, d, replace=False)
        us.append(np.full(d, 7 * h))
        vs.append(t)
    u, v = np.concatenate(us), np.concatenate(vs)
    keep = u != v
    w = rng.uniform(0.5, 2.0, int(keep.sum())).astype(np.float32) if weighted else None
    return gen.from_edges(n, u[keep], v[keep], w)


CASES = {
    "two_rows": lambda wt: gen.path_graph(2, None if not wt else np.array([1.5], np.float32)),
    "degrees_31_to_33": lambda wt: _hubs(3000, [29, 30, 31], wt, 13),
    "degrees_to_32": lambda wt: _hubs(3000, [29, 30, 30], wt, 14),
    "n64": lambda wt: _ring(64, wt, 1),
    "n65_isolated": lambda wt: _ring(65, wt, 2, isolated=9),
    "n1025": lambda wt: _ring(1025, wt, 3),
    "n2048": lambda wt: _ring(2048, wt, 4),
    "n2049": lambda wt: _ring(2049, wt, 5),
    "long_stream_in_registers": lambda wt: _ring(2000, wt, 6, extra=14.0),
    "degrees_127_to_129": lambda wt: _hubs(3000, [125, 126, 127, 128, 129], wt, 7),
    "chunked_rows": lambda wt: _hubs(5000, [255, 256, 257, 513, 4000], wt, 8),
    "dense": lambda wt: _ring(300, wt, 9, extra=60.0),
    # the fullest LDS: p, q, a part per thread of two sums, and 240 chunk sums
    "n16384_chunked_rows": lambda wt: _hubs(16384, [4000] * 15, wt, 15),
    "n16384": lambda wt: _ring(16384, wt, 10, extra=1.0),
    "n16385": lambda wt: _ring(16385, wt, 11, extra=1.0),
    "n32768": lambda wt: _ring(32768, wt, 12, extra=1.0),
}


@pytest.mark.parametrize("precond", ["none", "jacobi"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_resident_matches_block_kernels(name, weighted, dtype, precond):
    E = _gpu()
    g = CASES[name](weighted)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    tol = 1e-6 if dtype == "f32" else 1e-10
    # 21 columns in blocks of 6 (padded 16 or 8): one resident solve, four ragged blocks
    a, ia = G.resistance(21, 6, 1e-4, tol, 4000, 5, precond=precond)
    a = a.cpu().numpy()
    a2, _ = G.resistance(21, 6, 1e-4, tol, 4000, 5, precond=precond)
    np.testing.assert_array_equal(a2.cpu().numpy(), a)
    b, ib = G.resistance(21, 6, 1e-4, tol, 4000, 5, precond=precond, profile=True)
    b = b.cpu().numpy()
    assert ia["blocks"] == ib["blocks"] == 4
    assert ia["cols_unconverged"] == ib["cols_unconverged"] == 0
    assert np.max(np.abs(a - b) / b) <= (1e-9 if dtype == "f64" else 1e-4)
    if dtype == "f64" and precond == "none":
        assert np.max(np.abs(a - b) / b) <= 42 * 2.0 ** -53


def test_resident_iteration_cap_is_reported():
    E = _gpu()
    g = _ring(3000, True, 21)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype="f32")
    _, i3 = G.resistance(16, 16, 1e-4, 1e-6, 3, 5, raise_not_converged=False)
    assert i3["iters_max"] == 3 and i3["iters_total"] == 48 and i3["cols_unconverged"] == 16
    assert i3["max_final_relres"] > 1e-6


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,extra", [(2000, 4.0), (3000, 25.0), (3000, 50.0), (12000, 4.0)])
def test_fp32_rounds_no_worse_than_block_kernels(n, extra, weighted):
    """Against the fp64 solve of the same system, in the 2-norm over all edges: the fp32
    resident solve may not lie further off than the block kernels do (both are rounding of
    the same recurrence; sums of rows of 33 to 128 entries as one fp32 chain had made it 1.7
    times as far).  One realisation's norm over tens of thousands of edges is within a few per
    cent of its mean, so a fifth more is no chance."""
    E = _gpu()
    g = _ring(n, weighted, 31, extra=extra)
    kw = dict(K=64, k_block=16, delta=1e-5, tol=1e-6, seed=3)
    ref, _ = E.Graph(g.rowptr, g.col, g.w, solve_dtype="f64").resistance(**kw)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype="f32")
    res, _ = G.resistance(**kw)
    res = float((res - ref).norm() / ref.norm())
    blk, _ = G.resistance(profile=True, **kw)
    blk = float((blk - ref).norm() / ref.norm())
    print(f"n={n} extra={extra} weighted={weighted}: resident {res:.2e}, block kernels {blk:.2e}")
    assert res <= 1.2 * blk


def _one_launch(info):
    """A resident solve counts the iterations it took; the block kernels enqueue iterations a
    group ahead of the host's poll."""
    return info["launches"] == info["spmm_full"]


@pytest.mark.parametrize("n,extra,weighted,dtype,narrow", [
    (16000, 29.0, True, "f32", True), (24000, 40.0, False, "f32", False), (30000, 15.3, True, "f32", False),
    (8000, 19.5, True, "f64", True), (16000, 10.0, True, "f64", False), (16000, 45.0, False, "f64", False)])
def test_solver_by_cost_and_columns(n, extra, weighted, dtype, narrow):
    """The larger of the graphs with a resident plan take it for wide blocks or several only
    (kResNarrow32, kResNarrow64, kResWide); all routes agree."""
    E = _gpu()
    g = _ring(n, weighted, 41, extra=extra)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    tol, bar = (1e-6, 1e-4) if dtype == "f32" else (1e-10, 1e-9)
    kw = dict(delta=1e-3, tol=tol, seed=3, precond="jacobi")
    ref, ip = G.resistance(128, 64, profile=True, **kw)
    assert not _one_launch(ip)
    one, i1 = G.resistance(128, 128, **kw)
    two, i2 = G.resistance(128, 64, **kw)
    # the same columns in calls of one block each
    acc, ia = G.resistance(128, 64, col_end=64, **kw)
    acc = acc.clone()
    _, ib = G.resistance(128, 64, col_begin=64, out=acc, accumulate=True, **kw)
    assert _one_launch(i1) and _one_launch(i2)
    assert _one_launch(ia) == _one_launch(ib) == narrow
    for x in (one, two, acc):
        assert float(((x - ref).abs() / ref).max()) <= bar
    _, i3 = G.resistance(128, 16, col_end=48, **kw)  # three blocks of 16
    assert _one_launch(i3)
    _, i4 = G.resistance(128, 64, col_end=1, **kw)
    assert _one_launch(i4) == narrow

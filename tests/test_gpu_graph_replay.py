"""Replaying captured groups of CG iterations (HIP graphs) gives the same bits as
launching every kernel separately, and fails loudly on non-finite curvature.

Each solve replays its captured group several times per block, with the host's
convergence polls (stream synchronisations) between the replays; repeated solves on
the same handle reuse the cached graph.  Every replayed run is compared bit for bit
with a run that enqueues each launch on its own (ERC_NO_GRAPH), and with the oracle at
the path's tolerance.  The shapes cover fp64 and fp32, unit and weighted graphs, one
and several blocks, and rows split over several blocks of the SpMM (the hub rows of a
Chung-Lu graph, finished by their own launch).

Graphs of up to 32,768 nodes (16,384 in fp64) are solved by a single launch, on which these
flags change nothing: the cases of SMALL check just that.  Those of LARGE are above that
size, so that their iterations are launches, captured, replayed and stopped early; each
run of one asserts it (iterations are enqueued a group ahead of the host's poll, where a single
launch counts the iterations it took).
"""
import numpy as np
import pytest

import gen
from oracle import erc as OE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_27209_amd as E
    return E


SMALL = {
    # name: (graph, dtype, K, k_block, delta, tol)
    "er2k_f64": (lambda: gen.make_graph("er2k"), "f64", 32, 32, 1e-6, 1e-8),
    "sbm20k_f32": (lambda: gen.make_graph("sbm20k"), "f32", 64, 64, 1e-5, 1e-6),
    "sbm2k_f32_blocks": (lambda: gen.make_graph("sbm2k"), "f32", 160, 64, 1e-5, 1e-6),
    # 10,000 nodes, one row of 7554 entries split over two SpMM blocks, 394 isolated
    "chung_lu_split_hubs": (lambda: gen.chung_lu(n=10000, gamma=2.0, i0=0.2, m_target=50000,
                                                 seed=18, weighted=True),
                            "f32", 48, 16, 1e-4, 1e-6),
}
LARGE = {
    # two correct fp64 runs differ by about the error left at the stop, which falls with tau: the
    # oracle and the GPU by 2.9e-8 of R at tau = 1e-9 here, so by 3e-11 at 1e-12 (bar: 1e-9)
    "cl17k_f64": (lambda: gen.chung_lu(n=17000, gamma=3.0, i0=2000.0, m_target=70000, seed=3,
                                       weighted=True), "f64", 16, 16, 1e-2, 1e-12),
    "cl40k_f32": (lambda: gen.chung_lu(n=40000, gamma=2.6, i0=400.0, m_target=160000, seed=4,
                                       weighted=True), "f32", 8, 8, 1e-1, 1e-6),
    "cl33k_unit_blocks": (lambda: gen.chung_lu(n=33000, gamma=2.6, i0=400.0, m_target=120000, seed=5),
                          "f32", 12, 5, 1e-2, 1e-6),
    # rows above 4096 entries are split over several SpMM blocks
    "cl34k_split_hubs": (lambda: gen.chung_lu(n=34000, gamma=2.0, i0=0.2, m_target=140000, seed=6,
                                              weighted=True), "f32", 4, 2, 1e-1, 1e-6),
}
CASES = {**SMALL, **LARGE}
_GRAPHS = {}


def _make(name):
    if name not in _GRAPHS:
        _GRAPHS[name] = CASES[name][0]()
    return _GRAPHS[name]


def _launched(name, *infos):
    """The solves enqueued their iterations exactly where the case is a large one."""
    for i in infos:
        assert (i["launches"] > i["spmm_full"]) == (name in LARGE), name


@pytest.mark.parametrize("name", sorted(CASES))
def test_graph_replay_matches_separate_launches(name):
    E = _gpu()
    _, dtype, K, kb, delta, tol = CASES[name]
    g = _make(name)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    R0, i0 = G.resistance(K, kb, delta, tol, 10000, 17, graph=False)
    _launched(name, i0)
    ref = R0.cpu().numpy()
    assert i0["cols_unconverged"] == 0 and i0["breakdowns"] == 0
    for rep in range(3):
        R1, i1 = G.resistance(K, kb, delta, tol, 10000, 17)
        torch.cuda.synchronize()
        _launched(name, i1)
        assert i1["iters_total"] == i0["iters_total"], rep
        np.testing.assert_array_equal(R1.cpu().numpy(), ref)
        # eager work on the same stream between the replayed solves
        _ = G.curvature(R1)
        torch.cuda.synchronize()
    ora, _ = OE.resistance(g, K, kb, delta, tol, 10000, 17, dtype)
    rel = np.max(np.abs(ref - ora) / ora)
    assert rel <= (1e-9 if dtype == "f64" else 1e-4), rel
    print(f"{name}: {i0['iters_max']} iterations, graph replay bit-identical, oracle {rel:.2e}")


def test_split_rows_present_in_hub_case():
    """The hub cases really have rows split over several SpMM blocks (checked on the
    host plan through the C ABI's plan check, which also validates the plan)."""
    E = _gpu()
    from paper_2609_27209_amd import _abi
    for name in ("chung_lu_split_hubs", "cl34k_split_hubs"):
        g = _make(name)
        deg = np.diff(np.asarray(g.rowptr))
        assert deg.max() > 4096, "hub case lost its split rows"
        desc, keep = E._desc(g.rowptr, g.col, g.w, "f32")
        _abi.erc_debug_check_plan(desc)
        del keep


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_curvature_is_reported(bad):
    E = _gpu()
    from paper_2609_27209_amd import _abi
    g = gen.make_graph("er2k")
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype="f64")
    kappa = torch.linspace(-1.0, 1.0, G.m, dtype=torch.float64, device="cuda")
    kappa[G.m // 3] = bad
    with pytest.raises(_abi.ErcError) as ei:
        G.sampling_probs(kappa, 1e-12)
    assert ei.value.status == _abi.ERC_E_NUMERIC
    # the same call on finite input succeeds afterwards (the flag starts at zero)
    kappa[G.m // 3] = 0.0
    pn, pe = G.sampling_probs(kappa, 1e-12)
    ref_pn, ref_pe = OE.sampling_probs(g, kappa.cpu().numpy(), 1e-12)
    np.testing.assert_allclose(pn.cpu().numpy(), ref_pn, rtol=1e-12, atol=0)
    np.testing.assert_allclose(pe.cpu().numpy(), ref_pe, rtol=1e-12, atol=0)


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("precond", ["none", "jacobi"])
def test_early_stop_test_changes_nothing_but_one_spmm(name, precond):
    """The early exact stopping test after each update (ERC_EARLY_STOP; by default only
    on graphs whose SpMM gathers several GB) gives the same bits and iteration counts as
    leaving the test to the next finishing step; it saves at most one SpMM per block,
    the one that would follow the block's last update.  Both with graph replay and with
    separate launches."""
    E = _gpu()
    _, dtype, K, kb, delta, tol = CASES[name]
    g = _make(name)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    for graph in (True, False):
        R0, i0 = G.resistance(K, kb, delta, tol, 10000, 17, graph=graph, precond=precond)
        R0 = R0.cpu().numpy()
        R1, i1 = G.resistance(K, kb, delta, tol, 10000, 17, graph=graph, precond=precond,
                              early_stop=True)
        _launched(name, i0, i1)
        np.testing.assert_array_equal(R1.cpu().numpy(), R0)
        assert i1["iters_total"] == i0["iters_total"] and i1["iters_max"] == i0["iters_max"]
        assert 0 <= i0["spmm_full"] - i1["spmm_full"] <= i0["blocks"]


@pytest.mark.parametrize("name", sorted(LARGE))
def test_early_stop_saves_the_spmm_of_jacobi_blocks(name):
    """With the Jacobi variant every update is predicted to be the last, so the early test
    always saves the SpMM after a block's last update."""
    E = _gpu()
    _, dtype, K, kb, delta, tol = CASES[name]
    g = _make(name)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    _, i0 = G.resistance(K, kb, delta, tol, 10000, 17, precond="jacobi")
    _, i1 = G.resistance(K, kb, delta, tol, 10000, 17, precond="jacobi", early_stop=True)
    assert i0["spmm_full"] - i1["spmm_full"] == i0["blocks"] == -(-K // kb)


@pytest.mark.parametrize("name", sorted(LARGE))
def test_polling_interval_and_iteration_cap(name):
    """Any interval of the host's polls gives the same bits, and a cap inside a captured
    group ends the solve there and is reported."""
    E = _gpu()
    _, dtype, K, kb, delta, tol = CASES[name]
    g = _make(name)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    R0, i0 = G.resistance(K, kb, delta, tol, 10000, 17)
    R0 = R0.clone()
    for check in (1, 3, 29):
        R1, i1 = G.resistance(K, kb, delta, tol, 10000, 17, check_every=check)
        _launched(name, i1)
        assert torch.equal(R0, R1) and i1["iters_total"] == i0["iters_total"]
    _, i2 = G.resistance(K, kb, delta, tol, 10000, 17, raise_not_converged=False)
    assert i2["cols_unconverged"] == 0
    for cap in (3, 16, 18):
        assert cap < i0["iters_max"]
        _, i3 = G.resistance(K, kb, delta, 1e-14, cap, 17, raise_not_converged=False)
        assert i3["iters_max"] == cap and i3["iters_total"] == cap * K and i3["cols_unconverged"] == K


@pytest.mark.parametrize("dtype,n,kb,K", [("f32", 33000, 256, 300), ("f64", 17000, 128, 150)])
@pytest.mark.parametrize("precond", ["none", "jacobi"])
def test_widest_blocks_by_launches(dtype, n, kb, K, precond):
    """The widest blocks of the launched iterations, the last one ragged, against narrow ones:
    the widths differ in the grouping of row sums alone.  What that grouping moves is amplified
    to about the error left at the stop, which falls with tau: in fp64 4e-10 of R at tau =
    1e-10, so 4e-12 at 1e-12 (bar: 1e-10)."""
    E = _gpu()
    g = gen.chung_lu(n=n, gamma=2.6, i0=400.0, m_target=4 * n, seed=7, weighted=True)
    G = E.Graph(g.rowptr, g.col, g.w, solve_dtype=dtype)
    tol, bar = (1e-6, 1e-5) if dtype == "f32" else (1e-12, 1e-10)
    a, ia = G.resistance(K, kb, 1e-2, tol, 5000, 21, precond=precond)
    a = a.clone()
    b, ib = G.resistance(K, 32, 1e-2, tol, 5000, 21, precond=precond)
    assert ia["blocks"] == 2 and ia["cols_unconverged"] == 0
    assert ia["launches"] > ia["spmm_full"] and ib["launches"] > ib["spmm_full"]
    assert float(((a - b).abs() / b).max()) <= bar

"""The device matching by proposals against the oracle, level by level and bit
by bit, where it can go wrong: a path whose edges grow along it (one proposal
displaces the next, the longest chain there is), a path of equal edges and a
grid of them (ties by the numbers of the endpoints), a graph of hubs whose
lists are long and mostly taken, random weights on a random graph, vertices
without an eligible edge; and a hierarchy that stalls below the dense limit,
whose last level is decided on the device.  The options that stop the coarsening
there (levels, sizes, ratio, with and without composition) against the host."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2210_16660_amd as pamg
from workloads import CSR, lap7, varcoef7

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


def laplacian(n, edges, weights, shift=1.0):
    """Graph Laplacian of positive edge weights plus a diagonal shift."""
    lo, hi = np.minimum(edges[:, 0], edges[:, 1]), np.maximum(edges[:, 0], edges[:, 1])
    U = sp.csr_matrix((-weights, (lo, hi)), shape=(n, n))
    A = (U + U.T + sp.diags(np.asarray(-(U + U.T).sum(axis=1)).ravel() + shift)).tocsr()
    A.sort_indices()
    M = CSR(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), np.ascontiguousarray(A.data, dtype=np.float64))
    M.check()
    return M


def path(n, growth):
    i = np.arange(n - 1)
    return laplacian(n, np.stack([i, i + 1], axis=1), 1.0 + growth * i)


def hubs(n, count, seed):
    rng = np.random.default_rng(seed)
    leaf = np.arange(count, n)
    edges = np.concatenate([np.stack([leaf % count, leaf], axis=1), np.stack([leaf[:-1], leaf[1:]], axis=1)])
    weights = rng.uniform(0.5, 2.0, len(edges))
    weights[:len(leaf)] *= 40.0
    return laplacian(n, edges, weights)


def random_graph(n, degree, seed, isolated=0):
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n - isolated, size=(n * degree // 2, 2))
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    return laplacian(n, e, rng.uniform(0.1, 10.0, len(e)))


CASES = {
    "growing_path": lambda: path(9000, 1e-2),
    "shrinking_path": lambda: path(9000, -1e-4),
    "equal_path": lambda: path(9001, 0.0),
    "equal_grid": lambda: lap7(21),
    "hubs": lambda: hubs(9500, 64, 3),
    "random": lambda: random_graph(8300, 9, 5),
    "isolated": lambda: random_graph(8500, 6, 6, isolated=50),
    "stalled": lambda: varcoef7(22, seed=5000),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_matching_is_the_oracles(case):
    A = CASES[case]()
    H = pamg.Hierarchy(A, device_setup=1)
    O = oracle.Hierarchy(A, max_coarse=200, max_dense=8192)
    print(case, "device levels", H.info().device_levels, "of", H.levels, flush=True)
    assert H.info().device_levels >= 3
    assert H.levels == O.nlevels
    for l in range(H.levels - 1):
        assert np.array_equal(H.aggregates(l), O.agg(l)), f"level {l} aggregates differ"
    for l in range(H.levels):
        rp, ci, v = H.level_csr(l)
        orp, oci, ov = O.level(l)
        assert np.array_equal(rp, orp) and np.array_equal(ci, oci), f"level {l} pattern differs"
        assert np.array_equal(v.view(np.uint64), ov.view(np.uint64)), f"level {l} values differ"


STOPS = [{"max_levels": 2}, {"max_levels": 4}, {"max_coarse": 3000}, {"min_ratio": 1.9}, {"min_ratio": 3.0},
         {"max_levels": 3, "agg_steps": 2}, {"max_coarse": 700, "agg_steps": 3}, {"min_ratio": 1.9, "agg_steps": 2}]


@pytest.mark.parametrize("kw", STOPS, ids=str)
@pytest.mark.parametrize("make", [lambda: lap7(22), lambda: varcoef7(22, seed=11)], ids=["lap7", "varcoef"])
def test_coarsening_stops_where_the_hosts_does(make, kw):
    A = make()

    def build(device):
        try:
            return pamg.Hierarchy(A, device_setup=device, **kw)
        except pamg.PamgError as e:
            return e.code

    D, R = build(1), build(0)
    if isinstance(R, int):
        assert D == R
        return
    assert D.levels == R.levels and R.info().device_levels == 0
    for l in range(D.levels):
        for a, b in zip(D.level_csr(l), R.level_csr(l)):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), l
    for l in range(D.levels - 1):
        assert np.array_equal(D.aggregates(l), R.aggregates(l)), l

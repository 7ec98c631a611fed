"""The FP64 form of the Panther++ search at the edges of its kernels: tiles of
8 queries, 8 coordinates staged a step, rounds of 1,024 rows, one slice per
4,096 rows while the queries leave the chip idle, and merges of more than the
1,024 pairs that the merge sorts at a time.  Ids and distances equal the
oracle's bit for bit (the same chain of fused multiply-adds and the same total
order, so no tolerance)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _equal(P, oracle, theta, q, D, k, what):
    print(f"case: fp64 knn {what} D={D} nq={len(q)} k={k}", flush=True)
    ids, dist = P.pp_topk(q, D, k)
    uq, inv = np.unique(q, return_inverse=True)
    wi, wd = oracle.knn(theta, uq, k)
    assert (ids == wi[inv]).all()
    assert (dist.view(np.uint64) == np.ascontiguousarray(wd)[inv].view(np.uint64)).all()


def _setup(oracle, inputs, n, R, isolated=0):
    """n vertices, the last `isolated` of them without an edge (zero rows)."""
    from paper_1504_02577_amd.panther import Panther

    rng = np.random.default_rng(n)
    top = n - isolated
    g = inputs.graph_from_edges(n, np.concatenate([[[0, 1]], rng.integers(0, top, (4 * top, 2))]),
                                rng.integers(1, 50, 4 * top + 1))
    T, seed = 5, 3
    paths = oracle.walk(g, T, R, seed)
    ptr, pid = oracle.index(g.n, paths)
    P = Panther(0)
    P.load_graph(g)
    P.sample_paths(T, R, seed)
    P.set_option("pp.form", 0)
    return P, rng, lambda D: oracle.features(g.n, paths, ptr, pid, D)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 4095, 4096, 4097, 8193])
def test_tile_edges(oracle, inputs, n):
    P, rng, features = _setup(oracle, inputs, n, 4 * n, isolated=n // 3)
    for D in (1, 7, 8, 9, 64):
        theta = features(D)
        for nq, k in ((1, 256), (7, 10), (8, 63), (9, 64), (15, 65), (17, 1)):
            _equal(P, oracle, theta, rng.integers(0, n, nq).astype(np.int32), D, k, f"n={n}")
    P.close()


# n = 131,072 gives 32 slices for few queries; the slices' pairs of a query:
# 2,560 (10 slices x 256), 4,096 (16 x 256), 1,024 and 1,056 (32 and 33 x 32)
@pytest.mark.parametrize("n,nq,k", [(40_000, 8, 256), (131_072, 1, 256), (131_072, 9, 32),
                                    (131_073, 9, 32), (131_073, 9, 1), (131_072, 301, 200)])
def test_merges(oracle, inputs, n, nq, k):
    """Half of the vertices are isolated, so that queries among them have more
    equal distances than any k."""
    P, rng, features = _setup(oracle, inputs, n, 2 * n, isolated=n // 2)
    D = 9
    theta = features(D)
    q = rng.integers(0, n // 2, nq).astype(np.int32)
    q[::3] = rng.integers(n // 2, n, len(q[::3]))
    if nq > 100:  # the oracle scans every row per query
        q = rng.choice(q[:24], nq)
    _equal(P, oracle, theta, q, D, k, f"n={n}")
    P.close()


def test_more_queries_than_rows(oracle, inputs):
    """40,000 queries in one launch, a slice each."""
    n = 1500
    P, rng, features = _setup(oracle, inputs, n, 4 * n, isolated=100)
    _equal(P, oracle, features(65), rng.integers(0, n, 40_000).astype(np.int32), 65, 10, f"n={n}")
    P.close()

"""Walk kernels at the edges of their launch: the lanes of a quad load each
other's guide records, so path counts that leave a quad, a wavefront or a
work-group partly empty, weightless rows (no record) and rows that end inside
a record are walked at every path length class and both weight widths."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _graph(inputs, wide):
    # a hub of degree 300 with skewed weights, a chain, zero-weight entries,
    # a row of weight zero only, and isolated vertices (the last ones too)
    edges = [(0, i) for i in range(1, 301)] + [(i, i + 1) for i in range(1, 340)] + [(345, 346)]
    rng = np.random.default_rng(5)
    w = rng.integers(1, 1000, len(edges))
    w[:300:7] = 100_000
    w[5:300:11] = 0
    w[-1] = 0
    if wide:
        w = w * 42_000  # row sums past 2^32
    return inputs.graph_from_edges(350, edges, w.astype(np.uint32))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("start_all", [False, True])
def test_walk_edges(oracle, inputs, wide, start_all):
    from paper_1504_02577_amd.panther import PANTHER_START_ALL_VERTICES, Panther

    g = _graph(inputs, wide)
    assert (oracle.row_weights(g).max() >= 1 << 32) == wide
    P = Panther(0)
    P.load_graph(g, flags=PANTHER_START_ALL_VERTICES if start_all else 0)
    for T in (1, 3, 5, 9, 20, 63):
        for R in (1, 2, 3, 5, 63, 66, 255, 257, 5001):
            print(f"case: walk wide={wide} start_all={start_all} T={T} R={R}", flush=True)
            P.sample_paths(T, R, 40 + R)
            want = oracle.walk(g, T, R, 40 + R, start_all=start_all)
            assert (P.paths() == want).all(), (T, R)
    P.close()


def test_walk_without_edges(oracle, inputs):
    """Every vertex isolated: no guide record at all, the walk stays put."""
    from paper_1504_02577_amd.panther import PANTHER_START_ALL_VERTICES, Panther

    print("case: walk without edges", flush=True)
    g = inputs.Graph(n=7, row_ptr=np.zeros(8, np.int32), col=np.zeros(0, np.int32),
                     w=np.zeros(0, np.uint32))
    P = Panther(0)
    P.load_graph(g, flags=PANTHER_START_ALL_VERTICES)
    P.sample_paths(5, 130, 3)
    paths = P.paths()
    assert (paths == paths[:, :1]).all() and set(paths[:, 0]) <= set(range(7))
    P.close()

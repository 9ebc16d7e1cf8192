"""The device side of an edit batch at its edges: a leaf painted many times in
one batch keeps its last payload, and a link rebuild whose frontier outgrows
the kept lists (2^18 nodes) gives the records of a fresh upload."""
import numpy as np
import pytest

from canvasgen import LEAF, LEAF_DTYPE, LEAF_F64, LEAF_RGBA8_F16, NONE, Canvas, StrokeSet
from canvasgen import build_from_strokes, trees

from editmodel import COARSEN, PAINT, REFINE

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    s = Session(0)
    yield s
    s.close()


def _payloads(rng, n, fmt):
    p = np.zeros(n, LEAF_DTYPE[fmt])
    if fmt == LEAF_F64:
        for k in ("r", "g", "b", "kappa"):
            p[k] = rng.uniform(0.0, 1.0, n)
    else:
        for k in "rgba":
            p[k] = rng.integers(0, 256, n)
        p["kappa"] = rng.uniform(0.0, 4.0, n).astype(np.float16).view(np.uint16)
    return p


@pytest.mark.parametrize("fmt", [LEAF_RGBA8_F16, LEAF_F64])
@pytest.mark.parametrize("n", [1, 63, 5000])
def test_last_paint_of_a_batch_stays(sess, fmt, n):
    from paper_1704_02724_amd import cvx
    cv = trees.random_tree(1, 4, seed=33, max_nodes=600, leaf_format=fmt)
    sess.upload(0, cv)
    rng = np.random.Generator(np.random.PCG64(34 + n))
    leaves = np.nonzero(cv.nodes[:, 0] >= LEAF)[0]
    leaves = leaves[leaves >= 8]
    for _ in range(3):  # the marks of one batch are below those of the next
        node = rng.choice(leaves[:40], n)
        pays = _payloads(rng, n, fmt)
        order = rng.permutation(n)  # payload indices in any order
        sess.edit(0, [(PAINT, int(node[j]), int(order[j])) for j in range(n)], pays)
        got = cvx.cvx_read_payloads(sess.ctx, 0, LEAF_DTYPE[fmt])
        for i in np.unique(node):
            last = order[np.nonzero(node == i)[0][-1]]
            assert got[i] == pays[last]


def test_frontier_beyond_the_kept_lists(sess):
    """Root 0 of 8 is a leaf; its three face neighbours are refined to depth 7
    inside a sphere each, so refining it walks frontiers of about 400,000."""
    from paper_1704_02724_amd import cvx
    c = np.array([[0.75, 0.25, 0.25], [0.25, 0.75, 0.25], [0.25, 0.25, 0.75]])
    r = 0.24
    st = StrokeSet(np.full(3, r), np.full((3, 3), 0.5), np.full(3, 2.0), np.arange(4),
                   np.concatenate([c, np.full((3, 1), r)], axis=1))
    cv = build_from_strokes(st, 2, 7, 50.0, LEAF_RGBA8_F16)
    assert cv.nodes[0, 0] >= LEAF
    refined_at_6 = (cv.stats["leaf_depth_hist"][7]) // 8
    assert refined_at_6 > 1 << 18
    sess.upload(0, cv)
    n0 = cv.n_nodes
    start = cvx.cvx_read_records(sess.ctx, 0)
    rng = np.random.Generator(np.random.PCG64(5))
    pays = _payloads(rng, 9, LEAF_RGBA8_F16)
    first = sess.edit(0, [(REFINE, 0, 0)], pays)
    assert first[0] == n0
    nodes = np.concatenate([cv.nodes, np.zeros((8, 2), np.uint32)])
    nodes[0, 0] = n0
    nodes[n0:, 0] = LEAF | (cv.n_leaves + np.arange(8))
    nodes[n0:, 1] = 0
    nodes[0, 1] = NONE
    sess.upload(1, Canvas(nodes, np.concatenate([cv.leaves, pays[:8]]), 2, 7, LEAF_RGBA8_F16))
    np.testing.assert_array_equal(cvx.cvx_read_records(sess.ctx, 0),
                                  cvx.cvx_read_records(sess.ctx, 1))
    sess.edit(0, [(COARSEN, 0, 8)], pays)
    np.testing.assert_array_equal(cvx.cvx_read_records(sess.ctx, 0, 0, n0), start)
    sess.free(0)
    sess.free(1)

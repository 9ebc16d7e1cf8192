"""Edits around the size up to which one workgroup applies a batch, against the
host model, and a small batch whose links outgrow that workgroup's lists."""
import numpy as np
import pytest

from canvasgen import LEAF, LEAF_DTYPE, LEAF_F64, LEAF_RGBA8_F16, StrokeSet
from canvasgen import build_from_strokes, make_view, trees

from editmodel import COARSEN, PAINT, REFINE, PoolModel

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


def _same_as_upload(sess, model, fmt):
    """Records, payloads of the leaves, and a frame that reads the top-level table."""
    from paper_1704_02724_amd import cvx
    cv = model.canvas()
    sess.upload(1, cv)
    a, b = (cvx.cvx_read_records(sess.ctx, i) for i in (0, 1))
    np.testing.assert_array_equal(a, b)
    leaf = (b[:, 0] & 1 == 1) & (b[:, 0] != 0xFFFFFFFF)
    a, b = (cvx.cvx_read_payloads(sess.ctx, i, LEAF_DTYPE[fmt])[leaf] for i in (0, 1))
    assert a.tobytes() == b.tobytes()
    c = 0.5 * cv.R * cv.root_edge
    variant = "fp32_rebased" if fmt == LEAF_RGBA8_F16 else "fp64_plain"
    a, b = (sess.render([make_view((c, c, -2.0 * c), (0.0, 0.0, 1.0), 0.9, 32, 32, canvas_id=i)],
                        variant).cpu().numpy() for i in (0, 1))
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("fmt", [LEAF_RGBA8_F16, LEAF_F64])
@pytest.mark.parametrize("n", [1, 8, 511, 512, 513])
def test_batch_against_the_model(sess, n, fmt):
    cv = trees.random_tree(2, 7, seed=61, p_split=0.5, max_nodes=9000, leaf_format=fmt)
    sess.upload(0, cv)
    model = PoolModel(cv)
    rng = np.random.Generator(np.random.PCG64(62 + n))
    leaves = np.array([i for i in sorted(model.leaves_list()) if model.state[i] < 7])
    pick = rng.choice(leaves, n, replace=False)
    pays = _payloads(rng, 8 * n + 64, fmt)
    do = [(REFINE, int(i), 8 * k) for k, i in enumerate(pick)]
    first = sess.edit(0, do, pays)
    np.testing.assert_array_equal(first, model.apply(do, pays))
    _same_as_upload(sess, model, fmt)
    # half of them merged again, one of these refined once more, leaves painted
    # twice, all in one batch
    undo = [(COARSEN, int(i), 8 * k) for k, i in enumerate(pick[:(n + 1) // 2])]
    undo += [(REFINE, int(pick[0]), 1), (PAINT, int(first[-1]) + 3 if n > 1 else int(pick[0]), 5)][
        :2 if n > 1 else 1]
    other = np.setdiff1d(leaves, pick)[:20]
    undo += [(PAINT, int(i), 8 * n + int(k)) for k, i in enumerate(np.concatenate([other, other]))]
    sess.edit(0, undo, pays)
    model.apply(undo, pays)
    _same_as_upload(sess, model, fmt)


def test_links_beyond_the_workgroups_lists(sess):
    """One refined root next to three spheres: frontiers above 2,048 nodes, from
    some level on, and within the lists of the launches per level."""
    c = np.array([[0.75, 0.25, 0.25], [0.25, 0.75, 0.25], [0.25, 0.25, 0.75]])
    st = StrokeSet(np.full(3, 0.24), np.full((3, 3), 0.5), np.full(3, 2.0), np.arange(4),
                   np.concatenate([c, np.full((3, 1), 0.24)], axis=1))
    cv = build_from_strokes(st, 2, 5, 12.0, LEAF_RGBA8_F16)
    assert cv.nodes[0, 0] >= LEAF
    assert 2 * 2048 < cv.stats["leaf_depth_hist"][5] // 8 < 1 << 18
    sess.upload(0, cv)
    model = PoolModel(cv)
    pays = _payloads(np.random.Generator(np.random.PCG64(7)), 9, LEAF_RGBA8_F16)
    for edits in ([(REFINE, 0, 0)], [(COARSEN, 0, 8)]):
        sess.edit(0, edits, pays)
        model.apply(edits, pays)
        _same_as_upload(sess, model, LEAF_RGBA8_F16)

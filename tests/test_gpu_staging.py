"""How a call's views reach the device: as kernel arguments, 16 a launch, up to
32 views, by one copy above.  At every edge of the two each view's image is
the one it has when rendered alone, in cvx_render (eager and replayed) and
cvx_render_noalloc, and a smaller call after a larger one sees none of it."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    s = Session(0)
    for i in range(3):
        s.upload(i, trees.random_tree(1 + i, 5, seed=91 + i, max_nodes=3000,
                                      leaf_format=LEAF_RGBA8_F16))
    yield s
    s.close()


def _views(n):
    rng = np.random.Generator(np.random.PCG64(n))
    vs, off = [], 0
    for j in range(n):
        e = rng.uniform(0.1, 0.9, 3) if j % 3 else rng.uniform(1.2, 1.6, 3)
        w, h = 5 + j % 13, 4 + j % 9
        vs.append(make_view(e, rng.uniform(0.3, 0.7, 3) - e, 0.7, w, h, canvas_id=j % 3,
                            out_offset_px=off, alpha_stop=1.0 if j % 4 else 0.9))
        off += w * h
    return vs


@pytest.mark.parametrize("n", [64, 33, 32, 31, 17, 16, 15, 1])
def test_views_at_the_edges(sess, n):
    views = _views(n)
    alone = np.concatenate([sess.render([dict(v, out_offset_px=0)]).cpu().numpy() for v in views])
    assert (alone[:, 3] > 0).any()
    for kw in (dict(), dict(use_graph=True), dict(use_graph=True), dict(noalloc=True)):
        np.testing.assert_array_equal(sess.render(views, **kw).cpu().numpy(), alone)


@pytest.mark.parametrize("variant", ["fp32_rebased", "fp64_plain"])
def test_graph_follows_the_canvas(sess, variant):
    """The kernel depends on whether a canvas can have leaves of depth 0: a
    replay after the canvas under the same views has changed, by an upload or
    by an edit, and mixed views, render as an eager call does."""
    from canvasgen.pool import LEAF_DTYPE
    from editmodel import COARSEN
    views = [make_view((0.4, 0.45, -0.4), (0.02, 0.03, 1.0), 0.5, 40, 24, canvas_id=9),
             make_view((0.6, 0.3, 0.2), (0.3, 0.4, 0.8), 0.9, 16, 40, canvas_id=9,
                       out_offset_px=960)]
    one = trees.single_cell((0.2, 0.5, 0.9), 1.5, LEAF_RGBA8_F16)
    two = trees.uniform_tree(1, 1, seed=4, leaf_format=LEAF_RGBA8_F16)
    for cv in (trees.random_tree(1, 4, seed=7, leaf_format=LEAF_RGBA8_F16),
               trees.random_tree(2, 3, seed=8, p_split=0.4, leaf_format=LEAF_RGBA8_F16),
               one, two):
        sess.upload(9, cv)
        for vs in (views, [views[0], dict(views[1], canvas_id=1)],
                   [views[0], dict(views[1], canvas_id=0)]):
            ref = sess.render(vs, variant).cpu().numpy()
            for _ in range(2):
                got = sess.render(vs, variant, use_graph=True).cpu().numpy()
                np.testing.assert_array_equal(got, ref)
            for j, v in enumerate(vs):  # and each view as it is alone
                alone = sess.render([dict(v, out_offset_px=0)], variant).cpu().numpy()
                o = v["out_offset_px"]
                np.testing.assert_array_equal(ref[o:o + len(alone)], alone)
    # the refined root becomes a leaf of depth 0
    leaf = np.zeros(1, LEAF_DTYPE[LEAF_RGBA8_F16])
    leaf["r"], leaf["kappa"] = 255, np.float16(0.75).view(np.uint16)
    sess.edit(9, [(COARSEN, 0, 0)], leaf)
    got = sess.render(views, variant, use_graph=True).cpu().numpy()
    np.testing.assert_array_equal(got, sess.render(views, variant).cpu().numpy())
    assert got[:, 1].max() == 0.0 and got[:, 0].max() > 0.2

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

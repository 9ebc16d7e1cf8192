"""Renders run on torch's current stream: in order with the work before and
after them there, on whichever stream that is, across switches between streams
and with edits between them; the session's own stream comes after them."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees
from canvasgen.pool import LEAF_DTYPE

from editmodel import PAINT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    s = Session(0)
    s.cv = trees.random_tree(1, 6, seed=51, max_nodes=4000, leaf_format=LEAF_RGBA8_F16)
    s.upload(0, s.cv)
    yield s
    s.close()


VIEWS = [make_view((0.4, 0.5, -0.5), (0.0, 0.05, 1.0), 0.5, 96, 80),
         make_view((0.45, 0.55, 0.5), (1.0, 0.1, 0.2), 0.8, 50, 33, out_offset_px=96 * 80)]


@pytest.mark.parametrize("kw", [dict(), dict(use_graph=True), dict(noalloc=True)])
def test_order_on_changing_streams(sess, kw):
    torch = sess.torch
    ref = sess.render(VIEWS).cpu().numpy()
    a, b = torch.cuda.Stream(sess.device), torch.cuda.Stream(sess.device)
    busy = torch.ones((2048, 2048), device=sess.device)
    out = torch.empty((len(ref), 4), device=sess.device)
    torch.cuda.synchronize()
    got = []
    for st in (a, torch.cuda.default_stream(sess.device), b, a, b, sess.stream, a):
        with torch.cuda.stream(st):
            for _ in range(4):
                busy @ busy          # the render has to wait for what follows it
            o = out if st is a else torch.empty_like(out)
            o.fill_(-1.0)
            sess.render(VIEWS, out=o, **kw)
            got.append(o.clone())    # and this for the render
            o.fill_(-2.0)
    torch.cuda.synchronize()
    for o in got:
        np.testing.assert_array_equal(o.cpu().numpy(), ref)


def test_own_stream_follows(sess):
    torch = sess.torch
    ref = sess.render(VIEWS).cpu().numpy()
    for _ in range(3):
        o = sess.render(VIEWS)
        with torch.cuda.stream(sess.stream):
            c = o.clone()
        torch.cuda.current_stream(sess.device).wait_stream(sess.stream)
        np.testing.assert_array_equal(c.cpu().numpy(), ref)


def test_edits_between_renders_on_streams(sess):
    """An edit is seen by the renders after it, and not by those before."""
    torch = sess.torch
    st = torch.cuda.Stream(sess.device)
    before = sess.render(VIEWS).cpu().numpy()
    leaf = np.nonzero(sess.cv.nodes[:, 0] >= 0x80000000)[0]
    leaf = leaf[leaf >= 8]
    old = sess.cv.leaves[sess.cv.nodes[leaf, 0] & 0x7FFFFFFF]
    new = np.zeros(len(leaf), LEAF_DTYPE[LEAF_RGBA8_F16])
    new["g"], new["kappa"] = 200, np.float16(0.5).view(np.uint16)
    edits = [(PAINT, int(i), j) for j, i in enumerate(leaf)]
    with torch.cuda.stream(st):
        first = sess.render(VIEWS)
    sess.edit(0, edits, new)
    with torch.cuda.stream(st):
        second = sess.render(VIEWS)
    third = sess.render(VIEWS)
    sess.edit(0, edits, old)
    fourth = sess.render(VIEWS)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(first.cpu().numpy(), before)
    np.testing.assert_array_equal(second.cpu().numpy(), third.cpu().numpy())
    assert np.abs(third.cpu().numpy() - before).max() > 0.05
    np.testing.assert_array_equal(fourth.cpu().numpy(), before)

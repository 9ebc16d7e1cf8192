"""Streams that are gone, shared or captured: uploads, edits and strokes do not
go to the stream of the last render, which its owner may have destroyed, renders
are in order with a caller's work on the session's stream, and renders captured
on several streams of one capture follow one another."""
import ctypes

import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees
from canvasgen.pool import LEAF_DTYPE

from editmodel import PAINT

pytestmark = pytest.mark.gpu

VIEW = [make_view((0.4, 0.5, -0.5), (0.0, 0.05, 1.0), 0.5, 96, 80)]


@pytest.fixture
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    with Session(0) as s:
        s.cv = trees.random_tree(1, 6, seed=51, max_nodes=4000, leaf_format=LEAF_RGBA8_F16)
        s.upload(0, s.cv)
        yield s


def _render_on_a_stream_that_goes(sess):
    from paper_1704_02724_amd import cvx
    hip, torch = cvx.library(), sess.torch   # the library's own HIP runtime
    h = ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(h)) == 0
    ext = torch.cuda.ExternalStream(h.value, device=sess.device)
    with torch.cuda.stream(ext):
        img = sess.render(VIEW).cpu().numpy()
    ext.synchronize()
    assert hip.hipStreamDestroy(h) == 0
    return img


@pytest.mark.parametrize("what", ["edit", "upload", "stroke", "free", "read", "render", "close"])
def test_after_the_renders_stream_is_gone(sess, what):
    from paper_1704_02724_amd import cvx
    ref = sess.render(VIEW).cpu().numpy()
    records = cvx.cvx_read_records(sess.ctx, 0)
    np.testing.assert_array_equal(_render_on_a_stream_that_goes(sess), ref)
    if what == "edit":
        leaf = int(np.nonzero(sess.cv.nodes[8:, 0] >= 0x80000000)[0][0]) + 8
        sess.edit(0, [(PAINT, leaf, 0)],
                  sess.cv.leaves[sess.cv.nodes[leaf, 0] & 0x7FFFFFFF].reshape(1))
    elif what == "upload":
        sess.upload(0, sess.cv)
    elif what == "stroke":
        n = sess.stroke_begin(0, np.array([[0.5, 0.5, 0.5, 0.05]]), (1.0, 0.0, 0.0), 0.0, 0.05, 2.0)
        while n:
            n = sess.stroke_step(0)
        sess.upload(0, sess.cv)
    elif what == "free":
        sess.free(0)
        sess.upload(0, sess.cv)
    elif what == "read":
        np.testing.assert_array_equal(cvx.cvx_read_records(sess.ctx, 0), records)
        leaves = cvx.cvx_read_payloads(sess.ctx, 0, LEAF_DTYPE[LEAF_RGBA8_F16])
        assert len(leaves) == len(records)
    if what != "close":
        np.testing.assert_array_equal(sess.render(VIEW).cpu().numpy(), ref)


@pytest.mark.parametrize("kw", [dict(), dict(use_graph=True)])
def test_work_on_the_sessions_stream(sess, kw):
    """A copy of a frame on the session's stream, kept by the caller, comes after
    that frame and before the next one overwrites it."""
    torch = sess.torch
    other = [make_view((0.45, 0.55, 0.5), (1.0, 0.1, 0.2), 0.8, 96, 80)]
    ref = [sess.render(v).clone() for v in (VIEW, other)]
    out = torch.empty_like(ref[0])
    busy = torch.ones((2048, 2048), device=sess.device)
    own = sess.stream
    got = []
    for i in range(6):
        sess.render((VIEW, other)[i % 2], out=out, **kw)
        with torch.cuda.stream(own):
            for _ in range(4):
                busy @ busy
            got.append(out.clone())
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        assert torch.equal(g, ref[i % 2])


@pytest.mark.parametrize("noalloc", [False, True])
def test_renders_on_the_streams_of_one_capture(sess, noalloc):
    """Two streams forked before either render: only the context orders them."""
    torch = sess.torch
    small = [make_view((0.45, 0.55, 0.5), (1.0, 0.1, 0.2), 0.8, 50, 33)]
    jobs = [VIEW, small, VIEW, small]
    ref = [sess.render(v, noalloc=noalloc).clone() for v in jobs]
    out = [torch.empty_like(r) for r in ref]
    streams = [torch.cuda.Stream(sess.device) for _ in jobs]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cur = torch.cuda.current_stream(sess.device)
        for st in streams:
            st.wait_stream(cur)
        for st, v, o in zip(streams, jobs, out):
            with torch.cuda.stream(st):
                sess.render(v, out=o, noalloc=noalloc)
        for st in streams:
            cur.wait_stream(st)
    for _ in range(4):
        for o in out:
            o.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        for o, r in zip(out, ref):
            assert torch.equal(o, r)
        assert torch.equal(sess.render(VIEW), ref[0])   # eager work between the replays
    with pytest.raises(Exception, match="captured"):
        other = torch.cuda.Stream(sess.device)
        with torch.cuda.graph(torch.cuda.CUDAGraph(), capture_error_mode="thread_local"):
            sess.render(VIEW, out=out[0], noalloc=noalloc)
            with torch.cuda.stream(other):
                sess.render(VIEW, out=out[0], noalloc=noalloc)
    assert torch.equal(sess.render(VIEW), ref[0])

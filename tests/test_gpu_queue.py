"""The work queue's edges: every work item is rendered exactly once whatever the
number of items against the number of wavefronts (fewer, as many, more; ranges
no wavefront starts on), in one or eight ranges, eagerly, replayed, and in two
calls in a row."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees
from oracle import oracle

from gpu_common import rgba_err

pytestmark = pytest.mark.gpu
# (W, H) of the views: 1, 7, 8 + 1, 33 + 8 + 1 and 260 tiles of 8x8
VIEWS = [[(5, 3)], [(56, 8)], [(64, 8), (3, 8)], [(264, 7), (64, 8), (8, 1)], [(160, 104)]]


@pytest.fixture(scope="module")
def sess():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    s = Session(0)
    s.cv = trees.random_tree(2, 5, seed=71, max_nodes=4000, leaf_format=LEAF_RGBA8_F16)
    s.upload(0, s.cv)
    yield s
    s.close()


def _views(sizes):
    vs, off = [], 0
    for j, (w, h) in enumerate(sizes):
        vs.append(make_view((0.5, 0.5, -0.6 - 0.1 * j), (0.05, 0.02, 1.0), 0.6, w, h,
                            out_offset_px=off))
        off += w * h
    return vs


@pytest.mark.parametrize("sizes", VIEWS)
@pytest.mark.parametrize("wg_size", [64, 256])
@pytest.mark.parametrize("single_queue", [0, 1])
def test_every_item_once(sess, sizes, wg_size, single_queue):
    views = _views(sizes)
    orc = oracle.render([sess.cv], views)
    ok = orc["flags"] == 0
    ref = sess.render(views).cpu().numpy()
    assert ok.any() and rgba_err(ref, orc["rgba"], ok) <= 1e-3
    n = len(ref)
    for wgs in (1, 3, 8, 9, 31, 0):
        kw = dict(workgroups=wgs, wg_size=wg_size, single_queue=single_queue)
        stats = sess.new_stats()
        out = sess.torch.full((n, 4), -1.0, device=sess.device)
        sess.render(views, out=out, stats=stats, **kw)
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
        assert int(stats.cpu()[0]) == n  # each ray once
        out.fill_(-1.0)
        for graph in (False, True, True):
            sess.render(views, out=out, use_graph=graph, **kw)
            np.testing.assert_array_equal(out.cpu().numpy(), ref)

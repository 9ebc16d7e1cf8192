"""Batches that free child groups and give them out again deeper, where stored
links name nodes that have moved: records, payloads and a frame are those of a
fresh upload, in one workgroup and in the launches per level."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, trees

from editmodel import COARSEN, REFINE, PoolModel
from test_gpu_small_batches import _payloads, _same_as_upload

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


class _Pool:
    """A pool and its model, edited alike; op(...) returns REFINE's first child."""

    def __init__(self, sess):
        cv = trees.from_refinement(1, 9, lambda d, c: False, lambda d, c: (0.5, 0.5, 0.5, 1.0),
                                   LEAF_RGBA8_F16)
        sess.upload(0, cv)
        self.sess, self.model, self.edits = sess, PoolModel(cv), []
        self.pays = _payloads(np.random.Generator(np.random.PCG64(3)), 64, LEAF_RGBA8_F16)

    def op(self, op, node):
        edit = (op, node, len(self.edits) % 56)
        self.edits.append(edit)
        return int(self.model.apply([edit], self.pays)[0])

    def flush(self):
        self.sess.edit(0, self.edits, self.pays)
        self.edits = []


@pytest.mark.parametrize("pad", [0, 600])
@pytest.mark.parametrize("stays", [False, True])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_reused_groups(sess, pad, stays, axis):
    """A and B are neighbouring cells of depth 1, refined.  B's group goes to a
    leaf of depth 3, whose first child is refined too.  Then a child of A that
    touches B is refined: one that the batch made in A's old group (stays =
    False), or one that was there before (True).  Either way its stored link
    names a node of B's old group, now of depth 4."""
    p = _Pool(sess)
    top = p.op(REFINE, 0)
    a, b = top, top + (1 << axis)
    kids_a, kids_b = p.op(REFINE, a), p.op(REFINE, b)
    g = p.op(REFINE, top + 7)
    deep = p.op(REFINE, g)  # leaves of depth 3
    # more than a workgroup's worth of leaves, far away
    spare = [p.op(REFINE, g + 7)]
    for i in range(96 if pad else 0):
        spare.append(p.op(REFINE, spare[i // 8] + i % 8))
    p.flush()
    if not stays:
        p.op(COARSEN, a)
    p.op(COARSEN, b)
    assert p.op(REFINE, deep) == kids_b
    if not stays:
        assert p.op(REFINE, a) == kids_a
    p.op(REFINE, kids_a + (1 << axis))
    p.op(REFINE, kids_b)
    for i in range(pad):
        p.op(REFINE, spare[13 + i // 8] + i % 8)
    p.flush()
    _same_as_upload(sess, p.model, LEAF_RGBA8_F16)

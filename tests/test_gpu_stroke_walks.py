"""A stroke whose walk outgrows the kept lists (2^16 cells): a large brush over a
uniform depth-5 canvas reaches 20,000 cells on one level, leaves about 18,000
waiting and walks 140,000 new children; it ends on the stroke oracle's canvas.
Fewer and more stamps than the eight lanes of a cell on a small one."""
import numpy as np
import pytest

from canvasgen import LEAF_F64, LEAF_RGBA8_F16, StrokeSet, build_from_strokes, trees
from oracle import stroke as so

from test_gpu_strokes import _device_pool, _same_leaves

pytestmark = pytest.mark.gpu


def _run(cv, stamps, radius, k):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    rgb, sigma = np.array([0.2, 0.6, 1.0]), 3.0
    with Session(0) as s:
        s.upload(0, cv)
        waiting = [s.stroke_begin(0, stamps, rgb, sigma, radius, k)]
        while waiting[-1]:
            waiting.append(s.stroke_step(0))
        _, got = _device_pool(s, 0, cv)
    want = so.canonical_from_pool(cv.nodes, cv.leaves, cv.R)
    want, _ = so.apply_stroke(want, cv.leaf_format, cv.R, cv.max_depth, cv.root_edge, cv.origin,
                           stamps, rgb, sigma, radius, k)
    _same_leaves(got, want, cv.leaf_format)
    return waiting


def test_large_frontier():
    ball = StrokeSet([1.0], np.full((1, 3), 0.25), [1.0], [0, 1], [[0.5, 0.5, 0.5, 1.0]])
    cv = build_from_strokes(ball, 1, 5, 32.0, LEAF_RGBA8_F16)
    assert cv.stats["leaf_depth_hist"] == [0, 0, 0, 0, 0, 8 ** 5]
    cv.max_depth = 8
    waiting = _run(cv, np.array([[0.5, 0.5, 0.5, 0.5]]), 0.5, 20.0)
    assert waiting[0] > 8192 and len(waiting) == 2


@pytest.mark.parametrize("fmt", [LEAF_RGBA8_F16, LEAF_F64])
@pytest.mark.parametrize("n_stamps", [1, 7, 8, 9, 17])
def test_stamps_over_the_lanes_of_a_cell(fmt, n_stamps):
    cv = trees.random_tree(2, 4, seed=44, max_nodes=800, leaf_format=fmt)
    cv.max_depth = 7
    rng = np.random.Generator(np.random.PCG64(45 + n_stamps))
    stamps = np.concatenate([rng.uniform(0.2, 0.8, (n_stamps, 3)),
                             rng.uniform(0.02, 0.09, (n_stamps, 1))], axis=1)
    assert _run(cv, stamps, 0.06, 2.0)[0] > 0

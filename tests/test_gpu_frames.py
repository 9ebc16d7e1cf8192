"""The FP32 frame's length guard: a ray that crosses thousands of equal small
leaves, and one that flies far before it comes to them, must rebase on the way
(the plane values' error grows with the distance from the frame's origin), and
each visits the oracle's leaves with the oracle's lengths and colours."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees
from oracle import oracle

from gpu_common import all_ray_ids, compare_traces, rgba_err

pytestmark = pytest.mark.gpu
DEPTH = 11


def _rod(axis, first):
    """A root refined to DEPTH around a line along `axis` (from cell `first` of
    the 2^DEPTH along it), uniform coarse leaves elsewhere."""
    t = [0.3, 0.6]
    rng = np.random.Generator(np.random.PCG64(17 + axis))

    def refine(d, c):
        n = 1 << d
        across = [c[a] for a in range(3) if a != axis]
        return (all(int(t[j] * n) == across[j] for j in range(2)) and
                (c[axis] + 1) << (DEPTH - d) > first)

    return trees.from_refinement(1, DEPTH, refine,
                                 lambda d, c: (*rng.uniform(0, 1, 3), rng.uniform(0.0, 0.02)),
                                 LEAF_RGBA8_F16)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("up", [True, False])
@pytest.mark.parametrize("first", [0, 3 << (DEPTH - 2)])
def test_long_runs_of_small_leaves(axis, up, first):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    cv = _rod(axis, first)
    h = 2.0 ** -DEPTH
    eye, fwd = np.zeros(3), np.zeros(3)
    across = [a for a in range(3) if a != axis]
    eye[axis], fwd[axis] = (-0.25, 1.0) if up else (1.25, -1.0)
    for a, t in zip(across, (0.3, 0.6)):
        eye[a] = (np.floor(t / h) + 0.37) * h   # inside the rod's middle cells
    views = [make_view(eye, fwd, 0.6 * h, 8, 8)]  # the rays drift by about one leaf
    ids = all_ray_ids(views)
    ml = 3 << DEPTH
    orc = oracle.render([cv], views, ids, max_leaves=ml)
    with Session(0) as s:
        s.upload(0, cv)
        gpu = s.trace(views, ids, ml)
        img = s.render(views).cpu().numpy()
    # the longest ray crosses the whole rod, leaf by leaf
    assert int(orc["n_leaves"].max()) >= (1 << DEPTH) - first
    cmp = compare_traces(orc, gpu, ml, len_atol=1e-3)  # the guard keeps lengths to 2^-10
    assert cmp["seq_mismatch"] == 0 and cmp["len_bad"] == 0, cmp
    assert cmp["flagged"] < len(ids)
    assert rgba_err(img, orc["rgba"], cmp["ok_mask"]) <= 1e-3
    np.testing.assert_array_equal(img, gpu["rgba"])

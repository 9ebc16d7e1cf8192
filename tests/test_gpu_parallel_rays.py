"""Rays whose direction has a component too small for a reciprocal (below
2^-1000): from a plane of the grid they run along the cells on the side that the
component points to, as a ray without it does from just inside that side."""
import numpy as np
import pytest

from canvasgen import LEAF_F64, LEAF_RGBA8_F16, make_view, trees

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [LEAF_F64, LEAF_RGBA8_F16])
@pytest.mark.parametrize("tiny", [2.0 ** -1001, 1e-310, 5e-324])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_tiny_components(fmt, tiny, axis):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    cv = trees.random_tree(1, 6, seed=29, p_split=0.75, max_nodes=20000, leaf_format=fmt)
    along, third = (axis + 1) % 3, (axis + 2) % 3
    with Session(0) as s:
        s.upload(0, cv)

        def pixel(plane, c, variant):
            eye, fwd = np.zeros(3), np.zeros(3)
            eye[axis], eye[along], eye[third] = plane, -0.25, 0.4321
            fwd[axis], fwd[along] = c, 1.0
            view = make_view((0, 0, 0), np.eye(3)[along], 0.5, 1, 1)
            view.update(eye=tuple(eye), fwd=tuple(fwd))
            return s.render([view], variant, out_f64=variant == "fp64_plain").cpu().numpy()

        differ = 0
        for k in range(1, 16):
            plane = k / 16.0
            for variant in ("fp64_plain",) + (("fp32_rebased",) if fmt != LEAF_F64 else ()):
                lo, hi = (pixel(np.nextafter(plane, x), 0.0, variant) for x in (0.0, 1.0))
                np.testing.assert_array_equal(pixel(plane, -tiny, variant), lo)
                np.testing.assert_array_equal(pixel(plane, tiny, variant), hi)
                differ += bool((lo != hi).any())
        assert differ > 0

"""A graph of a render in chord pieces serves the view count it was captured
with: with another one every view is still merged."""
import pytest

from canvasgen import LEAF_RGBA8_F16, make_view, trees

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(2, 1, 2), (1, 3, 2), (3, 1, 1)])
def test_view_counts(counts):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    cv = trees.random_tree(1, 7, seed=19, p_split=0.6, max_nodes=9000, leaf_format=LEAF_RGBA8_F16)
    side = 256
    shape = dict(chord_pieces=2, workgroups=256, wg_size=256)  # the same launch for every count
    views = [make_view((0.5, 0.5, -1.0 - 0.1 * i), (0.0, 0.0, 1.0), 0.5, side, side,
                       out_offset_px=i * side * side) for i in range(3)]
    with Session(0) as s:
        s.upload(0, cv)
        out = torch.empty((3 * side * side, 4), device="cuda")
        ref = s.render(views, out=out, **shape).clone()
        for n in counts:
            for _ in range(2):  # captured, then replayed
                out.fill_(-1.0)
                s.render(views[:n], out=out, use_graph=True, **shape)
                assert torch.equal(out[:n * side * side], ref[:n * side * side])
                assert bool((out[n * side * side:] == -1.0).all())

"""A stroke that only repaints leaves needs next to no device memory: with the
device nearly full, where the blocks that a context keeps for strokes have no
room, it paints what it does otherwise."""
import numpy as np
import pytest

from canvasgen import LEAF_RGBA8_F16, trees
from canvasgen.pool import LEAF_DTYPE

pytestmark = pytest.mark.gpu

STROKE = dict(stamps=np.array([[0.4, 0.5, 0.6, 0.2], [0.5, 0.5, 0.5, 0.25]]), rgb=(0.2, 0.8, 0.4),
              sigma=3.0, radius=0.25, k_refine=1.0 / 64.0)  # every leaf is fine enough


def test_stroke_on_a_full_device():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd import cvx
    from paper_1704_02724_amd.session import Session
    cv = trees.random_tree(1, 5, seed=13, leaf_format=LEAF_RGBA8_F16)

    def leaves(s):
        return cvx.cvx_read_payloads(s.ctx, 0, LEAF_DTYPE[LEAF_RGBA8_F16]).tobytes()

    with Session(0) as s:
        s.upload(0, cv)
        before = leaves(s)
        assert s.stroke_begin(0, **STROKE) == 0
        ref = leaves(s)
    assert ref != before
    with Session(0) as s:   # a new one keeps no blocks yet
        s.upload(0, cv)
        fill = []
        try:
            while True:
                free, _ = torch.cuda.mem_get_info(s.device)
                chunk = min(free - (4 << 20), 16 << 30)
                if chunk < (12 << 20):   # torch allocates smaller ones in blocks of 20 MiB
                    break
                fill.append(torch.empty(chunk, dtype=torch.uint8, device=s.device))
            assert free <= 16 << 20      # two blocks of 8 MiB and more do not fit
            assert s.stroke_begin(0, **STROKE) == 0
        finally:
            del fill
            torch.cuda.synchronize()
            torch.cuda.empty_cache()
        assert leaves(s) == ref

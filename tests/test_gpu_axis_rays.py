"""Rays parallel to one or two axes (components of exactly zero, whose planes
are never reached and whose side of a mid-plane is the eye's), through root
arrays and abrupt depth changes, in both leaf formats and both product casters:
the oracle's leaves and colours."""
import numpy as np
import pytest

from canvasgen import LEAF_F64, LEAF_RGBA8_F16, trees
from oracle import oracle

from gpu_common import all_ray_ids, compare_traces, rgba_err
from helpers import ray_views

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,depth", [(1, 8), (2, 6), (3, 5)])
@pytest.mark.parametrize("fmt,variant,tol", [(LEAF_RGBA8_F16, "fp32_rebased", 1e-3),
                                             (LEAF_RGBA8_F16, "fp64_plain", 2.0 ** -23),
                                             (LEAF_F64, "fp64_plain", 2.0 ** -23)])
def test_axis_parallel_rays(R, depth, fmt, variant, tol):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    cv = trees.random_tree(R, depth, seed=61 + R, p_split=0.5, max_nodes=9000, leaf_format=fmt)
    rng = np.random.Generator(np.random.PCG64(62))
    eyes, dirs = [], []
    for zeros in (1, 2):
        for axis in range(3):
            for _ in range(12):
                d = np.zeros(3)
                d[axis] = rng.choice([-1.0, 1.0])
                if zeros == 1:
                    d[(axis + 1) % 3] = rng.uniform(-1.0, 1.0)
                eyes.append(rng.uniform(0.02, 0.98, 3) - (1.5 * d if rng.random() < 0.5 else 0.0))
                dirs.append(d)
    views = ray_views(eyes, dirs)
    for i, v in enumerate(views):
        v["out_offset_px"] = i
    ids = all_ray_ids(views)
    orc = oracle.render([cv], views, ids, max_leaves=512)
    with Session(0) as s:
        s.upload(0, cv)
        gpu = s.trace(views, ids, 512, variant)
        img = s.render(views, variant).cpu().numpy()
    cmp = compare_traces(orc, gpu, 512)
    assert cmp["seq_mismatch"] == 0 and cmp["flagged"] < len(ids) // 2, cmp
    assert (orc["n_leaves"] > 4).sum() > len(ids) // 3
    # an FP64 image is rounded to float32 (2^-24 relative, values up to 1)
    assert rgba_err(img, orc["rgba"], cmp["ok_mask"]) <= tol

"""Pixels of FP32 images that depend on the frames of the traversal: how far a
frame reaches (8 levels below its first leaf, lengths within 2^-10 of an edge)
and which planes its rounded values belong to.  A frame kept longer, or counted
from another plane, is as well within the image bar, but moves single pixels by
up to 2e-3 and small images away from the 64-bit ones.

tests/golden/fp32_frame_pixels.txt holds the pixels that such a change moved
most.  The plane values are the same in every build of these frames, so what is
left is the rounding of the composite: three roundings of 2^-24 of values up to
1 (absorbed share, transmittance, colour) per leaf."""
import os

import numpy as np
import pytest

from canvasgen import (LEAF_RGBA8_F16, build_from_strokes, eye_near_stroke, gen_strokes, make_view)

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fp32_frame_pixels.txt")
LEAVES = 300  # more than any ray of the scenes crosses

# name: strokes, lg of the smallest and largest radius, roots, depth, image size, eye
SCENES = {"outside": (16, -8.0, -4.0, 1, 12, 64, 64, "outside"),
          "roots": (60, -9.0, -4.0, 3, 11, 333, 217, "outside"),
          "inside": (100, -14.0, -3.0, 1, 17, 96, 96, "inside")}


def scene(name, seed):
    n, lo, hi, roots, depth, w, h, where = SCENES[name]
    rng = np.random.Generator(np.random.PCG64(seed))
    st = gen_strokes(rng, n, lo, hi)
    cv = build_from_strokes(st, roots, depth, 4.0, LEAF_RGBA8_F16,
                            split_depth=5 if roots == 1 else 0)
    if where == "inside":
        eye, fwd, _ = eye_near_stroke(rng, st, 2.0 ** -12)
        return cv, make_view(eye, fwd, 1.0, w, h)
    u = rng.normal(size=3)
    u /= np.linalg.norm(u)
    return cv, make_view(np.full(3, 0.5) - rng.uniform(1.1, 1.6) * u, u, 0.5, w, h)


def golden():
    rows = {}
    for line in open(GOLDEN):
        f = line.split("#")[0].split()
        if f:
            rows.setdefault((f[0], int(f[1])), []).append([float(x) for x in f[2:]])
    return {k: np.array(v) for k, v in rows.items()}


@pytest.mark.parametrize("name,seed", sorted(golden()))
@pytest.mark.parametrize("refill", [False, True])
def test_pixels(name, seed, refill):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1704_02724_amd.session import Session
    rows = golden()[name, seed]
    cv, view = scene(name, seed)
    with Session(0) as s:
        s.upload(0, cv)
        img = s.render([view], rays_per_wave=256 if refill else 0).cpu().numpy()
    at = (rows[:, 1] * view["W"] + rows[:, 0]).astype(np.int64)
    assert np.abs(img[at].astype(np.float64) - rows[:, 2:]).max() <= LEAVES * 3 * 2.0 ** -24

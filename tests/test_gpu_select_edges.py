"""Point selection at the edges of its blocks: images that end inside the first
block, at a block's end and just past it, and on both sides of the size from
which the blocks' ranks are scanned, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

from test_gpu_select import _check, cvo  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,D", [((15, 64), 3), ((16, 64), 1), ((17, 65), 9), ((32, 32), 24), ((33, 32), 0),
                                     ((1024, 2048), 2), ((1025, 2048), 2)])
def test_select_block_edges(cvo, shape, D):  # noqa: F811
    rng = np.random.default_rng(shape[0] + shape[1])
    gray = rng.integers(0, 256, size=shape, dtype=np.uint8)
    gray = np.where(rng.random(shape) < 0.2, gray, 128).astype(np.uint8)
    depth = rng.uniform(0.5, 12.0, size=shape).astype(np.float32)
    feat = rng.random(shape + (D,)).astype(np.float32) if D else None
    cam = dict(fx=60.0, fy=58.5, cx=shape[1] / 2 - 0.5, cy=shape[0] / 2 + 0.25, depth_min=1.0, depth_max=10.0)
    for cap in (0, 37, shape[0] * shape[1]):
        _check(cvo, gray, depth, feat, cam, cap)

"""Morphology with balls around the size of the grid, against the oracle: erosions that leave the
middle of a solid mask, one voxel of it or nothing, dilations whose rows mostly leave the grid."""

import numpy as np
import pytest
import torch

from oracle import masks as K
from paper_1605_02060_amd import lddmm as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 6, 40), (9, 2, 70), (2, 11, 33), (1, 7, 64)])
@pytest.mark.parametrize("radius", [0.5, 1.0, 2.0, 2.5, 4.0, 5.2, 9.0])
def test_ball_around_the_extent(shape, radius):
    print(f"[gpu-case] morphology {shape} r={radius}", flush=True)
    rng = np.random.default_rng(31)
    solid = np.ones(shape, bool)
    holed = rng.random(shape) > 0.02
    points = rng.random(shape) > 0.98
    t = lambda a: torch.as_tensor(a.astype(np.float32), device="cuda")
    for A, op, ref in ((solid, L.MORPH_ERODE, K.erode), (holed, L.MORPH_ERODE, K.erode),
                       (points, L.MORPH_DILATE, K.dilate), (holed, L.MORPH_OPEN, K.opening),
                       (points, L.MORPH_CLOSE, K.closing)):
        got = L.lddmm_morphology(t(A), op, radius).cpu().numpy()
        np.testing.assert_array_equal(got > 0, ref(A, radius, 1.0), err_msg=str(op))

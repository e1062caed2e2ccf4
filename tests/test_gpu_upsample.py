"""The 2x upsampling at its smallest and raggedest grids: extents of 2 (every
neighbour clamped on one side), odd extents, and one axis long."""

import numpy as np
import pytest
import torch

from oracle import lddmm as O
from paper_1605_02060_amd import cnn as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,h,w", [(2, 2, 2), (2, 3, 5), (3, 2, 67), (9, 4, 2), (5, 33, 3)])
def test_expand_velocity_edges(d, h, w):
    print(f"[gpu-case] upsample {d} {h} {w}", flush=True)
    T = 2
    out = np.random.default_rng(3).normal(size=(d, h, w, 3 * T)).astype(np.float32)
    v = G.expand_velocity(torch.as_tensor(out, device="cuda"), T, 0.5).cpu().numpy()
    f = 0.5 * out.astype(np.float64).transpose(3, 0, 1, 2)
    ref = np.stack([O.upsample2_clamp(O.upsample2_clamp(c, (2 * d, 2 * h, 2 * w)),
                                      (4 * d, 4 * h, 4 * w)) for c in f]).reshape(v.shape)
    # two trilinear steps of seven FP32 blends each: 2 * 7 * 2^-23 of the largest value
    assert np.abs(v - ref).max() <= 14 * 2.0 ** -23 * np.abs(f).max()

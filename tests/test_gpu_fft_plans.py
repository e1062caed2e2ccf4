"""The smoothing operator on every length with a compile-time plan of its own and no other
test, along each axis, against the oracle.

Tolerance of the smoothing as for every other length: 1e-5 of the largest magnitude (FP32
butterflies, FP64 tables rounded once)."""

import numpy as np
import pytest
import torch

from oracle import lddmm as O
from paper_1605_02060_amd import lddmm as L

pytestmark = pytest.mark.gpu
LENGTHS = [24, 25, 27, 28, 30, 35, 36, 42, 45, 48, 49, 50, 54, 56, 63, 168, 180, 192, 196, 210,
           224, 225, 256, 162, 200, 216, 252, 270, 288, 300, 320]


@pytest.mark.parametrize("n", LENGTHS)
def test_smooth_on_each_length(n):
    for P in ((6, 10, n), (6, n, 10), (n, 6, 10)):
        print(f"[gpu-case] smooth {P}", flush=True)
        b = np.random.default_rng(n).normal(size=(3,) + P)
        # a first element off the 16-byte boundary goes through a copy
        buf = torch.empty(b.size + 1, device="cuda")
        odd = buf[1:].view(b.shape)
        odd.copy_(torch.as_tensor(b))
        out = L.lddmm_smooth(torch.as_tensor(b, dtype=torch.float32, device="cuda"), 0.1, 0.02, 1.0)
        ref = O.apply_K(b, 0.02, 1.0, 0.1)
        assert np.abs(out.cpu().numpy() - ref).max() < 1e-5 * np.abs(ref).max()
        assert torch.equal(out, L.lddmm_smooth(odd, 0.1, 0.02, 1.0))

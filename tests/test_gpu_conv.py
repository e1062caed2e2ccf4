"""The convolution kernels that load fragments or stage the source tile in LDS, at
their edges: every source channel count with a variant of its own (16, 32, 64,
128, 192), ones without (6, 96), row counts around 16, 32, 64, 128 and 192, and
extents of one voxel, below, at and just past a tile, odd and even for both
strides.  Oracle, operands and bound as in test_gpu_cnn."""

import numpy as np
import pytest
import torch

from oracle import cnn as C
from paper_1605_02060_amd import cnn as G
from test_gpu_cnn import bf, bound, host

pytestmark = pytest.mark.gpu

# (n, (d, h, w), ci, co, stride)
CASES = [
    (1, (1, 1, 1), 32, 16, 1), (1, (4, 4, 8), 32, 32, 1), (2, (5, 5, 9), 32, 17, 1),
    (1, (3, 4, 9), 64, 48, 1), (1, (2, 9, 7), 128, 20, 1), (1, (5, 4, 8), 192, 70, 1),
    (1, (4, 5, 6), 64, 192, 1), (1, (3, 5, 8), 96, 33, 1), (1, (3, 5, 8), 6, 10, 1),
    (1, (9, 8, 17), 16, 32, 2), (1, (1, 2, 3), 32, 64, 2), (1, (9, 8, 17), 32, 64, 2),
    (2, (8, 9, 15), 64, 128, 2), (1, (5, 6, 7), 96, 96, 2), (1, (7, 8, 9), 128, 32, 2),
]


@pytest.mark.parametrize("n,dims,ci,co,stride", CASES)
def test_forward(n, dims, ci, co, stride):
    print(f"[gpu-case] conv fwd {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(5)
    xq, xg = bf(rng.normal(size=(n,) + dims + (ci,)))
    wq, wg = bf(rng.normal(size=(co, 3, 3, 3, ci)) / np.sqrt(27 * ci))
    b = rng.normal(size=co).astype(np.float32).astype(np.float64)
    bg = torch.as_tensor(b, dtype=torch.float32, device="cuda")
    y = host(G.conv3d_forward(xg, wg, bg, stride, relu=False, out_dtype=torch.float32))
    lim = bound(27 * ci, C.conv3d(np.abs(xq), np.abs(wq), np.abs(b), stride))
    assert np.all(np.abs(y - C.conv3d(xq, wq, b, stride)) <= lim)


@pytest.mark.parametrize("n,dims,ci,co,stride", [(n, d, co, ci, s) for n, d, ci, co, s in CASES])
def test_backward_data(n, dims, ci, co, stride):
    """The same list with the channel counts exchanged: the gradient's source has co."""
    print(f"[gpu-case] conv dgrad {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(6)
    out = tuple(G.out_extent(v, stride) for v in dims)
    wq, wg = bf(rng.normal(size=(co, 3, 3, 3, ci)) / np.sqrt(27 * co))
    dq, dg = bf(rng.normal(size=(n,) + out + (co,)))
    mq, mg = bf(rng.normal(size=(n,) + dims + (ci,)))
    aq, ag = bf(rng.normal(size=(n,) + dims + (ci + 3,)))
    dx = host(G.conv3d_backward_data(dg, (n,) + dims + (ci,), G.transpose_weight(wg), stride,
                                     mask=mg, add=ag, add_off=2, out_dtype=torch.float32))
    shp = (n,) + dims + (ci,)
    ref = C.conv3d_dgrad(dq, wq, shp, stride) * (mq > 0) + aq[..., 2:2 + ci]
    lim = bound(27 * co, C.conv3d_dgrad(np.abs(dq), np.abs(wq), shp, stride)
                + np.abs(aq[..., 2:2 + ci]))
    assert np.all(np.abs(dx - ref) <= lim)


@pytest.mark.parametrize("n,dims,ci,co,stride", [
    (1, (1, 1, 1), 16, 16, 1), (1, (2, 8, 8), 16, 32, 1), (2, (3, 9, 7), 16, 40, 2),
    (1, (5, 17, 16), 16, 30, 2), (1, (4, 7, 9), 32, 17, 1), (1, (5, 15, 18), 32, 64, 2),
    (2, (3, 8, 9), 64, 30, 1), (1, (3, 5, 8), 48, 33, 2), (1, (4, 9, 8), 96, 70, 1),
    (1, (1, 1, 1), 2, 16, 1), (2, (5, 9, 17), 2, 16, 1), (1, (3, 8, 10), 2, 9, 1),
    (1, (4, 6, 7), 2, 40, 1),
])
def test_backward_weight(n, dims, ci, co, stride):
    print(f"[gpu-case] conv wgrad {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(7)
    xq, xg = bf(rng.normal(size=(n,) + dims + (ci,)))
    dq, dg = bf(rng.normal(size=(n,) + tuple(C.out_size(v, stride) for v in dims) + (co,)))
    dw, db = G.conv3d_backward_weight(dg, xg, stride)
    ref_w, ref_b = C.conv3d_wgrad(dq, xq, stride)
    abs_w, abs_b = C.conv3d_wgrad(np.abs(dq), np.abs(xq), stride)
    K = int(np.prod(dq.shape[:4]))          # as test_gpu_cnn: the K-term sequential bound
    assert np.all(np.abs(host(dw) - ref_w) <= bound(K + 1024, abs_w))
    assert np.all(np.abs(host(db) - ref_b) <= bound(K + 1024, abs_b))
    only = torch.empty_like(dw)
    again, _ = G.conv3d_backward_weight(dg, xg, stride, dw=only)
    assert torch.equal(again, dw)           # deterministic

"""Convolution operands that start 4 and 8 bytes past a 16-byte boundary: the kernels that load
16 bytes straight to LDS leave them to the others.  Forward and input gradient have the bits of
aligned operands (the same products in the same order); the weight gradient, summed otherwise,
is checked against the oracle with the bound of test_gpu_conv."""

import numpy as np
import pytest
import torch

from oracle import cnn as C
from paper_1605_02060_amd import cnn as G
from test_gpu_cnn import bf, bound, host

pytestmark = pytest.mark.gpu


def shifted(t, off):
    """A copy of t that starts `off` elements past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    assert buf.data_ptr() % 16 == 0
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("off", [2, 4])
@pytest.mark.parametrize("n,dims,ci,co,stride", [
    (1, (5, 9, 10), 2, 16, 1), (1, (5, 6, 7), 16, 32, 2), (2, (5, 9, 10), 32, 64, 1),
    (1, (6, 10, 9), 64, 32, 2), (1, (3, 5, 8), 96, 64, 1), (1, (5, 4, 9), 192, 64, 1),
])
def test_shifted_operands(n, dims, ci, co, stride, off):
    print(f"[gpu-case] conv offset {off} {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(9)
    out = tuple(C.out_size(v, stride) for v in dims)
    xq, x = bf(rng.normal(size=(n,) + dims + (ci,)))
    _, w = bf(rng.normal(size=(co, 3, 3, 3, ci)))
    dq, dy = bf(rng.normal(size=(n,) + out + (co,)))
    wt, b = G.transpose_weight(w), torch.zeros(co, device="cuda")
    xs, ds = shifted(x, off), shifted(dy, off)
    y = G.conv3d_forward(x, w, b, stride, relu=False, out_dtype=torch.float32)
    assert torch.equal(y, G.conv3d_forward(xs, w, b, stride, relu=False, out_dtype=torch.float32))
    dx = G.conv3d_backward_data(dy, tuple(x.shape), wt, stride, out_dtype=torch.float32)
    assert torch.equal(dx, G.conv3d_backward_data(ds, tuple(x.shape), wt, stride,
                                                  out_dtype=torch.float32))
    ref_w, ref_b = C.conv3d_wgrad(dq, xq, stride)
    abs_w, abs_b = C.conv3d_wgrad(np.abs(dq), np.abs(xq), stride)
    K = int(np.prod(dq.shape[:4]))
    for args in ((ds, x), (dy, xs), (ds, xs)):
        dw, db = G.conv3d_backward_weight(*args, stride)
        assert np.all(np.abs(host(dw) - ref_w) <= bound(K + 1024, abs_w))
        assert np.all(np.abs(host(db) - ref_b) <= bound(K + 1024, abs_b))

"""The first layer's kernel (two source channels) at the edges of its tile, against the
oracle; and the row split of the staged kernels: a large batch takes blocks of many rows, its
samples alone blocks of few, and both sum in the same order, so they are compared bit for
bit.  Oracle, operands and bound as in test_gpu_cnn."""

import numpy as np
import pytest
import torch

from oracle import cnn as C
from paper_1605_02060_amd import cnn as G
from test_gpu_cnn import bf, bound, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dims,co", [(1, (1, 1, 1), 16), (2, (4, 4, 32), 16), (1, (5, 5, 33), 17),
                                       (1, (3, 9, 31), 6), (2, (6, 3, 70), 48),
                                       (1, (9, 7, 47), 16), (2, (17, 4, 16), 32)])
def test_two_channels(n, dims, co):
    print(f"[gpu-case] two channels {n} {dims} -> {co}", flush=True)
    rng = np.random.default_rng(7)
    xq, xg = bf(rng.normal(size=(n,) + dims + (2,)))
    wq, wg = bf(rng.normal(size=(co, 3, 3, 3, 2)) / np.sqrt(54))
    b = rng.normal(size=co).astype(np.float32).astype(np.float64)
    bg = torch.as_tensor(b, dtype=torch.float32, device="cuda")
    y = host(G.conv3d_forward(xg, wg, bg, 1, relu=False, out_dtype=torch.float32))
    lim = bound(54, C.conv3d(np.abs(xq), np.abs(wq), np.abs(b), 1))
    assert np.all(np.abs(y - C.conv3d(xq, wq, b, 1)) <= lim)
    # bf16 results are those rounded, whichever way they are stored
    yb = G.conv3d_forward(xg, wg, bg, 1, relu=True)
    yf = G.conv3d_forward(xg, wg, bg, 1, relu=True, out_dtype=torch.float32)
    assert torch.equal(yb, yf.to(torch.bfloat16))


@pytest.mark.parametrize("n,dims,ci,co,stride", [
    (40, (8, 8, 16), 192, 64, 1), (40, (8, 8, 16), 64, 192, 1), (20, (8, 8, 16), 64, 128, 1),
    (40, (8, 8, 16), 128, 48, 1), (40, (16, 16, 16), 64, 128, 2), (20, (16, 16, 32), 32, 64, 2),
    (40, (8, 8, 16), 64, 30, 1)])
def test_rows_split_by_the_size_of_the_launch(n, dims, ci, co, stride):
    print(f"[gpu-case] row split {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(8)
    x = bf(rng.normal(size=(n,) + dims + (ci,)))[1]
    w = bf(rng.normal(size=(co, 3, 3, 3, ci)) / np.sqrt(27 * ci))[1]
    y = G.conv3d_forward(x, w, None, stride, relu=False, out_dtype=torch.float32)
    out = y.shape[1:4]
    dy = bf(rng.normal(size=(n,) + tuple(out) + (co,)))[1]
    wt = G.transpose_weight(w)
    dx = None
    if co % 2 == 0:
        dx = G.conv3d_backward_data(dy, tuple(x.shape), wt, stride, out_dtype=torch.float32)
    for k in (0, n - 1):
        assert torch.equal(y[k:k + 1], G.conv3d_forward(x[k:k + 1].contiguous(), w, None, stride,
                                                        relu=False, out_dtype=torch.float32))
        if dx is not None:
            one = G.conv3d_backward_data(dy[k:k + 1].contiguous(), (1,) + tuple(x.shape[1:]), wt,
                                         stride, out_dtype=torch.float32)
            assert torch.equal(dx[k:k + 1], one)

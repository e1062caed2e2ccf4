"""An infinite value reaches exactly the results that use it, in every variant of the
convolution kernels: the other results keep the bits of a run without it.  Extents leave
tiles and chunks ragged, and the value sits on the last voxel, the first, or inside."""

import numpy as np
import pytest
import torch

from oracle import cnn as C
from paper_1605_02060_amd import cnn as G
from test_gpu_cnn import bf

pytestmark = pytest.mark.gpu
TAPS = [(kz, ky, kx) for kz in range(3) for ky in range(3) for kx in range(3)]

# (n, (d, h, w), ci, co, stride): each variant of the weight gradient and of the others
CASES = [
    (1, (5, 9, 10), 2, 16, 1), (1, (5, 9, 10), 16, 32, 1), (2, (6, 10, 12), 16, 32, 2),
    (1, (6, 10, 12), 16, 40, 2), (1, (3, 7, 13), 32, 30, 1), (1, (6, 18, 10), 32, 64, 2),
    (1, (3, 9, 9), 64, 70, 1), (1, (3, 5, 9), 192, 64, 1), (1, (5, 9, 10), 6, 10, 1),
]


def places(dims):
    return [tuple(v - 1 for v in dims), (0, 0, 0), tuple(v // 2 for v in dims)]


def outputs_of(p, out, stride):
    """(tap, output voxel) pairs that read input voxel p."""
    for t in TAPS:
        o = [p[a] + 1 - t[a] for a in range(3)]
        if all(v % stride == 0 and 0 <= v // stride < out[a] for a, v in enumerate(o)):
            yield t, tuple(v // stride for v in o)


def check(clean, dirty, hit):
    hit = torch.as_tensor(hit, device=clean.device)
    assert torch.isfinite(clean).all()
    assert torch.equal(dirty[~hit], clean[~hit])
    assert not torch.isfinite(dirty[hit]).any()


@pytest.mark.parametrize("n,dims,ci,co,stride", CASES)
def test_weight_gradient(n, dims, ci, co, stride):
    print(f"[gpu-case] nonfinite wgrad {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(3)
    out = tuple(C.out_size(v, stride) for v in dims)
    _, x = bf(rng.normal(size=(n,) + dims + (ci,)))
    _, dy = bf(0.5 + rng.random(size=(n,) + out + (co,)))
    for p in places(dims):
        at = (n - 1,) + p + (ci - 1,)
        x[at] = 0.0
        dw, db = G.conv3d_backward_weight(dy, x, stride)
        x[at] = float("inf")
        dw1, db1 = G.conv3d_backward_weight(dy, x, stride)
        x[at] = 1.0
        hit = np.zeros(dw.shape, bool)
        for t, _ in outputs_of(p, out, stride):
            hit[:, t[0], t[1], t[2], ci - 1] = True
        check(dw, dw1, hit)
        assert torch.equal(db, db1)


@pytest.mark.parametrize("n,dims,ci,co,stride", CASES)
def test_forward(n, dims, ci, co, stride):
    print(f"[gpu-case] nonfinite fwd {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(4)
    out = tuple(C.out_size(v, stride) for v in dims)
    _, x = bf(rng.normal(size=(n,) + dims + (ci,)))
    _, w = bf(0.5 + rng.random(size=(co, 3, 3, 3, ci)))
    b = torch.zeros(co, device="cuda")
    for p in places(dims):
        at = (n - 1,) + p + (ci - 1,)
        x[at] = 0.0
        y = G.conv3d_forward(x, w, b, stride, relu=False, out_dtype=torch.float32)
        x[at] = float("inf")
        y1 = G.conv3d_forward(x, w, b, stride, relu=False, out_dtype=torch.float32)
        x[at] = 1.0
        hit = np.zeros(y.shape, bool)
        for _, o in outputs_of(p, out, stride):
            hit[(n - 1,) + o] = True
        check(y, y1, hit)


@pytest.mark.parametrize("n,dims,ci,co,stride", [(n, d, co, ci, s) for n, d, ci, co, s in CASES])
def test_input_gradient(n, dims, ci, co, stride):
    print(f"[gpu-case] nonfinite dgrad {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(5)
    out = tuple(C.out_size(v, stride) for v in dims)
    shape = (n,) + dims + (ci,)
    _, dy = bf(rng.normal(size=(n,) + out + (co,)))
    wt = G.transpose_weight(bf(0.5 + rng.random(size=(co, 3, 3, 3, ci)))[1])
    for o in places(out):
        at = (n - 1,) + o + (co - 1,)
        dy[at] = 0.0
        dx = G.conv3d_backward_data(dy, shape, wt, stride, out_dtype=torch.float32)
        dy[at] = float("inf")
        dx1 = G.conv3d_backward_data(dy, shape, wt, stride, out_dtype=torch.float32)
        dy[at] = 1.0
        hit = np.zeros(shape, bool)
        for t in TAPS:
            i = tuple(stride * o[a] + t[a] - 1 for a in range(3))
            if all(0 <= i[a] < dims[a] for a in range(3)):
                hit[(n - 1,) + i] = True
        check(dx, dx1, hit)

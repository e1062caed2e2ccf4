"""The staged splat of the exact gradient, which runs on grids of at least 655360 voxels, against
the general one, which the smaller grids of test_gpu_splat and test_gpu_splat_reach check against
the oracle: a problem on a small grid (general) is embedded in zeros in a large one (staged), and
both see the same FP32 positions, so the gradients differ by the rounding of the splat's sums
alone.  (Against the oracle in 64 bits a single position within rounding of a cell face, where
the derivative jumps, decides the largest difference on grids of this size.)

The sums have at most 27 terms per output and step, whose weights add up to at most 8, and two
steps: 2 * 27 * 8 * 2^-24 = 2.6e-5 of the largest value."""

import numpy as np
import pytest
import torch

from oracle import lddmm as O
from paper_1605_02060_amd import lddmm as L
from paper_1605_02060_amd import synth

pytestmark = pytest.mark.gpu
T, H = 2, 0.5


def gradient(M0, M1, v):
    t = lambda a: torch.as_tensor(a, device="cuda")
    g, e = L.lddmm_gradient(t(M0), t(M1), None, None, t(v), L.Params(T=T, iters=(1,)),
                            kind=L.GRAD_L2, spacing=H)
    return g.cpu().numpy(), e.cpu().numpy()


# large grid, small grid, the small one's place (0: at the low end of the axis, -1: at the high
# end, else its first voxel), all z, y, x
@pytest.mark.parametrize("sign,dmax", [("mixed", (0.9, 0.9)), ("plus", (0.99, 0.5)),
                                       ("minus", (0.99, 0.9)), ("mixed", (0.9, 1.4))])
@pytest.mark.parametrize("large,small,at", [
    ((60, 84, 135), (20, 21, 70), (0, 0, 0)),        # low corner; across the tile edge at 64
    ((60, 84, 135), (20, 21, 70), (-1, -1, -1)),     # high corner: a tile of 7 columns
    ((100, 105, 63), (24, 20, 63), (37, 41, 0)),     # one tile of 63 columns, both its ends
    ((160, 64, 64), (20, 30, 64), (-1, 0, 0)),       # the smallest grid; a full tile
    ((1024, 5, 128), (40, 5, 128), (500, 0, 0)),     # one row past a tile, both ends of y and x
    ((2, 640, 512), (2, 24, 140), (0, 301, 100)),    # two planes, one run
])
def test_staged_splat_equals_the_general_one(large, small, at, sign, dmax):
    print(f"[gpu-case] staged splat {large} {small} {at} {sign} {dmax}", flush=True)
    for n in (large, small):
        assert tuple(O.smooth7(k) for k in n) == n
    assert np.prod(large) >= 655360 > np.prod(small)
    rng = np.random.default_rng(17)
    # fields end four voxels before a side that the grids do not share; the outer two of them are
    # not compared: what the periodic Laplacian squared carries across the grid's ends lies there
    window = np.ones(small)
    place, inner = [], []
    for ax in range(3):
        n, first = small[ax], at[ax] if at[ax] >= 0 else large[ax] - small[ax]
        place.append(slice(first, first + n))
        w = np.ones(n)
        lo, hi = first > 0, first + n < large[ax]
        if lo:
            w[:4] = 0.0
        if hi:
            w[-4:] = 0.0
        inner.append(slice(2 * lo, n - 2 * hi))
        window *= w.reshape([-1 if k == ax else 1 for k in range(3)])
    place, inner = (Ellipsis,) + tuple(place), (Ellipsis,) + tuple(inner)
    v = np.stack([synth.plane_wave_velocity(small, 40 + j, 1.0) for j in range(T)])
    if sign != "mixed":
        v = np.abs(v) * (1.0 if sign == "plus" else -1.0)
    v *= window
    for j in range(T):
        v[j] *= dmax[j] * T * H / np.abs(v[j]).max()
    v = v.astype(np.float32)
    M0, M1 = (((rng.random(small) > 0.5) * window).astype(np.float32) for _ in range(2))
    ga, ea = gradient(M0, M1, v)

    def embed(a):
        out = np.zeros(a.shape[:-3] + large, np.float32)
        out[place] = a
        return out

    gb, eb = gradient(embed(M0), embed(M1), embed(v))
    lim = 2.6e-5 * np.abs(ga).max()
    assert np.abs(gb[place] - ga)[inner].max() <= lim
    assert np.abs(eb[:3] - ea[:3]).max() <= 1e-6 * abs(ea[0])

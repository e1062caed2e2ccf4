"""The staged splat of the exact gradient at its edges: x around one and two
64-wide tiles, y around the four rows of a tile, one plane to several runs of
planes, displacements of one sign per axis (two source offsets per axis), of
mixed signs, and past one voxel (the general body)."""

import numpy as np
import pytest
import torch

from oracle import lddmm as O
from paper_1605_02060_amd import lddmm as L
from paper_1605_02060_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,sign,dmax", [
    ((2, 2, 2), "mixed", 0.9),
    ((7, 3, 64), "plus", 0.9),          # (z, y, x): one tile exactly along x
    ((7, 4, 63), "minus", 0.9),
    ((12, 5, 70), "mixed", 0.9),        # a second tile of 6 columns, a row left over
    ((13, 9, 128), "plus", 0.99),
    ((30, 8, 135), "mixed", 0.3),
    ((12, 5, 70), "mixed", 1.4),        # reach 2: the general body
])
def test_staged_splat_matches_oracle(shape, sign, dmax):
    print(f"[gpu-case] splat {shape} {sign} {dmax}", flush=True)
    T, h = 3, 0.5
    P = tuple(O.smooth7(n) for n in shape)
    rng = np.random.default_rng(17)
    v = np.stack([synth.plane_wave_velocity(P, 40 + j, 1.0) for j in range(T)])
    if sign != "mixed":
        v = np.abs(v) * (1.0 if sign == "plus" else -1.0)
    v *= dmax * T * h / np.abs(v).max()
    v = v.astype(np.float32)
    M0 = (rng.random(shape) > 0.5).astype(np.float32)
    M1 = (rng.random(shape) > 0.5).astype(np.float32)
    t = lambda a: torch.as_tensor(a, device="cuda")
    prm = L.Params(T=T, iters=(1,))
    g, e = L.lddmm_gradient(t(M0), t(M1), None, None, t(v), prm, kind=L.GRAD_L2, spacing=h)
    g_ref, st, _ = O.gradient(O.Problem(M0, M1), O.Params(T=T, spacing=h), v.astype(np.float64),
                              kind="L2")
    # FP32 samples of random masks: as the other exact-gradient tests
    assert np.abs(g.cpu().numpy() - g_ref).max() < 1e-4 * np.abs(g_ref).max()
    assert abs(float(e[0]) - st["E"]) < 1e-5 * abs(st["E"])

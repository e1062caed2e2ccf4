"""The exact gradient's splat beyond one voxel per step, on grids of many blocks, and with the
reach changing from step to step, so that each of its two kernels leaves steps to the other."""

import numpy as np
import pytest
import torch

from oracle import lddmm as O
from paper_1605_02060_amd import lddmm as L
from paper_1605_02060_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,dmax", [
    ((24, 27, 70), (1.4, 1.4, 1.4)),        # (z, y, x); reach 2 at every step
    ((24, 27, 70), (2.4, 1.9, 2.9)),        # 3, 2, 3
    ((24, 27, 70), (0.9, 1.4, 0.3)),        # 1, 2, 1
    ((32, 32, 32), (2.5, 0.5, 1.0)),        # 3, 1, 2
    ((8, 9, 10), (1.2, 2.2, 0.0)),          # 2, 3, 1 (no displacement)
])
def test_reach_matches_oracle(shape, dmax):
    print(f"[gpu-case] splat reach {shape} {dmax}", flush=True)
    T, h = len(dmax), 0.5
    P = tuple(O.smooth7(n) for n in shape)
    rng = np.random.default_rng(23)
    v = np.stack([synth.plane_wave_velocity(P, 60 + j, 1.0) for j in range(T)])
    for j in range(T):
        v[j] *= dmax[j] * T * h / np.abs(v[j]).max()
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

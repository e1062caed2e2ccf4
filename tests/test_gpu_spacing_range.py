"""Affine resampling and alignment at spacings and translations near the ends of FP64's range: the
position is the quotient by the spacing, as at any other."""

import numpy as np
import pytest
import torch

from paper_1605_02060_amd import lddmm as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interp", [L.INTERP_LINEAR, L.INTERP_NEAREST])
@pytest.mark.parametrize("h", [2.0 ** e for e in (-1040, -400, -333, -332, 0, 332, 333, 400, 1019)])
def test_identity_at_any_spacing(h, interp):
    """dst = src, powers of two around the ends of the fast division: positions x h / h are whole."""
    print(f"[gpu-case] identity at spacing {h} interp {interp}", flush=True)
    src = torch.rand((4, 5, 9), generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    S = np.eye(3, 4)
    out = L.lddmm_apply_affine(src, S, src.shape, src_spacing=h, dst_spacing=h, interp=interp)
    assert torch.equal(out, src)


@pytest.mark.parametrize("interp", [L.INTERP_LINEAR, L.INTERP_NEAREST])
@pytest.mark.parametrize("c,h", [(1e299, 1e-10), (-1e299, 1e-10), (1e250, 1e-70), (1e305, 0.05),
                                 (1e150, 1e-100)])
def test_far_translation_reads_outside(c, h, interp):
    print(f"[gpu-case] translation {c} at spacing {h} interp {interp}", flush=True)
    src = torch.ones((4, 5, 9), device="cuda")
    S = np.eye(3, 4)
    S[:, 3] = c
    out = L.lddmm_apply_affine(src, S, src.shape, src_spacing=h, dst_spacing=h, interp=interp)
    assert torch.equal(out, torch.zeros_like(out))


@pytest.mark.parametrize("h", [1e-120, 1e110])
def test_alignment_value_at_any_spacing(h):
    """The MSE of the identity does not depend on the spacing."""
    print(f"[gpu-case] alignment at spacing {h}", flush=True)
    rng = np.random.default_rng(5)
    I0, I1 = (rng.random((6, 7, 9)).astype(np.float32) for _ in range(2))
    t = lambda a: torch.as_tensor(a, device="cuda")
    _, trace = L.lddmm_align(t(I0), t(I1), affine=np.eye(3, 4), iters=0, template_spacing=h,
                             target_spacing=h)
    E = float(trace[0, 0])
    ref = float(np.mean((I0.astype(np.float64) - I1) ** 2))
    assert abs(E - ref) <= 1e-6 * ref

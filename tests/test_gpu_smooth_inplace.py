"""lddmm_smooth with out == b, which the interface allows, against separate buffers: the same bits
on a grid with fused x + y passes, with compile-time passes, with the plans of single FP32 calls,
with runtime-planned passes, and with b off the 16-byte boundary (copied first)."""

import ctypes

import pytest
import torch

from paper_1605_02060_amd import lddmm as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [(12, 40, 70), (60, 80, 140), (80, 64, 96), (42, 36, 56),
                               (16, 10, 21), (7, 18, 126)])          # z, y, x
@pytest.mark.parametrize("off", [0, 1])
def test_in_place_equals_separate(P, off):
    print(f"[gpu-case] smooth in place {P} offset {off}", flush=True)
    lib = L.load()
    dims = (ctypes.c_int32 * 3)(P[2], P[1], P[0])
    n = 3 * P[0] * P[1] * P[2]
    size = lib.lddmm_smooth_workspace_size(dims)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    b = torch.randn(n, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    want = L.lddmm_smooth(b.view((3,) + P), 0.1, 0.02, 1.0)
    buf = torch.empty(n + 1, device="cuda")
    x = buf[off:off + n]
    x.copy_(b)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = ctypes.c_void_p(x.data_ptr())
    rc = lib.lddmm_smooth(dims, 0.1, 0.02, 1.0, p, p, ctypes.c_void_p(ws.data_ptr()), size, stream)
    assert rc == 0
    assert torch.equal(x.view((3,) + P), want)

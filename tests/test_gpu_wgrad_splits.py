"""The weight gradient over many splits, for every width of its channel blocks: chunk counts
that the splits do not divide, a last split shorter than the others or empty, more and fewer
splits than a multiple of 8.  Oracle, operands and bound as in test_gpu_conv."""

import numpy as np
import pytest
import torch

from oracle import cnn as C
from paper_1605_02060_amd import cnn as G
from test_gpu_cnn import bf, bound, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dims,ci,co,stride", [
    (1, (17, 16, 24), 32, 32, 1),       # 54 chunks, 18 splits of 3 and 6 empty
    (1, (21, 24, 17), 32, 64, 1),       # 99 chunks, 33 splits (32 would leave 7 empty, of 4)
    (1, (29, 20, 24), 192, 64, 1),      # 135 chunks, 22 splits of 6, one of 3, one empty
    (1, (9, 17, 40), 64, 64, 1),        # 75 chunks, 19 splits, the last of 3, 4 empty
    (1, (50, 48, 66), 64, 32, 2),       # 195 chunks, 39 splits of 5, one empty
    (2, (33, 40, 50), 16, 32, 2),       # 216 chunks, 54 splits of 4, 2 empty
    (1, (33, 16, 24), 16, 32, 1),       # 102 chunks, 34 splits of 3, 6 empty
    (1, (25, 24, 24), 2, 16, 1),        # 117 chunks, 39 splits of 3, one empty
])
def test_splits_match_oracle(n, dims, ci, co, stride):
    print(f"[gpu-case] wgrad splits {n} {dims} {ci}->{co} s={stride}", flush=True)
    rng = np.random.default_rng(8)
    xq, xg = bf(rng.normal(size=(n,) + dims + (ci,)))
    dq, dg = bf(rng.normal(size=(n,) + tuple(C.out_size(v, stride) for v in dims) + (co,)))
    dw, db = G.conv3d_backward_weight(dg, xg, stride)
    ref_w, ref_b = C.conv3d_wgrad(dq, xq, stride)
    abs_w, abs_b = C.conv3d_wgrad(np.abs(dq), np.abs(xq), stride)
    K = int(np.prod(dq.shape[:4]))
    assert np.all(np.abs(host(dw) - ref_w) <= bound(K + 1024, abs_w))
    assert np.all(np.abs(host(db) - ref_b) <= bound(K + 1024, abs_b))
    # a run into memory full of NaN: every value is written, and with the same bits
    only = torch.full_like(dw, float("nan"))
    again, _ = G.conv3d_backward_weight(dg, xg, stride, dw=only)
    assert torch.equal(again, dw)

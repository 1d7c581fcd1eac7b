"""Activation transform of rows that are no whole 16-byte pieces, two-byte types: pairs of columns at the ends of a row, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import fused_ops
from paper_2412_05781_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# stored rows of one (single elements), two and three elements, of a strip and one more or less; channels off 64, one and several slabs
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("variant", [B.WINO_F2, B.WINO_F4])
@pytest.mark.parametrize("up", [0, 1])
@pytest.mark.parametrize("C,h,w_", [(8, 5, 1), (72, 3, 2), (130, 4, 3), (64, 9, 7), (136, 6, 9), (64, 7, 15), (8, 8, 17), (200, 5, 33)])
def test_ragged_rows(C, h, w_, up, variant, dtype):
    N, K, H, W = 2, 24, h << up, w_ << up
    if (W * 2) % 16 == 0:
        pytest.skip("whole pieces: another kernel")
    g = torch.Generator().manual_seed(C + 7 * w_ + up)
    x, w = torch.randn(N, C, h, w_, generator=g).to(dtype), (torch.randn(K, C, 3, 3, generator=g) / (9 * C) ** 0.5).to(dtype)
    num = lambda t: t.float().numpy().astype(np.float64)
    ref = oracle.conv2d_general(fused_ops.upsample_nearest2x(num(x)) if up else num(x), num(w), None, 1)
    filt = B.wino_filter_transform(w.to(DEV), variant)
    ws = torch.empty(B.wino_workspace_bytes(N, C, H, W, K, B.DTYPE_OF[dtype], variant), dtype=torch.uint8, device=DEV)
    y = torch.empty(N, K, H, W, dtype=dtype, device=DEV)
    B.wino_conv2d_fused(x.to(DEV), filt, None, y, ws, B.WINO_NCHW, upsample=bool(up))
    torch.cuda.synchronize()
    # the bounds of the storage types' rounding model (fp16: F(2x2) 5.4e-4, F(4x4) 3.1e-3; bf16 eight times), with few outputs twice that; a pair that is shifted
    # or masked wrongly is off by a tenth
    tol = {B.WINO_F2: 1.1e-3, B.WINO_F4: 6.2e-3}[variant] * (8 if dtype == torch.bfloat16 else 1)
    assert oracle.rel_l2(y.float().cpu().numpy(), ref) <= tol

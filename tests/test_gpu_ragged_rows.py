"""Activation transform of rows that are no whole 16-byte pieces, two-byte types: pairs of columns at the ends of a row, bit for bit against images that other
loads read, and against the oracle."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import fused_ops
from paper_2412_05781_amd import binding as B

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAME = {torch.float16: "f16", torch.bfloat16: "bf16"}

# stored rows of one (single elements), two and three elements, of a strip and one more or less; channels off 64, one and several slabs
SHAPES = [(8, 5, 1), (72, 3, 2), (130, 4, 3), (64, 9, 7), (136, 6, 9), (64, 7, 15), (8, 8, 17), (200, 5, 33)]


def _bits(t):
    return t.contiguous().view(torch.int16)


# V of the image, against V of the image with zeros beside it up to whole pieces, which another kernel loads: every tile sees the same window
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("variant", [B.WINO_F2, B.WINO_F4])
@pytest.mark.parametrize("C,H,W", SHAPES)
def test_ragged_rows_bits(C, H, W, variant, dtype):
    N, m, wide = 2, {B.WINO_F2: 2, B.WINO_F4: 4}[variant], -(-W // 8) * 8
    x = torch.randn(N, C, H, W, generator=torch.Generator().manual_seed(C + 5 * W)).to(dtype)
    V = B.wino_input_transform(x.to(DEV), variant)
    P = B.wino_input_transform(torch.nn.functional.pad(x, (0, wide - W)).to(DEV), variant)
    torch.cuda.synchronize()
    th, tw, twp = -(-H // m), -(-W // m), wide // m
    P = P.reshape(P.shape[0], N, th, twp, -1)[:, :, :, :tw]
    assert torch.equal(_bits(V.reshape(P.shape)), _bits(P))


# the whole call: read upsampled and stored upsampled give the same bits, with and without GroupNorm, and both the oracle's result
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("variant", [B.WINO_F2, B.WINO_F4])
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("C,h,w_", SHAPES)
def test_ragged_rows(C, h, w_, norm, variant, dtype):
    N, K, groups = 2, 24, 2
    g = torch.Generator().manual_seed(C + 7 * w_ + norm)
    x, w = torch.randn(N, C, h, w_, generator=g).to(dtype), (torch.randn(K, C, 3, 3, generator=g) / (9 * C) ** 0.5).to(dtype)
    gamma, beta = 1.0 + 0.1 * torch.randn(C, generator=g), 0.5 + 0.1 * torch.randn(C, generator=g)
    filt = B.wino_filter_transform(w.to(DEV), variant)
    fused = dict(gn_stats=B.wino_groupnorm_stats(x.to(DEV), groups), gn_gamma=gamma.to(DEV), gn_beta=beta.to(DEV), gn_groups=groups) if norm else {}
    num = lambda t: t.float().numpy().astype(np.float64)

    def run(image, up):
        H, W = image.shape[2] << up, image.shape[3] << up
        assert routes.onepass(N, C, K, H, W, NAME[dtype], False, norm=norm, up=bool(up))[0] == 0
        ws = torch.empty(B.wino_workspace_bytes(N, C, H, W, K, B.DTYPE_OF[dtype], variant), dtype=torch.uint8, device=DEV)
        y = torch.empty(N, K, H, W, dtype=dtype, device=DEV)
        B.wino_conv2d_fused(image.to(DEV), filt, None, y, ws, B.WINO_NCHW, upsample=bool(up), **fused)
        torch.cuda.synchronize()
        return y

    big = x.repeat_interleave(2, 2).repeat_interleave(2, 3)
    small, read, stored = run(x, 0), run(x, 1), run(big, 0)
    assert torch.equal(_bits(read), _bits(stored))
    # the bounds of the storage types' rounding model (fp16: F(2x2) 5.4e-4, F(4x4) 3.1e-3; bf16 eight times), with few outputs twice that; GroupNorm
    # is applied in fp32 and rounds nothing more
    tol = {B.WINO_F2: 1.1e-3, B.WINO_F4: 6.2e-3}[variant] * (8 if dtype == torch.bfloat16 else 1)
    for image, y, up in ((x, small, 0), (x, read, 1)):
        xs = fused_ops.silu(fused_ops.groupnorm(num(x), num(gamma), num(beta), groups)) if norm else num(x)
        ref = oracle.conv2d_general(fused_ops.upsample_nearest2x(xs) if up else xs, num(w), None, 1)
        assert oracle.rel_l2(y.float().cpu().numpy(), ref) <= tol

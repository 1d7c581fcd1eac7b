"""The blocks of the 16x16-tile direct kernel at the edges of their range, against the fp64 oracle, element by element."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import fused_ops
from paper_2412_05781_amd import binding as B
from paper_2412_05781_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one stage and several (fewer than the ring has slots, and more), tails in pixels and channels, images of one pixel, row and column (taps
# outside on both sides), channels and pixels that are no multiple of four, split reductions
CASES = [((1, 64, 16, 1, 1), 3, 1, 5), ((1, 64, 8, 1, 7), 3, 2, 5), ((1, 128, 24, 130, 127), 3, 1, 5), ((2, 192, 32, 33, 20), 1, 1, 5), ((1, 384, 64, 131, 130), 3, 1, 0), ((1, 128, 70, 9, 1), 3, 1, 0), ((2, 192, 33, 7, 9), 1, 2, 5), ((1, 1280, 40, 9, 6), 3, 2, 5), ((2, 192, 70, 7, 9), 1, 2, 0), ((1, 1280, 72, 9, 6), 3, 2, 0),
         ((2, 128, 192, 97, 95), 1, 1, 1), ((1, 192, 64, 300, 299), 1, 1, 1), ((1, 64, 190, 130, 127), 3, 1, 1), ((1, 704, 144, 57, 54), 3, 1, 1), ((2, 192, 320, 64, 63), 1, 1, 3),
         ((2, 64, 96, 128, 128), 1, 1, 2), ((1, 128, 500, 70, 121), 3, 1, 2), ((2, 64, 264, 65, 63), 3, 1, 3), ((1, 64, 130, 257, 254), 3, 2, 3),
         ((2, 64, 240, 128, 126), 1, 1, 4), ((2, 192, 330, 128, 126), 3, 1, 4),
         ((2, 64, 66, 181, 179), 3, 2, 6), ((1, 128, 130, 190, 131), 3, 2, 6), ((1, 832, 68, 95, 61), 3, 1, 6)]


def _check(y, ref, layout, dtype):
    y = y.float().cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)
    # only the output is rounded: half a unit in the last place, plus fp32 sums of up to 11520 products
    half_ulp = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8
    assert np.all(np.abs(y - ref) <= 1.001 * half_ulp * np.abs(ref) + 3e-5), np.abs(y - ref).max()


def _inputs(N, C, K, H, W, R, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    td = synth.TORCH_DTYPE[dtype]
    return (torch.randn(N, C, H, W, generator=g).to(td), (torch.randn(K, C, R, R, generator=g) / (R * R * C) ** 0.5).to(td),
            torch.randn(K, generator=g) * 0.1)


def _np(t):
    return t.float().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("shape,R,stride,block", CASES)
def test_block(shape, R, stride, block, layout, dtype):
    N, C, K, H, W = shape
    assert routes.block_plan(*shape, R, stride, dtype, layout == B.WINO_NHWC)[0] == block
    x, w, b = _inputs(*shape, R, dtype, 9100 + sum(shape))
    ref = oracle.conv2d_general(_np(x), _np(w), _np(b), stride)
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d_igemm(xd, w.to(DEV), b.to(DEV), stride, layout)
    torch.cuda.synchronize()
    _check(y, ref, layout, dtype)


# the additions of the epilogue and the upsampled read, on a block with whole and one with ragged channel groups; K = 66 and 22x17 pixels take the
# element-wise stores
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("N,C,K,h,w_", [(2, 64, 72, 9, 8), (1, 128, 66, 11, 7), (2, 64, 96, 64, 64), (2, 64, 264, 32, 34)])
@pytest.mark.parametrize("up", [0, 1])
def test_additions_and_upsampling(N, C, K, h, w_, up, layout, dtype):
    x, w, b = _inputs(N, C, K, h, w_, 3, dtype, 9300 + K + h)
    g = torch.Generator().manual_seed(K)
    td = synth.TORCH_DTYPE[dtype]
    H, W = h << up, w_ << up
    vec, res = torch.randn(N, K, generator=g), torch.randn(N, K, H, W, generator=g).to(td)
    xs = fused_ops.upsample_nearest2x(_np(x)) if up else _np(x)
    ref = oracle.conv2d_general(xs, _np(w), _np(b), 1) + _np(vec)[:, :, None, None] + _np(res)
    lay = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    filt = B.wino_filter_transform(w.to(DEV), B.WINO_DIRECT)
    ws = torch.empty(max(16, B.wino_workspace_bytes(N, C, H, W, K, B.DTYPE_OF[td], B.WINO_DIRECT)), dtype=torch.uint8, device=DEV)
    y = torch.empty_like(lay(res).to(DEV))
    B.wino_conv2d_fused(lay(x).to(DEV), filt, b.to(DEV), y, ws, layout, addvec=vec.to(DEV), residual=lay(res).to(DEV), upsample=bool(up))
    torch.cuda.synchronize()
    _check(y, ref, layout, dtype)

"""8-bit direct path, 3x3 at stride 1, where the three taps of a filter row share one fetch of the pixels: against the quantisation model."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import fp8_model as f8
from paper_2412_05781_amd import binding as B

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HALF_ULP = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}


# one and several chunks of channels, the last one partial; blocks that straddle images and rows, images one pixel wide and one high, planes of whole
# 16-byte pieces, pairs and an odd number of pixels, tails in pixels and channels; 256x256 blocks in NCHW (the last three; the last of
# all goes to another kernel channel-last)
CASES = [(1, 48, 20, 160, 161), (2, 144, 136, 113, 119), (1, 64, 200, 1, 13000), (1, 128, 200, 16385, 1), (3, 16, 300, 8, 460), (2, 400, 72, 100, 130), (1, 128, 132, 96, 136),
         (1, 144, 256, 256, 255), (1, 272, 250, 251, 258), (2, 256, 256, 128, 256)]


@pytest.mark.parametrize("additions", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("shape", CASES)
def test_rows(shape, layout, dtype, additions):
    N, C, K, H, W = shape
    assert routes.fp8_rows(*shape, dtype, layout == B.WINO_NHWC) == (layout == B.WINO_NCHW or shape != CASES[-1], layout == B.WINO_NCHW and shape in CASES[-3:])
    td = torch.float16 if dtype == "f16" else torch.bfloat16
    g = torch.Generator().manual_seed(700 + sum(shape))
    x, w = torch.randn(N, C, H, W, generator=g).to(td), (torch.randn(K, C, 3, 3, generator=g) / (9 * C) ** 0.5).to(td)
    b, vec, res = torch.randn(K, generator=g) * 0.1, torch.randn(N, K, generator=g), torch.randn(N, K, H, W, generator=g).to(td)
    num = lambda t: t.float().numpy().astype(np.float64)
    sx, sw = f8.power_of_two_scale(num(x)), f8.power_of_two_scale(num(w))
    ref = f8.conv2d_fp8(num(x), num(w), num(b), sx, sw, 1)
    if additions:
        ref = ref + num(vec)[:, :, None, None] + num(res)
    lay = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    kw = dict(addvec=vec.to(DEV), residual=lay(res).to(DEV)) if additions else {}
    y = B.conv2d_fp8(lay(x).to(DEV), w.to(DEV), b.to(DEV), sx, sw, 1, layout, **kw)
    torch.cuda.synchronize()
    y = y.float().cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)
    # The operands are exact and y is rounded once: half a unit in the last place of an output and, in the tensor's norm, less than 0.6 of that.  The
    # matrix instruction drops what lies beyond its alignment of 64 products, whose largest are some hundred times their sum: an eighth of a unit of
    # the largest output covers it (measured: a tenth of that).  A tap that is missing or too many is off by a hundred times as much.
    assert np.all(np.abs(y - ref) <= HALF_ULP[dtype] * np.abs(ref) + 0.25 * HALF_ULP["f16"] * np.abs(ref).max()), np.abs(y - ref).max()
    assert oracle.rel_l2(y, ref) <= 0.6 * HALF_ULP[dtype]

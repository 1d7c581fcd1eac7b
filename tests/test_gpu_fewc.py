"""The one-kernel F(4x4) path for few input channels in fp32 (csrc/wino_fewc.hip), against the fp64 oracle.

Tolerance: relative L2 1e-5 as for every fp32 path (measured 5e-7...8e-7), and element by element the bound of
tests/parity_util.py, which catches one wrong tile."""
import os
import sys

import numpy as np
import pytest
import torch

from oracle import fused_ops as fo
from paper_2412_05781_amd import binding as B
from paper_2412_05781_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity_util  # noqa: E402
import routes  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _np(t):
    return None if t is None else t.float().numpy().astype(np.float64)


# tile counts around the 16 of a wave, rows of tiles shorter and longer than 16, sizes off the tile edge, channels around
# the chunk of 8 and the limit of 16 (17 runs the chain), output channels off 16 and off 4; with the layouts that the one-kernel
# path takes (NCHW, channel-last), the others run the chain; the last has four workgroups to a compute unit
CASES = [((1, 4, 320, 64, 64), (True, True)), ((2, 9, 33, 5, 7), (False, False)), ((1, 1, 1, 1, 1), (True, False)), ((3, 16, 18, 4, 60), (False, False)),
         ((1, 8, 16, 68, 68), (True, True)), ((2, 15, 21, 9, 66), (False, False)), ((1, 17, 16, 8, 64), (False, False)), ((1, 5, 20, 6, 130), (True, True)),
         ((2, 7, 21, 9, 66), (True, False)), ((3, 8, 20, 4, 60), (True, True)), ((1, 6, 4, 3, 2), (True, True)), ((2, 9, 164, 90, 95), (True, True)), ((2, 16, 136, 66, 124), (True, True)),
         ((2, 15, 277, 70, 131), (True, True)), ((1, 5, 33, 258, 130), (True, True)), ((1, 16, 224, 251, 64), (True, True))]


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("post", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_few_channels(case, post, layout):
    case, taken = case
    N, C, K, H, W = case
    assert routes.fewc(N, C, K, H, W, "f32", layout == B.WINO_NHWC) == taken[layout == B.WINO_NHWC]
    x, w, b = synth.make_inputs(N, C, K, H, W, "f32", seed=500 + sum(case))
    g = torch.Generator().manual_seed(sum(case))
    addvec = torch.randn(N, K, generator=g) if post else None
    residual = torch.randn(N, K, H, W, generator=g) if post else None
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    dev = lambda t: None if t is None else t.to(DEV)
    y = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F4, layout, addvec=dev(addvec),
                       residual=dev(perm(residual)) if post else None)
    torch.cuda.synchronize()
    y = y.cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)
    ref = fo.conv2d_fused(_np(x), _np(w), _np(b), addvec=_np(addvec), residual=_np(residual))
    parity_util.check(y, ref, 1e-5, 4, "f32", what=(case, post, layout), channels=C)


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
def test_few_channels_upsampled(layout):
    N, C, K, h, w_ = 2, 6, 20, 9, 17
    assert routes.fewc(N, C, K, 2 * h, 2 * w_, "f32", layout == B.WINO_NHWC, up=True)
    x, w, b = synth.make_inputs(N, C, K, h, w_, "f32", seed=77)
    up = x.repeat_interleave(2, 2).repeat_interleave(2, 3).contiguous()
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    a = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F4, layout, upsample=True)
    c = B.conv2d(perm(up).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F4, layout)
    assert torch.equal(a, c)

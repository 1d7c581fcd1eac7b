"""The one-kernel F(2x2) path (csrc/wino_onepass.hip) against the fp64 oracle, element by element.

Tolerances: those of F(2x2) for the storage type (fp16 5e-3 with the variant's band around 5e-4, bf16 8e-3 around 4e-3), and the
element-wise bound of tests/parity_util.py.  The shapes are large enough for the library to take this path (about 130 blocks
of 4 x 8 tiles and output channels) and sit at its edges: tile rows and columns off the block, odd images, one and several
64-channel chunks, every number of 16-channel sub-tiles per wave, output channels off the block, rows that are and are not
whole 16-byte pieces."""
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

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {"f16": 1e-3, "bf16": 8e-3}


def _np(t):
    return None if t is None else t.float().numpy().astype(np.float64)


CASES = [(1, 64, 48, 127, 129), (2, 64, 160, 66, 74), (2, 128, 96, 64, 136), (1, 192, 144, 97, 96), (1, 64, 320, 101, 72), (1, 64, 16, 250, 126),
         (2, 64, 320, 128, 120)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_onepass(case, fused, layout, dtype):
    N, C, K, H, W = case
    td = synth.TORCH_DTYPE[dtype]
    x, w, b = synth.make_inputs(N, C, K, H, W, dtype, seed=900 + sum(case))
    g = torch.Generator().manual_seed(sum(case))
    gamma = beta = addvec = residual = None
    if fused:
        gamma, beta = 1 + 0.2 * torch.randn(C, generator=g), 0.3 * torch.randn(C, generator=g)
        addvec, residual = torch.randn(N, K, generator=g), torch.randn(N, K, H, W, generator=g).to(td)
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    dev = lambda t: None if t is None else t.to(DEV)
    y = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F2, layout, dev(gamma), dev(beta), 16, 1e-5, dev(addvec),
                       dev(perm(residual)) if fused else None)
    torch.cuda.synchronize()
    y = y.float().cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)
    ref = fo.conv2d_fused(_np(x), _np(w), _np(b), _np(gamma), _np(beta), 16, 1e-5, _np(addvec), _np(residual))
    parity_util.check(y, ref, TOL[dtype], 2, dtype, what=(case, fused, layout, dtype))


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
def test_onepass_upsampled(layout):
    N, C, K, h, w_ = 2, 64, 96, 36, 40
    x, w, b = synth.make_inputs(N, C, K, h, w_, "bf16", seed=78)
    up = x.repeat_interleave(2, 2).repeat_interleave(2, 3).contiguous()
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    a = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F2, layout, upsample=True)
    c = B.conv2d(perm(up).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F2, layout)
    assert torch.equal(a, c)

"""The one-kernel F(2x2) path (csrc/wino_onepass.hip) against the fp64 oracle, element by element.

Tolerances: those of F(2x2) for the storage type (fp16 5e-3 with the variant's band around 5e-4, bf16 8e-3 around 4e-3), and the
element-wise bound of tests/parity_util.py.  The shapes are large enough for the library to take this path (about 130 blocks
of 4 x 8 tiles and output channels; each test asks the rule for the kernel that it means) and sit at its edges: tile rows and columns off the block, odd images, one and several
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
import routes  # noqa: E402

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
    assert routes.onepass(N, C, K, H, W, dtype, layout == B.WINO_NHWC, norm=fused, residual=fused)[0] > 0
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


# every number of sub-tiles per wave with two and three chunks of 64 channels, for rows that are read element by element (mode 2: off the
# 16-byte piece, or upsampled), in whole pieces (1) and channel-last (0): the pixels of the next chunk are loaded and GroupNorm's
# coefficients replaced during the products of this one, and the filter ring goes on over the end of a chunk
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("variant,dtype", [(B.WINO_F2, "f16"), (B.WINO_F2, "bf16"), (B.WINO_FUSED_F2, "bf16")])
@pytest.mark.parametrize("ns,mode,up,case", [
    (2, 2, False, (1, 192, 16, 150, 130)), (2, 2, False, (1, 128, 48, 151, 131)), (2, 2, True, (1, 192, 16, 160, 120)), (3, 2, False, (2, 192, 80, 122, 102)),
    (3, 2, True, (1, 128, 96, 160, 120)), (4, 2, False, (2, 192, 112, 122, 102)), (4, 2, False, (1, 128, 112, 180, 130)), (4, 2, True, (1, 128, 112, 200, 136)),
    (4, 1, False, (1, 192, 320, 101, 72)), (5, 1, False, (1, 192, 400, 101, 72)),
    (2, 0, False, (1, 192, 16, 97, 75)), (3, 0, False, (1, 192, 400, 66, 66)), (4, 0, False, (2, 128, 240, 66, 66)), (4, 0, False, (1, 192, 320, 101, 72)),
    (5, 0, False, (2, 128, 320, 66, 66)), (5, 0, False, (1, 192, 400, 101, 72)), (5, 0, True, (2, 192, 320, 66, 66))])
def test_onepass_chunks(ns, mode, up, case, variant, dtype, norm):
    N, C, K, H, W = case
    layout = B.WINO_NHWC if mode == 0 else B.WINO_NCHW
    assert routes.onepass(N, C, K, H, W, dtype, mode == 0, variant == B.WINO_FUSED_F2, norm, up) == (ns, mode)
    h, w_ = (H // 2, W // 2) if up else (H, W)
    x, _, _ = synth.make_inputs(N, C, K, h, w_, dtype, seed=1300 + sum(case))
    _, w, b = synth.make_inputs(1, C, K, 4, 4, dtype, seed=1400 + sum(case))
    g = torch.Generator().manual_seed(sum(case))
    gamma, beta = (1 + 0.2 * torch.randn(C, generator=g), 0.3 * torch.randn(C, generator=g)) if norm else (None, None)
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    dev = lambda t: None if t is None else t.to(DEV)
    y = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), variant, layout, dev(gamma), dev(beta), 16, upsample=up)
    torch.cuda.synchronize()
    y = y.float().cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)
    ref = fo.conv2d_fused(_np(x), _np(w), _np(b), _np(gamma), _np(beta), 16, upsample=up)
    parity_util.check(y, ref, TOL[dtype], 2, dtype, what=(ns, mode, up, case, variant, dtype, norm), channels=C)


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
def test_onepass_upsampled(layout):
    N, C, K, h, w_ = 2, 64, 96, 36, 40
    assert routes.onepass(N, C, K, 2 * h, 2 * w_, "bf16", layout == B.WINO_NHWC, up=True)[0] > 0
    x, w, b = synth.make_inputs(N, C, K, h, w_, "bf16", seed=78)
    up = x.repeat_interleave(2, 2).repeat_interleave(2, 3).contiguous()
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    a = B.conv2d_fused(perm(x).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F2, layout, upsample=True)
    c = B.conv2d(perm(up).to(DEV), w.to(DEV), b.to(DEV), B.WINO_F2, layout)
    assert torch.equal(a, c)

"""The 8-bit (E4M3) direct convolution path against the oracle's quantisation model (oracle/fp8_model.py).

Two kinds of check: (1) against the MODEL of the quantised convolution - same quantised operands, exact products - the
GPU result differs only by fp32 accumulation and the output rounding, so the tolerance is that of the storage type of y;
this also proves that the kernel's roundings to E4M3 are the model's.  (2) against the UNquantised fp64 convolution the
error must sit in the band the model predicts (about 3.8e-2; tolerance of the path 6e-2)."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import fp8_model as f8
from oracle import fused_ops as fo
from paper_2412_05781_amd import binding as B
from paper_2412_05781_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OUT_TOL = {"f32": 1e-4, "f16": 6e-4, "bf16": 3e-3}      # against the model: the accumulation inside the 8-bit MFMA (measured ~1e-5) + one rounding of y


def _np(t):
    return None if t is None else t.float().numpy().astype(np.float64)


def _inputs(N, C, K, H, W, R, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    tdt = synth.TORCH_DTYPE[dtype]
    x = torch.randn(N, C, H, W, generator=g).to(tdt)
    w = (torch.randn(K, C, R, R, generator=g) / (R * R * C) ** 0.5).to(tdt)
    b = torch.randn(K, generator=g) * 0.1
    return x, w, b


SHAPES = [(1, 1, 1, 1, 1), (2, 5, 7, 6, 9), (1, 24, 40, 13, 18), (2, 72, 136, 17, 15), (1, 320, 200, 16, 16), (1, 130, 64, 33, 40),
          (2, 640, 96, 8, 8)]


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("R,stride", [(3, 1), (1, 1), (3, 2)])
@pytest.mark.parametrize("shape", SHAPES)
def test_fp8_against_the_quantisation_model(shape, R, stride, layout, dtype):
    N, C, K, H, W = shape
    x, w, b = _inputs(N, C, K, H, W, R, dtype, seed=15000 + sum(shape) + 10 * R + stride)
    sx, sw = f8.power_of_two_scale(_np(x)), f8.power_of_two_scale(_np(w))
    model = f8.conv2d_fp8(_np(x), _np(w), _np(b), sx, sw, stride)
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d_fp8(xd, w.to(DEV), b.to(DEV), sx, sw, stride, layout)
    torch.cuda.synchronize()
    y = y.float().cpu()
    if layout == B.WINO_NHWC:
        y = y.permute(0, 3, 1, 2)
    assert tuple(y.shape) == model.shape
    err = oracle.rel_l2(y.numpy(), model)
    assert err <= OUT_TOL[dtype], (shape, R, stride, layout, dtype, err)


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
def test_fp8_error_band_against_the_exact_convolution(layout):
    N, C, K, H, W = 2, 320, 96, 24, 24
    x, w, b = _inputs(N, C, K, H, W, 3, "f16", seed=3)
    ref = oracle.conv2d_general(_np(x), _np(w), None, 1)
    sx, sw = f8.power_of_two_scale(_np(x)), f8.power_of_two_scale(_np(w))
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d_fp8(xd, w.to(DEV), None, sx, sw, 1, layout)
    torch.cuda.synchronize()
    y = y.float().cpu()
    if layout == B.WINO_NHWC:
        y = y.permute(0, 3, 1, 2)
    err = oracle.rel_l2(y.numpy(), ref)
    assert 3.0e-2 <= err <= 4.5e-2 and err <= 6e-2, err


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_fp8_fused_operators(dtype, layout):
    """GroupNorm + SiLU before the quantisation, upsampling by address arithmetic, vector and residual adds after."""
    N, C, K, h, w_, G = 1, 64, 72, 8, 12, 8
    x, w, b = _inputs(N, C, K, h, w_, 3, dtype, seed=21)
    g = torch.Generator().manual_seed(9)
    gamma, beta = 1.0 + 0.2 * torch.randn(C, generator=g), 0.3 * torch.randn(C, generator=g)
    addvec = 0.5 * torch.randn(N, K, generator=g)
    residual = torch.randn(N, K, 2 * h, 2 * w_, generator=g).to(x.dtype)
    act = fo.upsample_nearest2x(fo.silu(fo.groupnorm(_np(x), _np(gamma), _np(beta), G, 1e-5)))
    sx, sw = f8.power_of_two_scale(act), f8.power_of_two_scale(_np(w))
    model = f8.conv2d_fp8(act, _np(w), _np(b), sx, sw) + _np(addvec)[:, :, None, None] + _np(residual)
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    y = B.conv2d_fp8(perm(x).to(DEV), w.to(DEV), b.to(DEV), sx, sw, 1, layout, gn_gamma=gamma.to(DEV), gn_beta=beta.to(DEV),
                     gn_groups=G, addvec=addvec.to(DEV), residual=perm(residual).to(DEV), upsample=True)
    torch.cuda.synchronize()
    y = y.float().cpu()
    if layout == B.WINO_NHWC:
        y = y.permute(0, 3, 1, 2)
    # the activation is computed in fp32 on the GPU and in fp64 in the model: a value that sits on a rounding boundary of
    # E4M3 may fall on the other side, so a handful of operands differ by one step; far below the 3.8e-2 of the format
    err = oracle.rel_l2(y.numpy(), model)
    assert err <= 5e-3, (dtype, layout, err)
    exact = fo.conv2d_fused(_np(x), _np(w), _np(b), _np(gamma), _np(beta), G, 1e-5, _np(addvec), _np(residual), upsample=True)
    assert oracle.rel_l2(y.numpy(), exact) <= 6e-2


# the kernel for whole reductions: blocks of 256x256 with one and several stages, the last one partial, blocks that straddle two images,
# planes that are and are not whole 16-byte pieces; blocks of 128x128 off the edge in both dimensions, images of an odd and an even number of
# pixels, stride 1; additions at the end; with the layouts that the kernel takes (NCHW, channel-last), the others run the older one
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("case,taken", [((2, 272, 256, 180, 184, 1), (True, False)), ((2, 80, 256, 181, 182, 1), (True, False)),
                                        ((1, 384, 256, 255, 259, 1), (True, False)), ((1, 112, 200, 24, 40, 3), (True, False)),
                                        ((2, 48, 136, 25, 40, 3), (True, False)), ((3, 112, 72, 9, 11, 3), (False, False)),
                                        ((1, 272, 136, 128, 129, 1), (True, True)), ((1, 128, 136, 128, 129, 3), (True, True)), ((2, 48, 330, 101, 99, 3), (True, True)),
                                        ((1, 112, 260, 150, 121, 3), (True, True)), ((2, 112, 7, 19, 23, 3), (False, True)), ((1, 144, 28, 9, 13, 1), (False, True)), ((3, 128, 1, 8, 16, 3), (False, True))])
def test_fp8_whole_reductions(case, taken, layout):
    N, C, K, H, W, R = case
    assert routes.fp8_tile(N, C, K, H, W, R, 1, "f16", layout == B.WINO_NHWC) == taken[layout == B.WINO_NHWC]
    x, w, b = _inputs(N, C, K, H, W, R, "f16", seed=400 + sum(case))
    g = torch.Generator().manual_seed(sum(case))
    addvec, residual = torch.randn(N, K, generator=g), torch.randn(N, K, H, W, generator=g).half()
    sx, sw = f8.power_of_two_scale(_np(x)), f8.power_of_two_scale(_np(w))
    model = f8.conv2d_fp8(_np(x), _np(w), _np(b), sx, sw, 1) + _np(addvec)[:, :, None, None] + _np(residual)
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    y = B.conv2d_fp8(perm(x).to(DEV), w.to(DEV), b.to(DEV), sx, sw, 1, layout, addvec=addvec.to(DEV), residual=perm(residual).to(DEV))
    y = y.float().cpu()
    y = (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy()
    assert oracle.rel_l2(y, model) <= OUT_TOL["f16"], (case, layout)
    assert np.abs(y - model).max() <= 4e-3 * np.abs(model).max(), (case, layout)       # two roundings of the largest output and the accumulation


@pytest.mark.parametrize("name,layout", [("E2_vae", B.WINO_NHWC), ("E3_vae", B.WINO_NCHW), ("C6_unet", B.WINO_NCHW)])
def test_fp8_full_size_layers_sampled(name, layout):
    """Full-size layers (256x256 blocks of 16 and of eight waves; a split reduction on the 8x8 one): 4096 sampled outputs and the
    image corners against the quantisation model, evaluated one output at a time."""
    layer = synth.LAYERS[name]
    x, w, b = synth.make_layer_inputs(layer)
    xn, wn = _np(x), _np(w)
    sx, sw = f8.power_of_two_scale(xn), f8.power_of_two_scale(wn)
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d_fp8(xd, w.to(DEV), b.to(DEV), sx, sw, 1, layout)
    torch.cuda.synchronize()
    y = y.float().cpu()
    if layout == B.WINO_NHWC:
        y = y.permute(0, 3, 1, 2)
    y = y.contiguous().numpy()
    rng = np.random.default_rng(layer.index)
    idx = rng.integers(0, y.size, size=4096)
    H, W = layer.H, layer.W
    idx[:5] = [0, W - 1, (H - 1) * W, H * W - 1, y.size - 1]
    xq, wq = f8.round_to_e4m3(xn * sx), f8.round_to_e4m3(wn * sw)
    ref = oracle.conv2d_direct_at(xq, wq, None, idx) / (sx * sw) + _np(b)[(idx // (H * W)) % layer.K]
    err = np.linalg.norm(y.ravel()[idx] - ref) / np.linalg.norm(ref)
    assert err <= OUT_TOL["f16"], (name, err)
    assert np.isfinite(y).all()


def test_fp8_argument_checks_and_sizes():
    assert B.wino_fp8_filter_bytes(8, 20, 3) == 9 * 8 * 32 + 32          # C rounded up to 16
    assert B.wino_fp8_filter_bytes(8, 8, 2) == 0
    assert B.wino_fp8_workspace_bytes(1, 20, 4, 4, 8, 3, 1) >= 16 * 32
    x, w, b = _inputs(1, 8, 8, 8, 8, 3, "f16", seed=1)
    xd, wd = x.to(DEV), w.to(DEV)
    w_q = B.wino_fp8_filter_quantize(wd, 64.0)
    y = torch.empty((1, 8, 8, 8), dtype=torch.float16, device=DEV)
    ws = torch.empty(B.wino_fp8_workspace_bytes(1, 8, 8, 8, 8, 3, 1), dtype=torch.uint8, device=DEV)
    L = B.lib()
    import ctypes
    cf = ctypes.c_float
    args = lambda **kw: [kw.get("x", xd.data_ptr()), w_q.data_ptr(), None, y.data_ptr(), 1, 8, 8, 8, 8, kw.get("R", 3), kw.get("st", 1),
                         kw.get("dt", B.WINO_F16), kw.get("layout", B.WINO_NCHW), cf(kw.get("sx", 64.0)), cf(64.0), None,
                         ws.data_ptr(), kw.get("wsb", ws.numel()), None]
    assert L.wino_fp8_conv2d(*args()) == B.WINO_OK
    assert L.wino_fp8_conv2d(*args(R=5)) == B.WINO_ERR_DIM
    assert L.wino_fp8_conv2d(*args(sx=0.0)) == B.WINO_ERR_DIM
    assert L.wino_fp8_conv2d(*args(sx=float("nan"))) == B.WINO_ERR_DIM
    assert L.wino_fp8_conv2d(*args(dt=9)) == B.WINO_ERR_DTYPE
    assert L.wino_fp8_conv2d(*args(layout=4)) == B.WINO_ERR_LAYOUT
    assert L.wino_fp8_conv2d(*args(wsb=8)) == B.WINO_ERR_WORKSPACE
    assert L.wino_fp8_conv2d(*args(x=None)) == B.WINO_ERR_NULL
    torch.cuda.synchronize()

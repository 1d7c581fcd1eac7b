"""WINO_FUSED_F2: steps (ii) and (iii) of Section "Techniques" in one kernel (the product of step (ii) is scattered
into the output accumulators position by position and never stored).  Parity against the CPU oracle, element by
element, through the C ABI; every block shape of the kernel on small ragged inputs; both layouts; all storage types;
agreement with the unfused F(2x2) path, whose sums it re-orders only in fp32."""
import os
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2412_05781_amd import binding as B
from paper_2412_05781_amd import synth

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity_util as pu  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {"f32": 1e-5, "f16": 5e-3, "bf16": 8e-3}

# N, C, K, H, W: odd sizes, ragged tiles, channel counts off every block edge, more rows / columns than one block
SHAPES = [(1, 1, 1, 1, 1), (1, 4, 3, 2, 3), (2, 5, 7, 5, 7), (1, 33, 65, 17, 30), (2, 64, 130, 33, 9), (1, 100, 40, 12, 40),
          (2, 136, 200, 16, 16), (1, 72, 129, 70, 6), (1, 200, 150, 37, 41)]


def _np(t):
    return t.float().numpy().astype(np.float64)


def _nchw(y, layout):
    y = y.float().cpu()
    return (y.permute(0, 3, 1, 2) if layout == B.WINO_NHWC else y).numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("shape", SHAPES)
def test_whole_path_small_shapes(shape, layout, dtype):
    N, C, K, H, W = shape
    x, w, b = synth.make_inputs(N, C, K, H, W, dtype, seed=7000 + sum(shape))
    ref = oracle.conv2d_direct(_np(x), _np(w), _np(b))
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d(xd, w.to(DEV), b.to(DEV), B.WINO_FUSED_F2, layout=layout)
    torch.cuda.synchronize()
    pu.check(_nchw(y, layout), ref, TOL[dtype], 2, dtype, what=(shape, layout, dtype), channels=C)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("block_shape", [0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("shape", [(2, 5, 7, 5, 7), (1, 33, 65, 17, 30), (2, 136, 200, 16, 16), (1, 200, 150, 37, 41), (1, 72, 300, 21, 39),
                                   (1, 64, 200, 30, 34), (2, 128, 320, 16, 32), (1, 192, 130, 64, 64)])
def test_every_block_shape(shape, block_shape, layout, dtype):
    """The stage call with a named block shape: each instantiation on inputs with ragged rows and columns, a ragged
    last reduction stage (C not a multiple of 64 / 32) and more than one block in both directions."""
    N, C, K, H, W = shape
    x, w, b = synth.make_inputs(N, C, K, H, W, dtype, seed=7100 + sum(shape))
    ref = oracle.conv2d_direct(_np(x), _np(w), _np(b))
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    filt = B.wino_filter_transform(w.to(DEV), B.WINO_FUSED_F2)
    assert filt.desc.variant == B.WINO_FUSED_F2
    U = filt.buf.view(x.dtype)
    V = B.wino_input_transform(xd, B.WINO_FUSED_F2, layout=layout)
    y = B.wino_fused_gemm_output(U, V, b.to(DEV), N, C, H, W, K, layout=layout, block_shape=block_shape)
    torch.cuda.synchronize()
    pu.check(_nchw(y, layout), ref, TOL[dtype], 2, dtype, what=(shape, block_shape, layout, dtype), channels=C)
    # the library's own choice of block differs at most in the order of fp32 additions
    y_auto = B.wino_fused_gemm_output(U, V, b.to(DEV), N, C, H, W, K, layout=layout)
    torch.cuda.synchronize()
    d = (y.float() - y_auto.float()).abs().max().item()
    assert d <= (2.0 ** -9 if dtype == "f16" else 1e-5) * max(1.0, y.float().abs().max().item())


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
def test_agrees_with_the_unfused_path(layout):
    """Same U and V as WINO_F2; the product is added into the outputs in fp32 in another order, so the two results
    differ by fp32 rounding before the one rounding to fp16: at most one unit in the last place, on few elements."""
    N, C, K, H, W = 2, 96, 80, 20, 22
    x, w, b = synth.make_inputs(N, C, K, H, W, "f16", seed=31)
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y1 = B.conv2d(xd, w.to(DEV), b.to(DEV), B.WINO_F2, layout=layout)
    y2 = B.conv2d(xd, w.to(DEV), b.to(DEV), B.WINO_FUSED_F2, layout=layout)
    torch.cuda.synchronize()
    d = (y1.float() - y2.float()).abs()
    assert d.max().item() <= 2.0 ** -10 * y1.float().abs().max().item()
    assert (d > 0).float().mean().item() < 0.05
    # workspace: V only
    assert B.wino_workspace_bytes(N, C, H, W, K, B.WINO_F16, B.WINO_FUSED_F2) < B.wino_workspace_bytes(N, C, H, W, K, B.WINO_F16, B.WINO_F2)


def test_zero_input_no_bias_and_determinism():
    x, w, b = synth.make_inputs(2, 40, 24, 10, 11, "f16", seed=5)
    xd, wd, bd = x.to(DEV), w.to(DEV), b.to(DEV)
    y0 = B.conv2d(torch.zeros_like(xd), wd, bd, B.WINO_FUSED_F2)
    torch.cuda.synchronize()
    assert torch.equal(y0.float().cpu(), b.to(torch.float16).float().view(1, -1, 1, 1).expand(2, 24, 10, 11))
    ref = oracle.conv2d_direct(_np(x), _np(w), None)
    y = B.conv2d(xd, wd, None, B.WINO_FUSED_F2)
    y_again = B.conv2d(xd, wd, None, B.WINO_FUSED_F2)
    torch.cuda.synchronize()
    pu.check(y.float().cpu().numpy().astype(np.float64), ref, 5e-3, 2, "f16")
    assert torch.equal(y, y_again)


def test_stage_calls_that_need_a_stored_product_reject_the_fused_variant():
    U = torch.zeros(256 * 8 * 8, dtype=torch.float16, device=DEV)      # larger than any variant value could ask for
    with pytest.raises(B.WinoError) as e:
        B.wino_batched_gemm(U, U, 8, 8, 8, B.WINO_FUSED_F2)
    assert e.value.status == B.WINO_ERR_VARIANT
    with pytest.raises(B.WinoError) as e:
        B.wino_fused_gemm_output(U, U, None, 1, 8, 4, 4, 8, block_shape=7)
    assert e.value.status == B.WINO_ERR_VARIANT


# ---- WINO_FUSED_F4: the same for F(4x4,3x3), two-byte storage types ---------------------------------------------------
TOL4 = {"f16": 5e-3, "bf16": 4e-2}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("shape", SHAPES + [(1, 64, 96, 40, 44), (2, 128, 70, 9, 64)])
def test_f4_whole_path_small_shapes(shape, layout, dtype):
    N, C, K, H, W = shape
    x, w, b = synth.make_inputs(N, C, K, H, W, dtype, seed=7300 + sum(shape))
    ref = oracle.conv2d_direct(_np(x), _np(w), _np(b))
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    y = B.conv2d(xd, w.to(DEV), b.to(DEV), B.WINO_FUSED_F4, layout=layout)
    torch.cuda.synchronize()
    pu.check(_nchw(y, layout), ref, TOL4[dtype], 4, dtype, what=(shape, layout, dtype), channels=C)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("block_shape", [0, 1])
@pytest.mark.parametrize("shape", [(2, 5, 7, 5, 7), (1, 33, 65, 17, 30), (2, 136, 200, 16, 16), (1, 200, 150, 37, 41), (1, 72, 300, 21, 39),
                                   (1, 64, 200, 30, 36), (2, 128, 320, 16, 32), (1, 192, 130, 64, 64)])
def test_f4_every_block_shape(shape, block_shape, layout, dtype):
    """The stage call with a named block shape on inputs with ragged rows and columns, a ragged last reduction stage (C not a
    multiple of 64) and more than one block in both directions; against the oracle and against the unfused F(4x4) stages."""
    N, C, K, H, W = shape
    x, w, b = synth.make_inputs(N, C, K, H, W, dtype, seed=7400 + sum(shape))
    ref = oracle.conv2d_direct(_np(x), _np(w), _np(b))
    xd = (x.permute(0, 2, 3, 1).contiguous() if layout == B.WINO_NHWC else x).to(DEV)
    filt = B.wino_filter_transform(w.to(DEV), B.WINO_FUSED_F4)
    assert filt.desc.variant == B.WINO_FUSED_F4
    U = filt.buf.view(x.dtype)
    V = B.wino_input_transform(xd, B.WINO_FUSED_F4, layout=layout)
    y = B.wino_fused_gemm_output(U, V, b.to(DEV), N, C, H, W, K, layout=layout, block_shape=block_shape, m=4)
    torch.cuda.synchronize()
    pu.check(_nchw(y, layout), ref, TOL4[dtype], 4, dtype, what=(shape, block_shape, layout, dtype), channels=C)
    # the unfused F(4x4) path on the same U and V adds the same products in fp32 in another order
    y_chain = B.conv2d(xd, w.to(DEV), b.to(DEV), B.WINO_F4, layout=layout)
    torch.cuda.synchronize()
    d = (y.float() - y_chain.float()).abs().max().item()
    assert d <= (2.0 ** -9 if dtype == "f16" else 2.0 ** -6) * max(1.0, y.float().abs().max().item())


def test_f4_zero_input_no_bias_determinism_and_workspace():
    x, w, b = synth.make_inputs(2, 40, 24, 10, 11, "f16", seed=5)
    xd, wd, bd = x.to(DEV), w.to(DEV), b.to(DEV)
    y0 = B.conv2d(torch.zeros_like(xd), wd, bd, B.WINO_FUSED_F4)
    torch.cuda.synchronize()
    assert torch.equal(y0.float().cpu(), b.to(torch.float16).float().view(1, -1, 1, 1).expand(2, 24, 10, 11))
    ref = oracle.conv2d_direct(_np(x), _np(w), None)
    y = B.conv2d(xd, wd, None, B.WINO_FUSED_F4)
    y_again = B.conv2d(xd, wd, None, B.WINO_FUSED_F4)
    torch.cuda.synchronize()
    pu.check(y.float().cpu().numpy().astype(np.float64), ref, 5e-3, 4, "f16")
    assert torch.equal(y, y_again)
    assert B.wino_workspace_bytes(2, 40, 10, 11, 24, B.WINO_F16, B.WINO_FUSED_F4) < B.wino_workspace_bytes(2, 40, 10, 11, 24, B.WINO_F16, B.WINO_F4)


def test_f4_fused_is_for_two_byte_storage_only():
    assert B.wino_resolve_variant(1, 8, 8, 8, 8, B.WINO_F32, B.WINO_FUSED_F4) == -1
    assert B.wino_filter_bytes(8, 8, B.WINO_F32, B.WINO_FUSED_F4) == 0
    assert B.wino_workspace_bytes(1, 8, 8, 8, 8, B.WINO_F32, B.WINO_FUSED_F4) == 0
    w = torch.zeros(8, 8, 3, 3, device=DEV)
    with pytest.raises(B.WinoError) as e:
        B.wino_filter_transform(w, B.WINO_FUSED_F4)
    assert e.value.status == B.WINO_ERR_VARIANT          # raised by the binding: wino_filter_bytes is 0 for this pair
    U = torch.zeros(36 * 8 * 8, dtype=torch.float32, device=DEV)
    with pytest.raises(B.WinoError) as e:
        B.wino_fused_gemm_output(U, U, None, 1, 8, 4, 4, 8, m=4)
    assert e.value.status == B.WINO_ERR_DTYPE
    Uh = U.half()
    with pytest.raises(B.WinoError) as e:
        B.wino_fused_gemm_output(Uh, Uh, None, 1, 8, 4, 4, 8, block_shape=2, m=4)
    assert e.value.status == B.WINO_ERR_VARIANT


@pytest.mark.parametrize("layout", [B.WINO_NCHW, B.WINO_NHWC])
@pytest.mark.parametrize("C", [8, 40, 96, 120, 136, 352])
def test_f4_ragged_stage_multiplies_zeros_only(C, layout):
    """Cp off the stage: the chunks beyond Cp are zeros, not the start of the next row of V or U.  A NaN in one tile (its pixel lies in that
    tile's window only) and one in the filter of one output channel stay there; everything else keeps its bits.  One, two and
    several stages per position, odd and even."""
    N, K, H, W = 1, 72, 16, 24
    x, w, b = synth.make_inputs(N, C, K, H, W, "f16", seed=7300 + C)
    perm = (lambda t: t.permute(0, 2, 3, 1).contiguous()) if layout == B.WINO_NHWC else (lambda t: t)
    run = lambda a, f: _nchw(B.conv2d(perm(a).to(DEV), f.to(DEV), b.to(DEV), B.WINO_FUSED_F4, layout=layout), layout)
    clean = run(x, w)
    pu.check(clean, oracle.conv2d_direct(_np(x), _np(w), _np(b)), TOL["f16"], 4, "f16", what=(C, layout), channels=C)
    xn, wn = x.clone(), w.clone()
    xn[0, 0, 9, 10] = float("nan")               # tile (2, 2)
    wn[33, 0, 1, 1] = float("nan")
    y = run(xn, w)
    hit = np.zeros((H, W), bool); hit[8:12, 8:12] = True
    assert np.isnan(y[:, :, hit]).all() and np.array_equal(y[:, :, ~hit], clean[:, :, ~hit])
    y = run(x, wn)
    rest = np.arange(K) != 33
    assert np.isnan(y[:, 33]).all() and np.array_equal(y[:, rest], clean[:, rest])

"""Which kernel the library takes, at sizes where both candidates were measured (times in the sources, beside the rules)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import routes  # noqa: E402


# direct path, two-byte types and whole stages: the block, channel-last and NCHW alike, at sizes where the blocks were timed against each other
@pytest.mark.parametrize("N,C,K,H,W,R,st,block", [
    (1, 128, 512, 256, 256, 1, 1, 4), (1, 256, 512, 512, 512, 3, 2, 4), (1, 256, 512, 240, 240, 3, 1, 4), (1, 256, 256, 512, 512, 3, 1, 4), (1, 256, 240, 512, 512, 3, 1, 4),
    (1, 512, 512, 256, 256, 3, 1, 4), (1, 128, 128, 1024, 1024, 3, 1, 4), (2, 128, 400, 129, 127, 3, 1, 4), (1, 512, 512, 128, 128, 3, 1, 4), (1, 64, 512, 180, 180, 3, 1, 4),
    (1, 256, 264, 512, 512, 1, 1, 2), (1, 512, 512, 99, 101, 3, 1, 2), (2, 256, 560, 144, 51, 1, 1, 2), (2, 640, 640, 64, 64, 3, 1, 2), (2, 1280, 640, 64, 64, 1, 1, 2),
    (2, 320, 320, 64, 64, 3, 1, 3), (2, 320, 320, 64, 64, 1, 1, 3), (2, 960, 320, 64, 64, 1, 1, 3),
    (2, 1856, 1184, 23, 57, 1, 1, 1), (1, 64, 256, 251, 250, 3, 2, 1), (2, 320, 320, 97, 121, 3, 1, 1), (2, 320, 320, 97, 121, 1, 1, 1), (8, 128, 128, 76, 212, 1, 2, 1),
    (2, 320, 320, 64, 64, 3, 2, 0), (1, 384, 48, 315, 249, 3, 1, 0), (1, 512, 64, 330, 354, 3, 1, 0), (1, 128, 384, 7, 215, 1, 1, 0), (1, 64, 16, 5, 5, 1, 1, 5), (1, 128, 24, 130, 127, 3, 1, 5)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_direct_path_blocks(N, C, K, H, W, R, st, block, dtype):
    for nhwc in (False, True):
        assert routes.block_plan(N, C, K, H, W, R, st, dtype, nhwc) == (block, 1)
        assert routes.block_plan(N, C, K, H, W, R, st, "f32", nhwc)[0] < 0 and routes.block_plan(N, C - 8, K, H, W, R, st, dtype, nhwc)[0] < (0 if C % 64 == 0 else 6)


# few pixels and a long reduction: ranges, never more than the workspace of either layout holds
@pytest.mark.parametrize("N,C,K,H,W,R,st,ranges", [(2, 640, 640, 32, 32, 3, 2, 3), (2, 1280, 1280, 16, 16, 3, 2, 6), (1, 1280, 72, 9, 6, 3, 2, 15), (2, 128, 128, 17, 13, 3, 1, 2), (2, 64, 128, 17, 13, 3, 1, 1)])
def test_direct_path_workspace_ranges(N, C, K, H, W, R, st, ranges):
    for dtype in ("f16", "bf16"):
        assert max(routes.igemm_split(N, C, K, H, W, R, st, dtype, nhwc) for nhwc in (False, True)) == ranges
        assert all(1 <= routes.block_plan(N, C, K, H, W, R, st, dtype, nhwc)[1] <= ranges for nhwc in (False, True))


# the blocks of conv_igemm.hip: what does not come in whole stages, and what is left to them
@pytest.mark.parametrize("N,C,K,H,W,R,st,shape", [(1, 24, 256, 256, 256, 3, 1, (256, 256)), (1, 24, 128, 256, 256, 3, 1, (256, 128)), (1, 24, 72, 256, 256, 3, 1, (128, 128)), (1, 24, 72, 64, 64, 3, 1, (64, 64)),
                                                 (1, 512, 512, 512, 512, 1, 1, (256, 256))])
def test_direct_path_blocks_of_the_other_kernel(N, C, K, H, W, R, st, shape):
    assert routes.igemm_shape(N * H * W, K) == shape
    assert all(routes.block_plan(N, C, K, H, W, R, st, dtype, nhwc)[0] < 0 for dtype in ("f16", "bf16") for nhwc in (False, True))


# Times by which the direct path's blocks are compared: times, so positive, and longer for more pixels, more channels and more stages; a block of which
# half the columns are empty is not credited for them.
@pytest.mark.parametrize("nhwc", [False, True])
@pytest.mark.parametrize("C,R", [(64, 1), (128, 1), (192, 1), (640, 1), (64, 3), (512, 3)])
@pytest.mark.parametrize("K", [16, 40, 64, 130, 192, 512, 999])
def test_block_times_are_times(K, C, R, nhwc):
    pixels = [64, 1000, 5000, 2 ** 14, 40000, 2 ** 16, 2 ** 18, 2 ** 20, 2 ** 24]
    for block in range(len(routes.BLOCKS)):
        t = [routes.block_time(block, T, T, K, C, R, nhwc) for T in pixels]
        assert t[0] > 0 and all(a <= b for a, b in zip(t, t[1:])), (block, t)
        assert t[-1] > 40 * t[5] and routes.block_time(block, 2 ** 18, 2 ** 18, 3 * K, C, R, nhwc) >= t[6]
        assert routes.block_time(block, 2 ** 18, 2 ** 18, K, C + 64, R, nhwc) > t[6]
        assert all(routes.block_time(block, 256, 256, K, C, R, nhwc, ranges) > 0 for ranges in (2, 16))


# ... and the block itself, 1x1 on large images: none with half of its columns empty, and 96 columns where they fit
@pytest.mark.parametrize("H,W", [(512, 512), (1024, 1024), (999, 1014), (400, 453)])
@pytest.mark.parametrize("C", [64, 128, 192])
@pytest.mark.parametrize("K", [33, 40, 48, 56, 64])
def test_direct_path_blocks_of_few_columns(K, C, H, W):
    for nhwc in (False, True):
        block, ranges = routes.block_plan(1, C, K, H, W, 1, 1, "f16", nhwc)
        assert routes.BLOCKS[block][1] == 64 and ranges == 1, (block, nhwc)


def test_direct_path_blocks_that_fit():
    assert all(routes.block_plan(1, C, 192, 512, 512, 1, 1, "f16", nhwc)[0] == 2 for C in (64, 128) for nhwc in (False, True))
    assert routes.block_plan(2, 64, 160, 568, 625, 1, 1, "f16", True)[0] == 2 and routes.block_plan(1, 832, 68, 311, 185, 3, 2, "f16", True) == (6, 1)
    # elements of a channel-last y, and full rounds of 256x256 blocks in long 1x1 reductions or on NCHW images of an odd number of pixels: conv_igemm.hip; without, here
    for N, C, K, H, W, nhwc, here in [(1, 64, 243, 544, 392, True, False), (4, 128, 1379, 22, 24, True, False), (1, 256, 118, 187, 154, True, False), (1, 64, 130, 159, 192, True, True),
                                      (1, 64, 126, 69, 77, True, True), (1, 64, 244, 544, 392, True, True), (1, 640, 512, 415, 473, False, False), (1, 64, 256, 829, 778, False, False),
                                      (1, 384, 768, 157, 189, False, True), (1, 640, 512, 233, 302, False, True), (1, 384, 512, 416, 473, False, True), (1, 512, 512, 512, 512, True, False), (1, 512, 512, 512, 512, False, False),
                                      (1, 512, 512, 256, 256, False, True), (1, 512, 1024, 256, 256, True, False), (1, 384, 256, 512, 512, True, True), (1, 640, 768, 128, 752, True, True), (1, 512, 516, 512, 512, True, True)]:
        assert (routes.block_plan(N, C, K, H, W, 1, 1, "bf16", nhwc)[0] >= 0) == here, (C, K)


# Buffer offsets of the direct kernels: what a lane reads, and the scalar that is added for all lanes, also to the offset 2^31 of a lane that
# must read zeros, have to stay within the descriptor's 2^31 - 1 bytes.  The widest admitted image of each form, a single row among them.
@pytest.mark.parametrize("C,e,fits,N,H,up,R", [(C, 2, "tile", *form) for C in (64, 192, 1280) for form in ((1, 1, 0, 3), (1, 2, 0, 3), (2, 1, 0, 3), (3, 5, 0, 3), (1, 2, 1, 3), (1, 1, 0, 1))] +
                         [(C, 1, "rows", *form) for C in (64, 160) for form in ((1, 1, 0, 3), (1, 2, 0, 3), (2, 1, 0, 3), (3, 5, 0, 3))])
def test_buffer_offsets_stay_in_range(C, e, fits, N, H, up, R):
    ok = (lambda W: routes.tile_fits(N, C, 8, H, W, R=R, up=up)) if fits == "tile" else (lambda W: routes.fp8_rows(N, C, 8, H, W, "f16", True)[0])
    lo, hi = 2 ** 15, 2 ** 31 // (N * H)                # admitted, refused; widths that can be read upsampled are even
    assert ok(lo)
    while hi - lo > 2:
        mid = (lo + hi) // 4 * 2
        lo, hi = (mid, hi) if ok(mid) else (lo, mid)
    for W in (lo, lo + 1):
        if not ok(W) or (up and W % 2):
            continue
        row, stored = C * e, W >> up
        lanes = (N * (H >> up) * stored + stored + 1) * row
        scalar = (0 if up or R == 1 else 2 * stored + 2) * row + row - 128 * (e == 2)
        if fits == "rows":                              # a block of up to 256 pixels and its neighbours beyond the last one
            lanes, scalar = lanes + 258 * row, scalar + 256 * row
        assert lanes <= 2 ** 31 - 1 and scalar <= 2 ** 31 - 1, (W, lanes, scalar)
    assert lo * N * H * C * e > 2 ** 29                  # and no more is given away than a single row needs


# one-kernel F(2x2): taken (True) or left to the paths that store V
@pytest.mark.parametrize("N,C,K,H,W,nhwc,fused,norm,up,taken", [
    # element by element: rows of no whole 16-byte pieces, and upsampling
    (2, 320, 320, 52, 78, False, False, True, False, False), (1, 256, 256, 250, 250, False, True, True, False, False), (1, 256, 256, 250, 250, False, False, True, False, False),
    (1, 128, 256, 200, 204, False, True, False, False, False), (1, 128, 256, 200, 204, False, True, False, True, False), (1, 192, 96, 500, 300, False, True, False, False, True),
    (1, 64, 128, 250, 250, False, True, False, False, False),
    (1, 128, 128, 300, 300, False, True, True, False, False), (1, 64, 320, 140, 142, False, True, True, False, False),
    (1, 64, 128, 250, 250, False, False, True, False, True), (1, 128, 128, 300, 300, False, False, False, True, True), (1, 192, 96, 500, 300, False, False, True, False, True),
    # whole pieces, channel-last
    (2, 640, 640, 64, 64, False, False, True, False, False), (1, 512, 512, 128, 128, False, False, True, False, False), (1, 512, 512, 256, 256, False, False, True, False, False),
    (1, 256, 256, 256, 256, False, True, True, False, False), (2, 320, 320, 64, 64, False, False, True, False, True), (2, 320, 320, 128, 128, False, True, True, False, True),
    (1, 256, 256, 256, 256, True, False, True, False, True), (2, 320, 320, 64, 64, True, True, True, False, True), (1, 512, 256, 128, 128, True, True, True, False, True),
    (4, 320, 320, 64, 96, True, True, True, False, True), (1, 512, 512, 128, 128, False, True, False, False, False), (2, 192, 192, 104, 152, False, False, True, False, True), (2, 1280, 1280, 32, 32, True, False, False, False, False),
    # large images
    (1, 256, 256, 512, 512, True, True, False, False, True), (1, 256, 256, 512, 512, True, True, True, False, True), (1, 512, 256, 256, 256, True, True, False, False, True),
    (1, 128, 352, 495, 744, True, True, False, False, True), (1, 640, 320, 256, 256, False, False, False, False, True), (1, 384, 384, 384, 384, False, False, False, False, True),
    (1, 256, 256, 512, 512, False, True, False, False, False), (1, 512, 512, 256, 256, False, True, False, False, False), (1, 512, 512, 256, 256, True, True, True, False, False), (1, 256, 512, 512, 512, False, True, True, False, False)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_one_kernel_f2(N, C, K, H, W, nhwc, fused, norm, up, taken, dtype):
    assert (routes.onepass(N, C, K, H, W, dtype, nhwc, fused, norm, up)[0] > 0) == taken


def test_one_kernel_f2_residual_and_bounds():
    for bad in (dict(C=120), dict(K=136), dict(dtype="f32")):
        assert routes.onepass(**{**dict(N=1, C=128, K=128, H=512, W=512, dtype="bf16", nhwc=True), **bad})[0] == 0
    assert routes.onepass(1, 192, 320, 128, 312, "bf16", True, True, True, residual=True)[0] > 0 and routes.onepass(1, 192, 320, 128, 312, "bf16", True, True, True)[0] == 0
    assert routes.onepass(1, 128, 128, 512, 512, "bf16", False)[1] == 1
    assert routes.onepass(1, 128, 128, 512, 512, "bf16", False, address=routes.ADDRESS + 2)[1] == 2


# 8-bit direct path, unsplit reductions: the pipelined kernel from one 128x128 block to a compute unit on, and in NCHW for short reductions
@pytest.mark.parametrize("N,C,K,H,W,R,st,nhwc,taken", [
    (1, 64, 128, 32, 32, 1, 1, True, False), (1, 256, 256, 64, 64, 3, 1, True, False), (1, 640, 640, 64, 64, 3, 1, True, False), (1, 128, 128, 57, 175, 3, 2, True, False),
    (1, 256, 256, 128, 128, 3, 1, True, True), (1, 64, 512, 96, 96, 1, 1, True, True), (1, 128, 128, 1024, 1024, 3, 1, True, True), (1, 256, 256, 512, 512, 3, 1, True, False),
    (1, 256, 256, 64, 64, 3, 1, False, False), (1, 1280, 320, 64, 64, 3, 1, False, False), (1, 640, 128, 180, 180, 3, 1, False, True), (1, 256, 256, 96, 96, 3, 1, False, True), (1, 256, 64, 180, 180, 3, 1, False, False), (1, 640, 640, 64, 64, 3, 1, False, True), (1, 64, 256, 64, 64, 3, 1, False, True),
    (1, 1280, 128, 64, 64, 1, 1, False, True), (1, 320, 320, 64, 64, 3, 1, False, True), (1, 64, 512, 60, 49, 1, 2, False, False), (1, 64, 512, 60, 50, 1, 2, False, False), (1, 128, 1024, 15, 12, 1, 1, False, False), (1, 128, 1024, 16, 12, 1, 1, False, True),
    # few output channels
    (1, 64, 8, 76, 16, 1, 1, True, True), (1, 16, 1, 54, 6, 1, 1, True, True), (1, 48, 20, 61, 344, 1, 1, True, True), (1, 320, 22, 141, 120, 1, 2, True, False), (1, 112, 64, 48, 157, 1, 1, True, False),
    (8, 64, 16, 118, 131, 3, 1, False, True), (4, 256, 16, 103, 128, 3, 1, False, True), (1, 128, 8, 91, 152, 3, 2, False, False), (1, 192, 8, 58, 71, 1, 1, False, False),
    (1, 256, 256, 128, 128, 3, 1, False, True), (1, 256, 256, 512, 512, 3, 1, False, True)])
def test_fp8_kernel(N, C, K, H, W, R, st, nhwc, taken):
    for dtype in ("f16", "bf16"):
        assert routes.fp8_tile(N, C, K, H, W, R, st, dtype, nhwc) == taken
    assert not routes.fp8_tile(N, C, K, H, W, R, st, "f32", nhwc) and not routes.fp8_tile(N, C, K, H, W, R, st, "f16", nhwc, nsplit=2)


# ... 3x3 at stride 1: the kernel that fetches the pixels of a filter row once, with 128x128 ("rows") or 256x256 blocks ("wide"), or the others ("")
@pytest.mark.parametrize("N,C,K,H,W,nhwc,kernel", [
    (1, 128, 128, 512, 512, False, "rows"), (1, 128, 128, 512, 512, True, "rows"), (1, 512, 320, 120, 72, True, "rows"), (2, 62, 192, 58, 106, True, ""), (1, 72, 256, 84, 160, True, "rows"), (2, 555, 126, 155, 58, False, ""),
    # outputs one by one: channels of a channel-last y, an odd number of pixels
    (1, 256, 58, 253, 104, True, ""), (1, 47, 150, 76, 205, True, ""), (1, 192, 222, 220, 60, True, ""), (1, 192, 93, 300, 128, True, "rows"), (1, 75, 23, 300, 104, True, "rows"),
    (1, 62, 64, 299, 87, False, ""), (1, 62, 64, 299, 115, False, "rows"), (2, 62, 64, 149, 87, False, ""), (1, 273, 253, 71, 181, False, "rows"),
    # full rounds of 256x256 blocks
    (1, 512, 512, 256, 256, False, ""), (1, 512, 512, 192, 320, False, ""), (1, 1024, 512, 256, 256, False, ""), (1, 768, 512, 141, 232, False, ""), (1, 640, 768, 156, 224, False, ""),
    (1, 512, 256, 512, 512, False, "wide"), (1, 640, 256, 286, 352, False, "rows"), (1, 256, 256, 512, 512, False, "wide"), (1, 448, 768, 566, 72, False, "wide"), (1, 704, 512, 349, 144, False, "wide"),
    (1, 512, 512, 128, 128, False, "rows"), (1, 512, 512, 320, 320, False, "rows"), (1, 448, 256, 512, 400, False, "rows"), (1, 448, 192, 224, 576, False, "wide"), (1, 512, 512, 257, 255, False, "rows"),
    (1, 256, 256, 256, 256, True, ""), (1, 512, 512, 256, 256, True, ""), (1, 512, 512, 192, 320, True, ""), (1, 512, 512, 384, 256, True, "rows"), (1, 256, 256, 512, 512, True, "rows"), (1, 320, 512, 256, 256, True, "rows"), (1, 640, 256, 512, 256, True, "rows"), (1, 448, 256, 224, 520, False, "wide")])
def test_fp8_rows_kernel(N, C, K, H, W, nhwc, kernel):
    for dtype in ("f16", "bf16"):
        taken, wide = routes.fp8_rows(N, C, K, H, W, dtype, nhwc)
        assert ("wide" if wide else "rows" if taken else "") == kernel
        assert not routes.fp8_rows(N, C, K, H, W, dtype, nhwc, nsplit=2)[0] and not routes.fp8_rows(N, C, K, H, W, dtype, nhwc, st=2)[0]
    assert not routes.fp8_rows(N, C, K, H, W, "f32", nhwc)[0]


# few input channels, fp32 F(4x4): with more than eight channels only from some number of tiles times output channels on
@pytest.mark.parametrize("N,C,K,H,W,nhwc,up,taken", [
    (1, 4, 8, 16, 16, False, False, True), (1, 8, 4, 5, 7, True, True, True), (1, 8, 3, 5, 7, False, True, True), (1, 4, 5, 96, 96, True, False, False), (2, 4, 5, 128, 128, True, False, True), (1, 9, 320, 16, 16, False, False, False), (1, 16, 8, 64, 64, True, False, False),
    (1, 16, 320, 64, 64, False, False, True), (1, 9, 64, 96, 96, True, False, True), (2, 9, 8, 96, 96, False, False, True), (1, 9, 8, 128, 125, False, False, False), (1, 16, 64, 78, 43, False, False, False), (1, 9, 320, 78, 43, False, False, True),
    (1, 16, 64, 78, 43, True, False, False), (1, 16, 64, 64, 64, False, True, False), (2, 16, 320, 64, 64, False, True, True), (1, 17, 320, 64, 64, False, False, False)])
def test_few_channels(N, C, K, H, W, nhwc, up, taken):
    assert routes.fewc(N, C, K, H, W, "f32", nhwc, up=up) == taken
    assert not routes.fewc(N, C, K, H, W, "f32", nhwc, norm=True, up=up) and not routes.fewc(N, C, K, H, W, "f16", nhwc, up=up)

"""Asks libwino which kernel it takes for a call: the rules themselves (C++ functions of the library, by their mangled names), without a GPU.

Tests use it to state which kernel they run, so that a change of a constant in a rule cannot quietly send them elsewhere."""
import ctypes

from paper_2412_05781_amd import binding as B

ADDRESS = 0x10000                  # stands for a 16-byte aligned tensor; the rules look at the alignment only


class Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in "N C H W K m alpha th tw T Cp".split()]


class ConvGeom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in "N C Cp H W K R st pad Ho Wo T up Hs Ws".split()]


class PreOp(ctypes.Structure):
    _fields_ = [("stats", ctypes.c_void_p), ("gamma", ctypes.c_void_p), ("beta", ctypes.c_void_p), ("groups", ctypes.c_int), ("cpg", ctypes.c_int),
                ("up", ctypes.c_int)]


class Pair(ctypes.Structure):
    _fields_ = [("a", ctypes.c_int), ("b", ctypes.c_int)]


DT = {"f32": B.WINO_F32, "f16": B.WINO_F16, "bf16": B.WINO_BF16}
INT, BOOL, PTR = ctypes.c_int, ctypes.c_bool, ctypes.c_void_p


def _fn(name, restype, *argtypes):
    f = getattr(B.lib(), name)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def _out(n, R, st):
    return (n + 2 * ((R - 1) // 2) - R) // st + 1


def winograd_geom(N, C, K, H, W, m):
    th, tw = -(-H // m), -(-W // m)
    return Geom(N, C, H, W, K, m, m + 2, th, tw, N * th * tw, -(-C // 8) * 8)


def pre_op(norm=False, up=False, C=1):
    return PreOp(ADDRESS if norm else None, ADDRESS, ADDRESS, 1, C, int(up))


def conv_geom(N, C, K, H, W, R=3, st=1, up=0, align=8):
    Ho, Wo = _out(H, R, st), _out(W, R, st)
    return ConvGeom(N, C, -(-C // align) * align, H, W, K, R, st, (R - 1) // 2, Ho, Wo, N * Ho * Wo, up, H >> up, W >> up)


def tile_fits(*geom, **kw):
    """Whether the operands of a two-byte direct call lie within the 16x16-tile kernel's offsets."""
    f = _fn("_ZN4wino15igemm_tile_fitsERKNS_8ConvGeomE", BOOL, ctypes.POINTER(ConvGeom))
    return f(ctypes.byref(conv_geom(*geom, **kw)))


def igemm_split(N, C, K, H, W, R, st, dtype, nhwc):
    """Reduction ranges that the workspace of a direct call is sized for, in this layout."""
    f = _fn("_ZN4wino11igemm_splitEiiiiiib", INT, INT, INT, INT, INT, INT, INT, BOOL)
    pixels = _out(H, R, st) * _out(W, R, st)
    return f(N * pixels, pixels, K, -(-C // 8) * 8, R, DT[dtype], nhwc)


def block_plan(N, C, K, H, W, R, st, dtype, nhwc):
    """(block, reduction ranges) of a direct call on the 16x16-tile kernel: 0 = 64x64, 1 = 128x64, 2 and 3 = 128x96 with two and three slots, 4 = 128x128,
    5 = 64x32, 6 = 64x80 (pixels x output channels); block < 0: the kernels of conv_igemm.hip."""
    f = _fn("_ZN4wino16igemm_block_planEiiiiiibi", Pair, INT, INT, INT, INT, INT, INT, BOOL, INT)
    pixels = _out(H, R, st) * _out(W, R, st)
    most = max(igemm_split(N, C, K, H, W, R, st, dtype, layout) for layout in (False, True))
    p = f(N * pixels, pixels, K, -(-C // 8) * 8, R, DT[dtype], nhwc, most)
    return p.a, p.b


BLOCKS = [(64, 64), (128, 64), (128, 96), (128, 96), (128, 128), (64, 32), (64, 80)]


def block_time(block, pixels, pixels_per_image, K, C, R, nhwc, ranges=1):
    """Time in us by which block_plan compares its choices."""
    f = _fn("_ZN4wino16igemm_block_timeEiiiiiibi", ctypes.c_double, INT, INT, INT, INT, INT, INT, BOOL, INT)
    return f(block, pixels, pixels_per_image, K, C, R, nhwc, ranges)


def fp8_rows(N, C, K, H, W, dtype, nhwc, nsplit=1, **kw):
    """Whether the 8-bit kernel that fetches the pixels of a filter row once takes a call, and whether its NCHW blocks are 256x256 (128x128 otherwise)."""
    g = conv_geom(N, C, K, H, W, align=16, **kw)
    f = _fn("_ZN4wino17igemm_fp8_rows_okERKNS_8ConvGeomEibi", BOOL, ctypes.POINTER(ConvGeom), INT, BOOL, INT)
    wide = _fn("_ZN4wino19igemm_fp8_rows_wideERKNS_8ConvGeomE", BOOL, ctypes.POINTER(ConvGeom))
    taken = f(ctypes.byref(g), DT[dtype], nhwc, nsplit)
    return taken, taken and not nhwc and H * W % 2 == 0 and wide(ctypes.byref(g))


def igemm_shape(pixels, K):
    """Block (pixels, output channels) of conv_igemm.hip."""
    p = _fn("_ZN4wino11igemm_shapeEii", Pair, INT, INT)(pixels, K)
    return p.a, p.b


def onepass(N, C, K, H, W, dtype, nhwc, fused_variant=False, norm=False, up=False, residual=False, address=ADDRESS):
    """(16-channel sub-tiles per wave, 0 channel-last / 1 rows of whole 16-byte pieces / 2 element by element) of the one-kernel F(2x2) path;
    0 sub-tiles: the paths that store V."""
    f = _fn("_ZN4wino12onepass_planEPKvRKNS_4GeomEibbPKNS_5PreOpEb", Pair, PTR, ctypes.POINTER(Geom), INT, BOOL, BOOL, ctypes.POINTER(PreOp), BOOL)
    p = f(address, ctypes.byref(winograd_geom(N, C, K, H, W, 2)), DT[dtype], nhwc, fused_variant, ctypes.byref(pre_op(norm, up, C)), residual)
    return p.a, p.b


def fp8_tile(N, C, K, H, W, R, st, dtype, nhwc, nsplit=1):
    """Whether the pipelined kernel takes an 8-bit direct call with an unsplit reduction."""
    f = _fn("_ZN4wino17igemm_fp8_tile_okERKNS_8ConvGeomEibi", BOOL, ctypes.POINTER(ConvGeom), INT, BOOL, INT)
    Ho, Wo = _out(H, R, st), _out(W, R, st)
    g = ConvGeom(N, C, -(-C // 16) * 16, H, W, K, R, st, (R - 1) // 2, Ho, Wo, N * Ho * Wo, 0, H, W)
    return f(ctypes.byref(g), DT[dtype], nhwc, nsplit)


def fewc(N, C, K, H, W, dtype, nhwc, norm=False, up=False):
    """Whether the one-kernel fp32 F(4x4) path for few input channels takes a call."""
    f = _fn("_ZN4wino12fewc_conv_okERKNS_4GeomEibPKNS_5PreOpE", BOOL, ctypes.POINTER(Geom), INT, BOOL, ctypes.POINTER(PreOp))
    return f(ctypes.byref(winograd_geom(N, C, K, H, W, 4)), DT[dtype], nhwc, ctypes.byref(pre_op(norm, up, C)))

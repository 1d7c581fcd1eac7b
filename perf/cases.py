"""Cases that performance work on this library is measured on: the convolutions of a Stable-Diffusion image, as a program calls them.

Every case is one convolution of a UNet or a VAE decoder through the public calls of ``paper_2412_05781_amd.binding``, with
the variant that ``wino_recommend_variant`` names, the filter prepared once and the workspace kept, as an inference program
does.  ``op`` says which call: "conv" = wino_conv2d_ex, "fused" = wino_conv2d_fused (after wino_groupnorm_stats when the
GroupNorm is fused in), "igemm" = wino_igemm_conv2d (1x1 and stride 2), "fp8" = wino_fp8_conv2d.  H and W are those of the
tensor the convolution sees (after upsampling, before striding).
"""
import math

import torch

from paper_2412_05781_amd import binding as B

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
GROUPS = 32                     # GroupNorm groups of the UNet and the VAE


def _case(name, op, N, C, K, H, W, dtype="f16", layout="nchw", R=3, stride=1, norm=False, vector=False, residual=False, upsample=False):
    case = dict(op=op, N=N, C=C, K=K, H=H, W=W, dtype=dtype, layout=layout, R=R, stride=stride, norm=norm, vector=vector,
                residual=residual, upsample=upsample)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # first convolution of the UNet on one latent, fp32 storage: a small call, latency and launches
        _case("conv_in_f32", "conv", 1, 4, 320, 64, 64, "f32"),
        # first half of a residual block at full latent size (512x512 image, guidance batch): GroupNorm + SiLU, convolution, time embedding
        _case("resblock_64", "fused", 2, 320, 320, 64, 64, norm=True, vector=True),
        # second half of a deep residual block, channel-last: GroupNorm + SiLU, convolution, skip connection
        _case("resblock_16_nhwc", "fused", 2, 1280, 1280, 16, 16, layout="nhwc", norm=True, residual=True),
        # first up-path convolution on 8x8: few pixels, a stream of weights
        _case("concat_8", "conv", 2, 2560, 1280, 8, 8),
        # up-path convolution on the concatenated skip tensor, channel-last
        _case("concat_32_nhwc", "conv", 2, 1920, 640, 32, 32, layout="nhwc"),
        # up-sampling convolution of a 416x624 image: latent sides that are no multiple of a tile or of a 16-byte chunk
        _case("upsample_ragged", "fused", 2, 640, 640, 52, 78, upsample=True),
        # second half of an SDXL residual block (1024x1024 image) with bfloat16 storage
        _case("resblock_128_bf16", "fused", 2, 320, 320, 128, 128, "bf16", norm=True, residual=True),
        # down-sampling convolution between two UNet levels: stride 2
        _case("downsample_64", "igemm", 2, 320, 320, 64, 64, stride=2),
        # 1x1 shortcut of a residual block that changes the number of channels, channel-last
        _case("shortcut_64_nhwc", "igemm", 2, 960, 320, 64, 64, layout="nhwc", R=1),
        # VAE decoder, middle of the up path: GroupNorm + SiLU, convolution, skip connection on a quarter-size image
        _case("vae_512_256", "fused", 1, 512, 512, 256, 256, norm=True, residual=True),
        # the VAE decoder's largest tensor, 128 channels at full image size, channel-last
        _case("vae_128_1024_nhwc", "conv", 1, 128, 128, 1024, 1024, layout="nhwc"),
        # the VAE decoder with 8-bit operands, for programs that accept three mantissa bits
        _case("vae_256_512_fp8", "fp8", 1, 256, 256, 512, 512),
    ]


MAX_FLOPS = 2.0 * 9 * 512 * 512 * 256 * 256      # direct multiply-adds of the largest listed convolutions
MAX_PIXELS = 128.0 * 1024 * 1024                 # ... and elements of the largest listed tensor


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _fits(c):
    return (2.0 * c["N"] * c["R"] ** 2 * c["C"] * c["K"] * c["H"] * c["W"] <= MAX_FLOPS
            and c["N"] * max(c["C"], c["K"]) * c["H"] * c["W"] <= MAX_PIXELS)


def _draw_once(rng):
    kind = rng.choice(["conv_in", "unet", "unet", "unet", "upsample", "down", "shortcut", "vae", "vae", "fp8"])
    layout = rng.choice(["nchw", "nhwc"])
    if kind == "conv_in":
        return _case(None, "conv", rng.choice([1, 2]), rng.choice([4, 8, 9]), 32 * rng.randint(8, 12), rng.randint(40, 128), rng.randint(40, 128),
                     "f32", layout)
    if kind == "unet":
        H = int(_log(rng, 8, 128)); W = max(8, min(160, int(H * _log(rng, 0.6, 1.7))))
        C, K = 32 * int(_log(rng, 10, 80)), 32 * int(_log(rng, 10, 40))
        fused = rng.random() < 0.6
        return _case(None, "fused" if fused else "conv", rng.choice([1, 2, 2, 4]), C, K, H, W, rng.choice(["f16", "f16", "f16", "bf16"]), layout,
                     norm=fused, vector=fused and rng.random() < 0.5, residual=fused and rng.random() < 0.5)
    if kind == "upsample":
        return _case(None, "fused", rng.choice([1, 2]), 64 * rng.randint(5, 20), 64 * rng.randint(5, 20), 2 * int(_log(rng, 8, 64)),
                     2 * int(_log(rng, 8, 64)), "f16", layout, upsample=True)
    if kind == "down":
        C = 64 * rng.randint(5, 20)
        return _case(None, "igemm", rng.choice([1, 2, 2]), C, C, int(_log(rng, 16, 128)), int(_log(rng, 16, 128)), "f16", layout, stride=2)
    if kind == "shortcut":
        return _case(None, "igemm", 2, 32 * int(_log(rng, 10, 80)), 32 * int(_log(rng, 10, 40)), int(_log(rng, 8, 96)), int(_log(rng, 8, 96)),
                     "f16", layout, R=1)
    H, W = 8 * int(_log(rng, 16, 128)), 8 * int(_log(rng, 16, 128))
    if kind == "vae":
        C, K = 64 * int(_log(rng, 2, 8.99)), 64 * int(_log(rng, 2, 8.99))
        fused = rng.random() < 0.6
        return _case(None, "fused" if fused else "conv", 1, C, K, H, W, rng.choice(["f16", "f16", "bf16"]), layout, norm=fused, residual=fused)
    return _case(None, "fp8", 1, 64 * int(_log(rng, 2, 8.99)), 64 * int(_log(rng, 2, 8.99)), H, W, "f16", layout)


def draw(rng):
    while True:
        case = _draw_once(rng)
        if _fits(case):
            return case


def _out_dims(c):
    pad = (c["R"] - 1) // 2
    return (c["H"] + 2 * pad - c["R"]) // c["stride"] + 1, (c["W"] + 2 * pad - c["R"]) // c["stride"] + 1


def _winograd_tile(c):
    """Output tile edge of the Winograd algorithm for the call: 4 where the storage type's error bound allows F(4x4) and the image
    has enough tiles for it, else 2; 0 for the calls that are direct convolutions by definition."""
    if c["op"] in ("igemm", "fp8"):
        return 0
    tiles = c["N"] * (-(-c["H"] // 4)) * (-(-c["W"] // 4))
    return 2 if c["dtype"] == "bf16" or (c["dtype"] == "f32" and c["C"] > 640) or tiles < 64 else 4


def prepare(case, seed):
    c = case
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    td = TORCH[c["dtype"]]
    layout = B.WINO_NHWC if c["layout"] == "nhwc" else B.WINO_NCHW
    N, C, K, H, W, R = c["N"], c["C"], c["K"], c["H"], c["W"], c["R"]
    up = 2 if c["upsample"] else 1
    Ho, Wo = _out_dims(c)

    def randn(shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, device=dev, generator=g, dtype=torch.float32) * std).to(dtype)

    s = {"case": c, "layout": layout}
    shape = lambda ch, h, w: (N, h, w, ch) if layout == B.WINO_NHWC else (N, ch, h, w)
    s["x"] = randn(shape(C, H // up, W // up), dtype=td)
    w = randn((K, C, R, R), 1.0 / math.sqrt(R * R * C), td)
    s["bias"] = randn((K,), 0.01)
    s["y"] = torch.empty(shape(K, Ho, Wo), dtype=td, device=dev)
    if c["norm"]:
        s["gamma"], s["beta"] = 1.0 + randn((C,), 0.1), randn((C,), 0.1)
        s["stats"] = torch.empty(B.wino_groupnorm_stats_bytes(N, GROUPS), dtype=torch.uint8, device=dev)
    s["vector"] = randn((N, K)) if c["vector"] else None
    s["residual"] = randn(shape(K, Ho, Wo), dtype=td) if c["residual"] else None
    if c["op"] == "igemm":
        s["filter"] = B.wino_igemm_filter_repack(w)
        ws = B.wino_igemm_workspace_bytes(N, C, H, W, K, R, c["stride"], B.DTYPE_OF[td], layout)
    elif c["op"] == "fp8":
        # largest powers of two that keep the scaled magnitudes within the format's 448
        s["scale_x"], s["scale_w"] = 64.0, 2.0 ** math.floor(math.log2(448.0 * math.sqrt(R * R * C) / 6.0))
        s["filter"] = B.wino_fp8_filter_quantize(w, s["scale_w"])
        ws = B.wino_fp8_workspace_bytes(N, C, H, W, K, R, c["stride"])
    else:
        v = B.wino_recommend_variant(N, C, H, W, K, B.DTYPE_OF[td])
        s["filter"] = B.wino_filter_transform(w, v)
        ws = B.wino_workspace_bytes(N, C, H, W, K, B.DTYPE_OF[td], v)
    s["workspace"] = torch.empty(max(16, ws), dtype=torch.uint8, device=dev)
    return s


def run(state):
    s, c = state, state["case"]
    if c["op"] == "conv":
        return B.wino_conv2d_ex(s["x"], s["filter"], s["bias"], s["y"], s["workspace"], s["layout"])
    if c["op"] == "igemm":
        return B.wino_igemm_conv2d(s["x"], s["filter"], s["bias"], s["y"], c["K"], c["R"], c["stride"], s["workspace"], s["layout"])
    if c["op"] == "fp8":
        return B.wino_fp8_conv2d(s["x"], s["filter"], s["bias"], s["y"], c["K"], c["R"], c["stride"], s["scale_x"], s["scale_w"],
                                 s["workspace"], s["layout"])
    if not c["norm"]:
        return B.wino_conv2d_fused(s["x"], s["filter"], s["bias"], s["y"], s["workspace"], s["layout"], addvec=s["vector"],
                                   residual=s["residual"], upsample=c["upsample"])
    stats = B.wino_groupnorm_stats(s["x"], GROUPS, layout=s["layout"], out=s["stats"])
    return B.wino_conv2d_fused(s["x"], s["filter"], s["bias"], s["y"], s["workspace"], s["layout"], gn_stats=stats, gn_gamma=s["gamma"],
                               gn_beta=s["beta"], gn_groups=GROUPS, addvec=s["vector"], residual=s["residual"], upsample=c["upsample"])


def work(case):
    """x, the weights, vectors and residual read once and y written once; multiply-adds of the Winograd algorithm, per output pixel
    (m + 2)^2 / m^2, or of the direct sum for the calls that are direct by definition."""
    c = case
    N, C, K, H, W, R = c["N"], c["C"], c["K"], c["H"], c["W"], c["R"]
    e = 4 if c["dtype"] == "f32" else 2
    Ho, Wo = _out_dims(c)
    up = 4 if c["upsample"] else 1
    m = _winograd_tile(c)
    nbytes = N * C * H * W * e // up + N * K * Ho * Wo * e + R * R * K * C * (1 if c["op"] == "fp8" else e) + 4 * K
    nbytes += 8 * C if c["norm"] else 0
    nbytes += 4 * N * K if c["vector"] else 0
    nbytes += N * K * Ho * Wo * e if c["residual"] else 0
    return {"bytes": nbytes, "flops": 2 * N * K * C * Ho * Wo * ((m + 2) ** 2 / m ** 2 if m else R * R)}


def tolerance(case):
    """Relative error between two correct evaluations with the same storage type.

    Measured as the distance of this path from an fp64 evaluation over the listed shapes: fp32 F(4x4) 1.2e-6, fp16 F(2x2)
    5.4e-4, F(4x4) 3.1e-3, direct 2.1e-4 (8-bit codes are decided exactly; only y rounds), bf16 F(2x2) 4.2e-3.  Four times
    that, and for fp16 F(4x4), whose promise is 5e-3 against an exact result, twice.
    """
    m = _winograd_tile(case)
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["dtype"] == "bf16":
        return {"rel": 1.6e-2}
    return {"rel": {4: 6e-3, 2: 2e-3, 0: 8e-4}[m]}

// Implicit-GEMM convolution, two-byte storage types: same operands and same staging as conv_igemm.hip (128-byte reduction stages,
// global -> LDS transfers into a ring, XOR-swizzled chunks), but built from 16x16 MFMA tiles with four waves, blocks small enough that
// two or three workgroups share a compute unit, and the fragments of the next step requested before the current one is multiplied.
//
// The layers of a UNet (1x1 shortcuts, stride 2, 8x8 ... 64x64 outputs) are bound by the latency of a stage - transfer, barrier, LDS
// read, MFMA - and what hides it is another workgroup on the same unit, not a deeper ring (64x64 blocks with 2, 3, 4 and 9 slots: within
// 3 %).  On large images the 128x128 block reaches 0.95 PFLOP/s (512 channels at 256x256 in 323 us).
//
// Rows of the block are the dimension that is contiguous in y - output channels for a channel-last y, pixels for NCHW - because a lane
// of a 16x16 accumulator holds four consecutive rows: they leave as one 8-byte store.  NCHW images with an odd number of
// pixels (no such store, nor pairs) keep the channels as rows: 16 lanes then write 16 neighbouring pixels.
#include "wino_internal.h"
#include "wino_mma.h"
#include "conv_igemm.h"

namespace wino {

// BP pixels x BK output channels per workgroup, WP x WK waves.  PIX_A: pixels are the rows (NCHW y), else output channels (channel-last y).
template <typename E, int BP, int BK, int WP, int WK, int NST, bool PIX_A>
__global__ void __launch_bounds__(WP * WK * 64)
conv_igemm_tile_kernel(const E* __restrict__ xh, const E* __restrict__ Wr, const E* __restrict__ zero_row, const float* __restrict__ bias,
                       E* __restrict__ y, float* __restrict__ part, ConvGeom g, IgemmPost post, int tiles_p, int tiles_k,
                       int total_blocks, int blocks_per_xcd, int nsplit, int vec_ok, int planes) {
    constexpr int RB = 128, CPR = RB / 16, BKE = RB / 2;  // stage: bytes, 16-byte chunks and reduction elements per row
    constexpr int BM = PIX_A ? BP : BK, BN = PIX_A ? BK : BP, WGM = PIX_A ? WP : WK, WGN = PIX_A ? WK : WP;
    constexpr int ROWS = BM + BN, NW = WP * WK;
    constexpr int LOADS = ROWS / 8, LPW = (LOADS + NW - 1) / NW;       // 1 KB transfers (8 rows) per stage, and per wave
    constexpr int WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 16, FN = WTN / 16;
    constexpr int STAGE_BYTES = ROWS * RB;
    static_assert(WTM % 16 == 0 && WTN % 16 == 0 && LOADS >= NW, "tile shape");
    static_assert(NST >= 2 && LPW * (NST - 1) < 64, "ring depth / vmcnt range");

    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int logical = (int)(blockIdx.x % 8) * blocks_per_xcd + (int)(blockIdx.x / 8);   // one contiguous range per XCD
    if (logical >= total_blocks) return;                        // uniform, before any barrier
    const int split = logical % nsplit, tile = logical / nsplit;
    int tp, tk;
    if (tiles_k <= tiles_p) { tk = tile % tiles_k; tp = tile / tiles_k; }
    else { tp = tile % tiles_p; tk = tile / tiles_p; }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int p0 = tp * BP, k0 = tk * BK;
    const int row_a0 = PIX_A ? p0 : k0, row_b0 = PIX_A ? k0 : p0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds;

    // Per-lane description of its transfers.  Filter rows: a pointer that advances with the tap.  Pixel rows: the first pixel of the image
    // and the top-left input coordinate of the output pixel.  Where the transfers do not divide by the waves the last ones
    // repeat a transfer of the same wave.
    const int lrow = lane / CPR, lchunk = lane % CPR;
    const int HoWo = g.Ho * g.Wo;
    const E* fptr[LPW];
    int pn[LPW], pi0[LPW], pj0[LPW], chunk_of[LPW];
    uint32_t dst_of[LPW];
    bool is_pix[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        int load = wave + NW * i;
        if (load >= LOADS) load -= NW;
        const int row = load * 8 + lrow;                    // row inside the stage, A rows first
        const int chunk = lchunk ^ ((row >> 1) & (CPR - 1));
        chunk_of[i] = chunk * 8;
        dst_of[i] = lds0 + (uint32_t)load * 1024u;
        const bool in_a = load * 8 < BM;
        is_pix[i] = in_a == PIX_A;                          // wave-uniform: BM is a multiple of 8
        int gr = in_a ? row_a0 + row : row_b0 + (row - BM);
        const int lim = is_pix[i] ? g.T : g.K;
        gr = gr < lim ? gr : lim - 1;                       // rows beyond the end repeat the last one; never stored
        fptr[i] = Wr + (size_t)gr * g.Cp + chunk_of[i];
        const int n = gr / HoWo, p = gr - n * HoWo;
        const int oi = p / g.Wo, oj = p - oi * g.Wo;
        pn[i] = n * g.Hs * g.Ws; pi0[i] = oi * g.st - g.pad; pj0[i] = oj * g.st - g.pad;
    }

    const int nkc = g.Cp / BKE;                             // whole stages per tap on this path
    const int nstage_all = g.R * g.R * nkc;
    const int q0 = (int)((long long)split * nstage_all / nsplit), q1 = (int)((long long)(split + 1) * nstage_all / nsplit);
    const int total = q1 - q0;

    int itap = q0 / nkc, ikc = q0 - (q0 / nkc) * nkc;
    const unsigned char* src[LPW];
    auto set_tap = [&]() __attribute__((always_inline)) {
        const int r = itap / g.R, s = itap - r * g.R;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const E* p;
            if (is_pix[i]) {
                const int ii = pi0[i] + r, jj = pj0[i] + s;
                const bool in = ii >= 0 && ii < g.H && jj >= 0 && jj < g.W;
                p = in ? xh + ((size_t)pn[i] + (size_t)(ii >> g.up) * g.Ws + (jj >> g.up)) * g.Cp + chunk_of[i] : zero_row + chunk_of[i];
            } else {
                p = fptr[i] + (size_t)itap * g.K * g.Cp;
            }
            src[i] = reinterpret_cast<const unsigned char*>(p + ikc * BKE);
        }
    };
    set_tap();
    auto issue = [&](int slot) __attribute__((always_inline)) {          // the next stage in order
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            dma_load_1k_v(src[i], dst_of[i] + (uint32_t)slot * STAGE_BYTES);
            src[i] += RB;
        }
        if (++ikc == nkc) { ikc = 0; if (++itap < g.R * g.R) set_tap(); }
    };

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // A stage holds two MFMA steps of 32 reduction elements.  The fragments of a step are requested one step ahead, across the
    // stage barrier, and waited for explicitly (as in the batched GEMM kernel).
    constexpr int NREAD = FM + FN;
    u32x4_t fa[2][FM], fb[2][FN];
    const int frow = lane & 15, fq = lane >> 4;
    const int rowA = wm * WTM + frow, rowB = BM + wn * WTN + frow;
    const uint32_t abase = lds0 + (uint32_t)rowA * RB + (uint32_t)((fq ^ ((rowA >> 1) & (CPR - 1))) << 4);
    const uint32_t bbase = lds0 + (uint32_t)rowB * RB + (uint32_t)((fq ^ ((rowB >> 1) & (CPR - 1))) << 4);
    auto read_step = [&](int slot, auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        const uint32_t a = (abase + (uint32_t)slot * STAGE_BYTES) ^ (uint32_t)(h * 64), b = (bbase + (uint32_t)slot * STAGE_BYTES) ^ (uint32_t)(h * 64);
        static_for<FM>([&](auto ic) { constexpr int i = decltype(ic)::value; lds_read16_async<i * 16 * RB>(fa[h][i], a); });
        static_for<FN>([&](auto jc) { constexpr int j = decltype(jc)::value; lds_read16_async<j * 16 * RB>(fb[h][j], b); });
    };
    auto await = [&](auto hc, auto newerc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        lds_wait<decltype(newerc)::value>();
#pragma unroll
        for (int i = 0; i < FM; ++i) pin(fa[h][i]);
#pragma unroll
        for (int j = 0; j < FN; ++j) pin(fb[h][j]);
    };
    auto mma = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) Mma16<E>::run(fa[h][i], fb[h][j], acc[i][j]);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using NR = std::integral_constant<int, NREAD>;
    static_assert(STAGE_BYTES % 128 == 0 && NREAD <= 15, "swizzle period; lgkmcnt range");

#pragma unroll
    for (int s = 0; s < NST; ++s)
        if (s < total) issue(s);
    if (NST - 1 >= total) wait_vmcnt<0>();
    else wait_vmcnt<(NST - 1) * LPW>();
    __syncthreads();
    read_step(0, I0());
    int slot = 0;
    for (int s = 0; s < total - 1; ++s) {
        const int next = slot + 1 == NST ? 0 : slot + 1;
        read_step(slot, I1());
        await(I0(), NR());
        __builtin_amdgcn_sched_barrier(0);
        mma(I0());
        __builtin_amdgcn_sched_barrier(0);
        if (s + NST >= total) wait_vmcnt<0>();              // stage s+1 has landed
        else wait_vmcnt<(NST - 2) * LPW>();
        await(I1(), I0());                                  // this wave has read all of stage s
        __syncthreads();
        if (s + NST < total) issue(slot);                   // stage s+NST, into the slot of stage s
        read_step(next, I0());
        __builtin_amdgcn_sched_barrier(0);
        mma(I1());
        __builtin_amdgcn_sched_barrier(0);
        slot = next;
    }
    read_step(slot, I1());
    await(I0(), NR());
    mma(I0());
    await(I1(), I0());
    mma(I1());

    // 16x16 accumulator layout: register r of lane l holds row 4*(l/16) + r, column l%16.  Outputs are numbered in y's own
    // order, [pixel][channel] or [channel][pixel]; partial sums are stored in that order.
    const int rowsA = PIX_A ? g.T : g.K, rowsB = PIX_A ? g.K : g.T;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int cb = row_b0 + wn * WTN + j * 16 + frow;
        if (cb >= rowsB) continue;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int ra = row_a0 + wm * WTM + i * 16 + 4 * fq;          // four rows ra .. ra+3
            if (ra >= rowsA) continue;
            f32x4_t v = acc[i][j];
            if (nsplit > 1) {
                float* dst = part + (size_t)split * rowsA * rowsB + (size_t)cb * rowsA + ra;
                if (rowsA % 4 == 0) *reinterpret_cast<f32x4_t*>(dst) = v;
                else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) if (ra + r < rowsA) dst[r] = v[r];
                }
                continue;
            }
            igemm_store4<E, PIX_A>(v, ra, cb, y, bias, g, post, vec_ok, planes);
        }
    }
}

template <typename E, int BP, int BK, int WP, int WK, int NST, bool PIX_A>
static hipError_t launch_tile_cfg(const E* xh, const E* Wr, const float* bias, E* y, float* part, int nsplit, const ConvGeom& g,
                                  const IgemmPost& post, bool planes, hipStream_t s) {
    const int tiles_p = (g.T + BP - 1) / BP, tiles_k = (g.K + BK - 1) / BK;
    const long long total = (long long)tiles_p * tiles_k * nsplit;
    if (total > 0x3fffffffLL) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    constexpr int lds_bytes = (BP + BK) * 128 * NST;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    auto kern = conv_igemm_tile_kernel<E, BP, BK, WP, WK, NST, PIX_A>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    const E* zero_row = Wr + (size_t)g.R * g.R * g.K * g.Cp;
    const int vec_ok = igemm_vec_ok<PIX_A>(g, y, post, planes);
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(WP * WK * 64), lds_bytes, s, xh, Wr, zero_row, bias, y, part, g, post,
                       tiles_p, tiles_k, (int)total, per_xcd, nsplit, vec_ok, planes ? 1 : 0);
    return hipGetLastError();
}

// Blocks on offer, pixels x output channels, with the time of a reduction stage: `alone` where a compute unit holds one workgroup,
// `each` per workgroup where it holds several, and `ends` for a workgroup's start and stores, which overlap a little (us, measured; without the last, 1x1 and other
// short reductions took the 128x128 block too often: 256 -> 560 1x1 at 144x51, N=2, 25.4 with it, 19.9 with 64x64).  Three workgroups of 64x64 or two of the others share a unit's LDS; rings
// deeper than that and fewer workgroups were slower on every shape (128x128 with three slots, one workgroup per unit, 1.3x).
struct TileShape { int bp, bk; double alone, each, ends; };
static const TileShape kTiles[3] = {{64, 64, 0.27, 0.20, 1.3}, {64, 80, 0.35, 0.295, 1.6}, {128, 128, 0.65, 0.57, 4.6}};

// The block and the number of reduction ranges with the least time by these figures, plus 6 us for the launch and, with a split reduction,
// 1.5 us and the traffic of the partial sums for the second kernel (3x3 128 channels at 17x13, N=2, NCHW: 15.5 us whole, 13.0 in two ranges).  Measured, channel-last, us, against the kernels of
// conv_igemm.hip: 1x1 960 -> 320 at 64x64 (N=2) 15.4 / 18.2, 1920 -> 640 at 64x64 36 / 45, stride 2 320 channels at 64x64 18.2 / 22.1, at
// 97x121 23.8 / 32.7, 512 channels at 256x256 88 / 110, 3x3 128 channels at 256x256 34 / 39, 512 at 256x256 323 / 338.
// Left to conv_igemm.hip: at least one round of its 256x256 blocks, of a number of channels that they divide, where that is the shorter time.
// That block fetches half as much per product, and its start and end cost less than those of four small ones; the stages themselves are
// 5 % longer, so a long reduction prefers the small blocks, and so does a last round that is not full.  Channel-last, us, here / there:
// 1x1 at 256x256 128 -> 512 53 / 40, 512 -> 512 75 / 63, 1024 -> 1024 203 / 180; 3x3 128 -> 512 121 / 101, 512 -> 512 313 / 307; at 128x128
// 1024 -> 1024 287 / 295; one and a half rounds (768 channels at 180x180) 1x1 128 in 39.7 / 36.5, 3x3 128 in 85 / 90, 1024 in 77 / 86 (1x1).
// An image of an odd number of pixels, NCHW (see below), 1x1: 192 -> 320 at 311x201 71 / 75 (with the 128x128 block 82), 256 at 181x181 41 / 38;
// 1856 -> 1184 at 23x57 (N=2) 45 / 40; but 3x3 256 at 181x181 72 / 74, 320 at 97x121 (N=2) 86 / 118.
// With a residual or a vector to add it loses: it reads them element by element (bf16 3x3, 256 -> 512 at 360x360: vector 355 / 378 NCHW, 338
// / 355 channel-last, residual 407 / 524, 380 / 439).  The number of reduction ranges is one either way.
// NCHW, where its stores are the narrower ones: 1x1 at 256x256 64 -> 512 52 / 48, 1024 -> 1024 261 / 246; 3x3 64 -> 512 89 / 81, 320 -> 512 234 / 233.
IgemmTilePlan igemm_tile_plan(int T, int HoWo, int K, int Cp, int R, int dt, bool nhwc, bool plain) {
    IgemmTilePlan best{-1, 1};
    if (!(dt == DT_F16 || dt == DT_BF16) || Cp % 64 != 0) return best;
    const int stages = R * R * (Cp / 64);
    const long long wide_blocks = (long long)((T + 255) / 256) * (K / 256);
    if (plain && K % 256 == 0 && wide_blocks >= 256) {      // one of them, or one of its 128x128 quarters, to a compute unit (us)
        const double share = (double)wide_blocks / 256.0, rounds = 0.4 * share + 0.6 * (double)((wide_blocks + 255) / 256);
        const long long small = (long long)((T + 127) / 128) * (K / 128);
        const double quarters = 0.5 * ((double)small / 256.0 + (double)((small + 255) / 256));
        if (rounds * (15.5 + 1.9 * stages) <= quarters * (nhwc ? 6.3 + 0.4425 * stages : 5.0 + 0.4525 * stages)) return best;
    }
    // never more ranges than the other kernel takes: the workspace of a call, and with it what fits the library's static scratch, stays
    // what it is there
    const int most_sp = igemm_split_rule(T, K, Cp, R, dt);
    double cost = 1e300;
    for (int id = 0; id < 3; ++id) {
        const TileShape& sh = kTiles[id];
        const long long blocks = (long long)((T + sh.bp - 1) / sh.bp) * ((K + sh.bk - 1) / sh.bk);
        for (int sp = 1; sp <= most_sp && (sp == 1 || sp * 8 <= stages); ++sp) {
            const double share = (double)(blocks * sp) / 256.0;            // workgroups per compute unit
            const double most = (double)((blocks * sp + 255) / 256), n = share < 2.0 ? 0.5 * (share + most) : most;
            const double stage = n * sh.each > sh.alone ? n * sh.each : sh.alone;
            double c = 6.0 + (double)((stages + sp - 1) / sp) * stage + (n > 1.0 ? 0.3 + 0.7 * n : 1.0) * sh.ends;
            if (sp > 1) c += 1.5 + (double)sp * K * T * 8.0 / 3e6;
            if (c < cost) { cost = c; best = {id, sp}; }
        }
    }
    // NCHW images that are no multiple of four pixels are stored one by one or in pairs, 16 lanes to 32 bytes, where the other kernel's
    // 32x32 tiles make runs of 64; with a short reduction that costs more than the stages gain, most of all with the 128x128 block
    if (plain && !nhwc && HoWo % 4 != 0) {
        const long long blocks2 = (long long)((T + 127) / 128) * ((K + 127) / 128);
        if (HoWo % 2 != 0 && stages <= 2) return {-1, 1};
        if (best.id == 2 && ((blocks2 < 256 && stages <= 32) || (HoWo % 2 != 0 && stages <= 8))) return {-1, 1};
    }
    // channel-last, a number of channels that is no multiple of four: 16 lanes to as many lines (63 -> 799 1x1 at 249x7, N=8, 54 / 33)
    if (nhwc && K % 4 != 0 && K >= 64 && best.split == 1) return {-1, 1};
    return best;
}

template <typename E, bool PIX_A>
static hipError_t launch_tile_t(const E* xh, const E* Wr, const float* bias, E* y, float* part, const IgemmTilePlan& plan, const ConvGeom& g,
                                const IgemmPost& post, bool planes, hipStream_t s) {
    switch (plan.id) {
        case 0: return launch_tile_cfg<E, 64, 64, 2, 2, 3, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 1: return launch_tile_cfg<E, 64, 80, 4, 1, 4, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 2: return launch_tile_cfg<E, 128, 128, 2, 2, 2, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_igemm_tile(const void* xh, const void* Wr, const float* bias, void* y, float* part, const IgemmTilePlan& plan,
                             const ConvGeom& g, const IgemmPost& post, int dt, bool nhwc, hipStream_t s) {
    auto run = [&](auto* tag) {
        using E = std::remove_pointer_t<decltype(tag)>;
        const bool planes = !nhwc && plan.split == 1 && g.Ho * g.Wo % 2 != 0;
        return nhwc || planes ? launch_tile_t<E, false>((const E*)xh, (const E*)Wr, bias, (E*)y, part, plan, g, post, planes, s)
                              : launch_tile_t<E, true>((const E*)xh, (const E*)Wr, bias, (E*)y, part, plan, g, post, false, s);
    };
    return dt == DT_F16 ? run(static_cast<__half*>(nullptr)) : run(static_cast<bf16_t*>(nullptr));
}

}  // namespace wino

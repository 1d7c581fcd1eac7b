// Implicit-GEMM convolution, two-byte storage types: same operands and same staging as conv_igemm.hip (128-byte reduction stages,
// global -> LDS transfers into a ring, XOR-swizzled chunks), but built from 16x16 MFMA tiles with eight waves, and the fragments of the next
// step requested before the current one is multiplied.
//
// The layers of a UNet (1x1 shortcuts, stride 2, 8x8 ... 64x64 outputs) have 2-8 us of stages between 4 us of start and stores, and a stage of
// a few hundred clocks is as long as the instructions that a wave issues in it, one in four clocks or more.  So nothing is computed
// per stage that can be computed once: a transfer is one buffer load with a fixed lane offset and a scalar that moves from stage to stage;
// what lies outside the image has an offset beyond the descriptor's range and reads zeros, so a tap is a mask and a scalar; divisions are
// multiplications prepared on the host; bias and addresses of the stores are found once.  Against pointers per transfer, tested taps and divisions
// per store (64x64 block): 320 channels at 64x64 (N=2), stride 2, channel-last 17.7 -> 14.4 us; eight waves instead of four 14.0.
// What is left of those 14.4: transfers alone 13.7, everything but the transfers 8.8, neither 4.2; the transfers run at 32 bytes per clock and
// unit (60 where every workgroup reads the same block), and neither a deeper ring nor staggered starts move that.  512 channels at
// 256x256, 3x3: 313 -> 306 us.
//
// Rows of the block are the dimension that is contiguous in y - output channels for a channel-last y, pixels for NCHW - because a lane
// of a 16x16 accumulator holds four consecutive rows: they leave as one 8-byte store.  NCHW images with an odd number of
// pixels (no such store, nor pairs) keep the channels as rows: 16 lanes then write 16 neighbouring pixels.
#include "wino_internal.h"
#include "wino_mma.h"
#include "conv_igemm.h"

namespace wino {

namespace {

struct TileGeom {
    FastDiv howo, wo, tiles, nsplit;       // divisions by Ho*Wo, Wo, the shorter tile dimension, the number of ranges
    int tiles_k_fast;                      // the shorter one is that of the output channels
    int total_blocks, blocks_per_xcd, nsplit_n, tiles_short;
};

}  // namespace

// BP pixels x BK output channels per workgroup, WP x WK waves.  PIX_A: pixels are the rows (NCHW y), else output channels (channel-last y).
template <typename E, int BP, int BK, int WP, int WK, int NST, bool PIX_A>
__global__ void __launch_bounds__(WP * WK * 64)
conv_igemm_tile_kernel(const E* __restrict__ xh, const E* __restrict__ Wr, const float* __restrict__ bias,
                       E* __restrict__ y, float* __restrict__ part, ConvGeom g, IgemmPost post, TileGeom q, int vec_ok, int planes) {
    constexpr int RB = 128, CPR = RB / 16, BKE = RB / 2;  // stage: bytes, 16-byte chunks and reduction elements per row
    constexpr int NW = WP * WK;
    constexpr int PL = BP / 8 / NW, KLOADS = BK / 8, KL = (KLOADS + NW - 1) / NW, LPW = PL + KL;      // 1 KB transfers (8 rows) per wave and stage
    constexpr int WTP = BP / WP, WTK = BK / WK, FP = WTP / 16, FK = WTK / 16;
    constexpr int STAGE_BYTES = (BP + BK) * RB;
    static_assert(BP % (8 * NW) == 0 && WTP % 16 == 0 && WTK % 16 == 0 && KLOADS >= NW, "tile shape");
    static_assert(NST >= 2 && LPW * (NST - 1) < 64, "ring depth / vmcnt range");

    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int logical = (int)(blockIdx.x % 8) * q.blocks_per_xcd + (int)(blockIdx.x / 8);   // one contiguous range per XCD
    if (logical >= q.total_blocks) return;                      // uniform, before any barrier
    const int tile = (int)divide((uint32_t)logical, q.nsplit), split = logical - tile * q.nsplit_n;
    const int t_hi = (int)divide((uint32_t)tile, q.tiles), t_lo = tile - t_hi * q.tiles_short;
    const int tk = q.tiles_k_fast ? t_lo : t_hi, tp = q.tiles_k_fast ? t_hi : t_lo;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave / WK, wk = wave % WK;
    const int p0 = tp * BP, k0 = tk * BK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds;
    const uint32_t row_bytes = (uint32_t)g.Cp * (uint32_t)sizeof(E);

    // Per-lane description of its transfers: a byte offset per transfer, fixed for the filter rows; for pixel rows that of the centre tap
    // and one bit per tap that lies inside the image.  The descriptor of x starts one row and one pixel early, so that
    // the offset of a tap, counted from the top left one, is a scalar and never negative; lanes outside read zeros.
    const int lrow = lane / CPR, lchunk = lane % CPR;
    uint32_t pbase[PL], poff[PL], inside[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        const int row = (wave + NW * i) * 8 + lrow;
        const int t = p0 + row;
        const uint32_t tc = (uint32_t)min(t, g.T - 1);
        const uint32_t n = divide(tc, q.howo), p = tc - n * (uint32_t)(g.Ho * g.Wo);
        const uint32_t oi = divide(p, q.wo), oj = p - oi * (uint32_t)g.Wo;
        const int ii = (int)oi * g.st, jj = (int)oj * g.st;
        pbase[i] = ((n * (uint32_t)g.Hs + (uint32_t)(ii >> g.up)) * (uint32_t)g.Ws + (uint32_t)(jj >> g.up)) * row_bytes +
                   (uint32_t)((lchunk ^ ((row >> 1) & (CPR - 1))) * 16);
        uint32_t m = 1u;
        if (g.R == 3) {
            const uint32_t cm = (jj > 0 ? 1u : 0u) | 2u | (jj + 1 < g.W ? 4u : 0u);
            m = (ii > 0 ? cm : 0u) | cm << 3 | (ii + 1 < g.H ? cm << 6 : 0u);
        }
        inside[i] = (t < g.T ? m : 0u) | (uint32_t)(ii & 1) << 16 | (uint32_t)(jj & 1) << 17;
    }
    uint32_t foff[KL], fdst[KL];
#pragma unroll
    for (int i = 0; i < KL; ++i) {
        int load = wave + NW * i;
        if (load >= KLOADS) load -= NW;                     // where the transfers do not divide by the waves, one is repeated
        const int row = load * 8 + lrow;
        fdst[i] = lds0 + (uint32_t)(BP / 8 + load) * 1024u;
        foff[i] = k0 + row < g.K ? (uint32_t)(k0 + row) * row_bytes + (uint32_t)((lchunk ^ (((BP + row) >> 1) & (CPR - 1))) * 16) : kOutside;
    }
    const uint32_t early = g.R == 3 ? (uint32_t)(g.Ws + 1) * row_bytes : 0u;
    const rsrc_t xr = make_rsrc(reinterpret_cast<const unsigned char*>(xh) - early);
    const rsrc_t wr = make_rsrc(Wr);

    const int nkc = g.Cp / BKE;                             // whole stages per tap on this path
    int total = g.R * g.R * nkc, itap = 0, ikc = 0;
    if (q.nsplit_n > 1) {
        const uint32_t all = (uint32_t)total;               // at most 16 ranges
        const int q0 = (int)divide((uint32_t)split * all, q.nsplit);
        total = (int)divide((uint32_t)(split + 1) * all, q.nsplit) - q0;
        itap = __builtin_amdgcn_readfirstlane(q0 / nkc);
        ikc = q0 - itap * nkc;
    }
    uint32_t soff_p = 0, soff_f = 0;
    const uint32_t tap_bytes = (uint32_t)g.K * row_bytes;
    auto set_tap = [&]() __attribute__((always_inline)) {
        const int r = itap * 11 >> 5, s = itap - 3 * r;       // itap / 3 (R == 1: one tap, 0)
        soff_f = (uint32_t)itap * tap_bytes + (uint32_t)ikc * RB;
        soff_p = (uint32_t)ikc * RB;
        if (!g.up) {
            soff_p += (uint32_t)(r * g.Ws + s) * row_bytes;
#pragma unroll
            for (int i = 0; i < PL; ++i) poff[i] = (inside[i] >> itap) & 1u ? pbase[i] : kOutside;
        } else {
#pragma unroll
            for (int i = 0; i < PL; ++i) {                  // the stored row and column move with every other tap (3x3: nothing else is read upsampled)
                const int dr = ((int)(inside[i] >> 16 & 1u) + r + 1) >> 1, dc = ((int)(inside[i] >> 17 & 1u) + s + 1) >> 1;
                poff[i] = (inside[i] >> itap) & 1u ? pbase[i] + (uint32_t)(dr * g.Ws + dc) * row_bytes : kOutside;
            }
        }
    };
    set_tap();
    auto issue = [&](uint32_t slot_off) __attribute__((always_inline)) {          // the next stage in order
#pragma unroll
        for (int i = 0; i < PL; ++i) dma_buffer_1k(xr, poff[i], soff_p, lds0 + slot_off + (uint32_t)(wave + NW * i) * 1024u);
#pragma unroll
        for (int i = 0; i < KL; ++i) dma_buffer_1k(wr, foff[i], soff_f, fdst[i] + slot_off);
        soff_p += RB; soff_f += RB;
        if (++ikc == nkc) { ikc = 0; ++itap; set_tap(); }
    };

    f32x4_t acc[FP][FK];
#pragma unroll
    for (int i = 0; i < FP; ++i)
#pragma unroll
        for (int j = 0; j < FK; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // A stage holds two MFMA steps of 32 reduction elements.  The fragments of a step are requested one step ahead, across the
    // stage barrier, and waited for explicitly (as in the batched GEMM kernel).
    constexpr int NREAD = FP + FK;
    u32x4_t fp[2][FP], fk[2][FK];
    const int frow = lane & 15, fq = lane >> 4;
    const int rowP = wp * WTP + frow, rowK = BP + wk * WTK + frow;
    const uint32_t pfrag = lds0 + (uint32_t)rowP * RB + (uint32_t)((fq ^ ((rowP >> 1) & (CPR - 1))) << 4);
    const uint32_t kfrag = lds0 + (uint32_t)rowK * RB + (uint32_t)((fq ^ ((rowK >> 1) & (CPR - 1))) << 4);
    auto read_step = [&](uint32_t slot_off, auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        const uint32_t a = (pfrag ^ (uint32_t)(h * 64)) + slot_off, b = (kfrag ^ (uint32_t)(h * 64)) + slot_off;
        static_for<FP>([&](auto ic) { constexpr int i = decltype(ic)::value; lds_read16_async<i * 16 * RB>(fp[h][i], a); });
        static_for<FK>([&](auto jc) { constexpr int j = decltype(jc)::value; lds_read16_async<j * 16 * RB>(fk[h][j], b); });
    };
    auto await = [&](auto hc, auto newerc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
        lds_wait<decltype(newerc)::value>();
#pragma unroll
        for (int i = 0; i < FP; ++i) pin(fp[h][i]);
#pragma unroll
        for (int j = 0; j < FK; ++j) pin(fk[h][j]);
    };
    auto mma = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int i = 0; i < FP; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) {
                if constexpr (PIX_A) Mma16<E>::run(fp[h][i], fk[h][j], acc[i][j]);
                else Mma16<E>::run(fk[h][j], fp[h][i], acc[i][j]);
            }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using NR = std::integral_constant<int, NREAD>;
    static_assert(STAGE_BYTES % 128 == 0 && NREAD <= 15, "swizzle period; lgkmcnt range");

    // requested ahead of the transfers, used after the last of them
    f32x4_t bv[FK];
#pragma unroll
    for (int j = 0; j < FK; ++j) {
        const int k = k0 + wk * WTK + j * 16 + (PIX_A ? frow : 4 * fq);
        bv[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (bias) {
            if constexpr (PIX_A) { bv[j] += bias[min(k, g.K - 1)]; }
            else {
#pragma unroll
                for (int r = 0; r < 4; ++r) bv[j][r] = bias[min(k + r, g.K - 1)];
            }
        }
    }
    constexpr uint32_t RING = NST * STAGE_BYTES;
    {
        const int first = total < NST ? total : NST;
#pragma unroll 1
        for (int s = 0; s < first; ++s) issue((uint32_t)s * STAGE_BYTES);
    }
    if (NST - 1 >= total) wait_vmcnt<0>();
    else wait_vmcnt<(NST - 1) * LPW>();
    __syncthreads();
    read_step(0u, I0());
    uint32_t slot = 0;
    auto stage = [&](auto morec, auto drainc) __attribute__((always_inline)) {
        uint32_t next = slot + STAGE_BYTES;
        next = next == RING ? 0u : next;
        read_step(slot, I1());
        await(I0(), NR());
        __builtin_amdgcn_sched_barrier(0);
        mma(I0());
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(drainc)::value) wait_vmcnt<0>();
        else wait_vmcnt<(NST - 2) * LPW>();                 // stage s+1 has landed
        await(I1(), I0());                                  // this wave has read all of stage s
        __syncthreads();
        if constexpr (decltype(morec)::value) issue(slot);  // stage s+NST, into the slot of stage s
        read_step(next, I0());
        __builtin_amdgcn_sched_barrier(0);
        mma(I1());
        __builtin_amdgcn_sched_barrier(0);
        slot = next;
    };
    int s = 0;
#pragma unroll 1
    for (; s + NST < total; ++s) stage(std::true_type(), std::false_type());
#pragma unroll 1
    for (; s < total - 1; ++s) stage(std::false_type(), std::true_type());
    read_step(slot, I1());
    await(I0(), NR());
    mma(I0());
    await(I1(), I0());
    mma(I1());

    // 16x16 accumulator layout: register r of lane l holds row 4*(l/16) + r, column l%16.  Outputs are numbered in y's own
    // order, [pixel][channel] or [channel][pixel]; partial sums are stored in that order.
    const int rowsA = PIX_A ? g.T : g.K, rowsB = PIX_A ? g.K : g.T;
    if (q.nsplit_n > 1) {
#pragma unroll
        for (int i = 0; i < FP; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) {
                const int pr = p0 + wp * WTP + i * 16, kr = k0 + wk * WTK + j * 16;
                const int ra = (PIX_A ? pr : kr) + 4 * fq, cb = (PIX_A ? kr : pr) + frow;
                if (ra >= rowsA || cb >= rowsB) continue;
                float* dst = part + (size_t)split * rowsA * rowsB + (size_t)cb * rowsA + ra;
                if (rowsA % 4 == 0) *reinterpret_cast<f32x4_t*>(dst) = acc[i][j];
                else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) if (ra + r < rowsA) dst[r] = acc[i][j][r];
                }
            }
        return;
    }
    if (!vec_ok) {
#pragma unroll
        for (int i = 0; i < FP; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) {
                const int pr = p0 + wp * WTP + i * 16, kr = k0 + wk * WTK + j * 16;
                const int ra = (PIX_A ? pr : kr) + 4 * fq, cb = (PIX_A ? kr : pr) + frow;
                igemm_store4<E, PIX_A>(acc[i][j], ra, cb, y, bias, g, post, vec_ok, planes);
            }
        return;
    }
    // the four outputs of a lane are adjacent and 8-byte aligned; the addresses along one dimension are found once
    const uint32_t howo = (uint32_t)(g.Ho * g.Wo);
    const E* res = static_cast<const E*>(post.residual);
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int pr = p0 + wp * WTP + i * 16 + (PIX_A ? 4 * fq : frow);           // first pixel of this lane
        const bool p_ok = pr < g.T;
        uint32_t n = 0;
        size_t prow;                                        // offset of (pixel, channel 0) in y
        if constexpr (PIX_A) {
            n = divide((uint32_t)min(pr, g.T - 1), q.howo);
            prow = (size_t)n * g.K * howo + ((uint32_t)pr - n * howo);
        } else {
            if (post.addvec) n = divide((uint32_t)min(pr, g.T - 1), q.howo);
            prow = (size_t)pr * g.K;
        }
        uint2 rr[FK];
        f32x4_t av[FK];
#pragma unroll
        for (int j = 0; j < FK; ++j) {
            const int k = k0 + wk * WTK + j * 16 + (PIX_A ? frow : 4 * fq);
            rr[j] = make_uint2(0u, 0u);
            av[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (!(p_ok && k < g.K)) continue;
            if (res) rr[j] = *reinterpret_cast<const uint2*>(res + prow + (PIX_A ? (size_t)k * howo : (size_t)k));
            if (post.addvec) {
                const float* a = post.addvec + (size_t)n * g.K + k;
                if constexpr (PIX_A) av[j] += a[0];
                else { av[j][0] += a[0]; av[j][1] += a[1]; av[j][2] += a[2]; av[j][3] += a[3]; }
            }
        }
#pragma unroll
        for (int j = 0; j < FK; ++j) {
            const int k = k0 + wk * WTK + j * 16 + (PIX_A ? frow : 4 * fq);
            if (!(p_ok && k < g.K)) continue;
            f32x4_t v = acc[i][j] + (bv[j] + av[j]);
            if (res) { v[0] += lo16<E>(rr[j].x); v[1] += hi16<E>(rr[j].x); v[2] += lo16<E>(rr[j].y); v[3] += hi16<E>(rr[j].y); }
            *reinterpret_cast<uint2*>(y + prow + (PIX_A ? (size_t)k * howo : (size_t)k)) = make_uint2(pack2<E>(v[0], v[1]), pack2<E>(v[2], v[3]));
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
    TileGeom q;
    q.tiles_k_fast = tiles_k <= tiles_p;
    q.tiles_short = q.tiles_k_fast ? tiles_k : tiles_p;
    q.howo = fast_div((uint32_t)(g.Ho * g.Wo)); q.wo = fast_div((uint32_t)g.Wo);
    q.tiles = fast_div((uint32_t)q.tiles_short); q.nsplit = fast_div((uint32_t)nsplit);
    q.total_blocks = (int)total; q.blocks_per_xcd = per_xcd; q.nsplit_n = nsplit;
    const int vec_ok = igemm_vec_ok<PIX_A>(g, y, post, planes);
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(WP * WK * 64), lds_bytes, s, xh, Wr, bias, y, part, g, post, q, vec_ok, planes ? 1 : 0);
    return hipGetLastError();
}

// Blocks on offer, pixels x output channels, of eight waves (but for 64x32 and 64x80, of four), and the two of conv_igemm.hip that are compared with
// them where outputs are stored one by one, with the time of a reduction stage: `alone` where a compute unit holds one workgroup, `each` per
// workgroup where it holds several; `first`, `more`: start and stores of the first workgroup of a unit, beyond those of a launch, and of each further
// one; and what 4096 outputs cost beyond that where they are no 8-byte pieces of y: single elements of a channel-last y, pairs and single
// elements of an NCHW y (us, fitted together to 2800 calls with up to eight blocks and ten numbers of ranges each, 31000 timings: 1x1, stride 2 and 3x3, 1 to 280
// stages, 8 to 1400 output channels, 40 to 1.5 million pixels, both layouts.  Every figure is a time, so a call's time grows with its pixels; it is within 12 % of the
// measured one, and the choice within 0.5 % of the best on average).  The 128x96 block with three slots fills a unit by itself: it is for calls of one
// round, where two slots leave the transfers waiting.
struct TileShape { int bp, bk; double alone, each, first, more, elem, pair, planes; };
constexpr int kTileBlocks = 7;
static const TileShape kTiles[kTileBlocks + 2] = {
    {64, 64, 0.15, 0.212, 0.32, 1.22, 1.10, 0.51, 0.53}, {128, 64, 0.20, 0.294, 1.45, 1.39, 1.35, 0.73, 0.82},
    {128, 96, 0.534, 0.414, 1.73, 1.92, 1.45, 0.69, 0.89}, {128, 96, 0.30, 0.417, 1.99, 5.56, 1.56, 0.73, 0.91},
    {128, 128, 0.30, 0.504, 3.77, 1.85, 1.45, 0.73, 0.79}, {64, 32, 0.181, 0.145, 0.01, 0.62, 2.10, 0.83, 0.72},
    {64, 80, 0.265, 0.28, 1.53, 2.06, 1.52, 0.85, 1.34},
    {64, 64, 0.419, 0.122, 3.28, 0.02, 0.02, 0., 0.}, {128, 128, 0.30, 0.48, 5.02, 1.55, 1.17, 0., 0.}};

// Time of a call by these figures, less what all its blocks share; split: reduction ranges, whose second kernel and partial sums it includes.
double igemm_block_time(int id, int T, int HoWo, int K, int Cp, int R, bool nhwc, int split) {
    const TileShape& sh = kTiles[id];
    const int stages = R * R * (Cp / 64);
    const long long blocks = (long long)((T + sh.bp - 1) / sh.bp) * ((K + sh.bk - 1) / sh.bk) * split;
    const double share = (double)blocks / 256.0, most = (double)((blocks + 255) / 256);                 // workgroups per compute unit
    double n = share < 2.0 ? 0.51 * share + 0.49 * most : most;
    if (n < 1.0) n = 1.0;
    const double stage = n * sh.each > sh.alone ? n * sh.each : sh.alone;
    double c = (double)((stages + split - 1) / split) * stage + sh.first + sh.more * (n - 1.0);
    if (split > 1) return c + 2.31 + (double)split * K * T * 8.0 * 0.295e-6;
    const double store = nhwc ? (K % 4 == 0 ? 0. : sh.elem) : (HoWo % 4 == 0 ? 0. : HoWo % 2 == 0 ? sh.pair : sh.planes);
    return c + n * store * (sh.bp * sh.bk / 4096.0);
}

// The block and the number of reduction ranges with the least time; a split reduction adds a second kernel and the traffic of the partial
// sums (stride 2, 1088 -> 23 at 16x17, NCHW: 36.0 us whole, 14.0 in eight ranges).  The 64x32 block is for up to 64 channels, 64x80 for more and up to 400, where
// it was measured: it is ahead on long reductions in one round (us, the other blocks / 64x80: 832 -> 68 at 311x185, stride 2, 47.7 / 39.3, 1088 -> 80 at
// 183x319, stride 2, NCHW 176 / 159, 1600 -> 144 at 57x55 (N=2) 67.2 / 62.5).  Short reductions on large images, which a block with empty columns used to
// take (us, channel-last, 128x128 / now): 1x1 64 -> 64 at 999x1014 86.1 / 68.9, 64 -> 48 at 400x453 14.8 / 12.2, 128 -> 56 at 645x659 43.3 / 37.8, 64 -> 160 at
// 568x625 (N=2) 128 / 112, 192 -> 192 at 121x177 (N=2) NCHW 43.4 / 37.6.  Against the kernels of conv_igemm.hip: 1x1 256 -> 256 at 414x300 (N=2) 91 / 99, 64 ->
// 1280 at 200x112 25.5 / 33.4, 3x3 320 -> 768 at 104x544 255 / 294, stride 2 64 -> 768 at 465x168 (N=2) 52 / 64.
IgemmTilePlan igemm_block_plan(int T, int HoWo, int K, int Cp, int R, int dt, bool nhwc, int most_sp) {
    IgemmTilePlan best{-1, 1};
    if (!(dt == DT_F16 || dt == DT_BF16) || Cp % 64 != 0) return best;
    const int stages = R * R * (Cp / 64);
    const auto blocks = [&](int bp, int bk) { return (long long)((T + bp - 1) / bp) * ((K + bk - 1) / bk); };
    // 1x1, full rounds of that file's 256x256 block, which moves half as much into LDS per product (us, 128x128 here / 256x256 there).  From seven
    // stages on: channel-last 512 -> 512 at 512x512 252 / 242, 1280 -> 512 at 296x432 245 / 218, 640 -> 256 at 664x456 191 / 181,
    // 896 -> 256 at 704x160 94.9 / 87.6, 640 -> 1024 at 408x232 214 / 201; NCHW 512 ->
    // 512 at 512x512 413 / 383, 832 -> 512 at 272x600 375 / 332, 896 -> 1024 at 256x576 574 / 498; but fewer stages (256 -> 256 at 496x592 105 / 118), a
    // last round that is not full (640 -> 768 at 128x752 155 / 166) and, NCHW, few rounds (512 -> 512 at 256x256 84 / 95, 512 -> 1024 at 256x256 142 / 157; channel-last
    // 66.8 / 64.9 and 125.6 / 123.3).  NCHW images that are no multiple of four pixels, of any number of stages: its 32x32 tiles store runs of 64
    // bytes, sixteen lanes of this kernel 32 (odd 640 -> 512 at 415x473 525 / 434, 64 -> 512 at 343x473 135 / 119, 512 -> 512 at 305x199 127 / 123; pairs 64 -> 256 at
    // 829x778 308 / 274, 320 -> 256 at 578x515 335 / 312, 128 -> 768 at 353x358 162 / 163; but 384 -> 768 at 157x189 64 / 72, 640 -> 512 at 233x302 163 /
    // 181).  3x3 it loses: 128 -> 768 at 221x333 189 / 218, and 260 calls of whole pieces.
    if (R == 1 && K % 256 == 0) {
        const bool ragged = !nhwc && HoWo % 4 != 0, few = K <= 512;
        const double share = (double)blocks(256, 256) / 256.0, fill = share / (double)((blocks(256, 256) + 255) / 256);
        const double least = ragged ? (HoWo % 2 != 0 ? 1.5 : 3.5) : nhwc ? 1.5 : few ? 2.5 : 6.5;
        if (share >= least && (ragged || stages >= 7) && fill >= (ragged ? 0.7 : nhwc && K == 256 ? 0.86 : few ? 0.91 : 0.96)) return best;
    }
    double cost = 1e300;
    for (int id = 0; id < kTileBlocks; ++id) {
        if ((id == 5 && K > 64) || (id == 6 && (K <= 64 || K > 400))) continue;
        for (int sp = 1; sp <= most_sp && (sp == 1 || sp * 8 <= stages); ++sp) {
            const double c = igemm_block_time(id, T, HoWo, K, Cp, R, nhwc, sp);
            if (c < cost) { cost = c; best = {id, sp}; }
        }
    }
    // one column of blocks: a long reduction prefers the smaller block, whose three workgroups to a unit hide each other's transfers (us, 128x64 / 64x64,
    // channel-last: 3x3 384 -> 48 at 315x249, 54 stages, 62.2 / 52.6, 512 -> 64 at 330x354 132 / 118, 704 -> 60 at 252x295 136 / 105; but 320 -> 62, 45
    // stages, 1.18 times, 256 -> 49, 36 stages, 1.16 times)
    if (best.id == 1 && best.split == 1 && K <= 64 && stages >= 54) best.id = 0;
    // 1x1, channel-last, a number of channels that is no multiple of four: outputs are stored one by one, 16 lanes to as many lines, where the
    // other file's 32x32 tiles make runs of 64 bytes (us, here / there: 64 -> 243 at 544x392 117 / 99, 128 -> 1379 at 22x24 (N=4) 11.4 / 8.6, 256 -> 118 at 187x154
    // 13.4 / 11.5, 640 -> 319 at 274x190 (N=4) 247 / 241; but 64 -> 130 at 159x192 14.0 / 16.2, 192 -> 306 21.1 / 31.1, 64 -> 126 at 5313 pixels 5.2 / 6.0)
    if (nhwc && R == 1 && K % 4 != 0 && K > 64 && best.split == 1 &&
        igemm_block_time(kTileBlocks + (blocks(128, 128) >= 256 ? 1 : 0), T, HoWo, K, Cp, R, nhwc, 1) < cost) return {-1, 1};
    return best;
}

// Reduction ranges that a call's workspace is sized for; 0: igemm_split_rule says.  The choice of an earlier set of blocks, 64x64, 64x80 and 128x128, with their
// stage times (us; `alone`: one workgroup to a compute unit, `each`: several, `ends`: a workgroup's start and stores).  Programs keep workspaces,
// and what fits the library's static scratch fits it, so this rule stays what it was whatever block runs a call; igemm_block_plan
// never takes more ranges than it grants.
struct RangeShape { int bp, bk; double alone, each, ends; };
static const RangeShape kRangeTiles[3] = {{64, 64, 0.27, 0.20, 1.3}, {64, 80, 0.35, 0.295, 1.6}, {128, 128, 0.65, 0.57, 4.6}};
int igemm_tile_ranges(int T, int HoWo, int K, int Cp, int R, int dt, bool nhwc) {
    if (!(dt == DT_F16 || dt == DT_BF16) || Cp % 64 != 0) return 0;
    const int stages = R * R * (Cp / 64);
    const long long wide_blocks = (long long)((T + 255) / 256) * (K / 256);
    if (K % 256 == 0 && wide_blocks >= 256) {               // a round of the 256x256 block of conv_igemm.hip, or of its 128x128 quarters (us)
        const double share = (double)wide_blocks / 256.0, rounds = 0.4 * share + 0.6 * (double)((wide_blocks + 255) / 256);
        const long long small = (long long)((T + 127) / 128) * (K / 128);
        const double quarters = 0.5 * ((double)small / 256.0 + (double)((small + 255) / 256));
        if (rounds * (15.5 + 1.9 * stages) <= quarters * (nhwc ? 6.3 + 0.4425 * stages : 5.0 + 0.4525 * stages)) return 0;
    }
    const int most_sp = igemm_split_rule(T, K, Cp, R, dt);  // never more ranges than the other kernel takes
    int best = 0, ranges = 1;
    double cost = 1e300;
    for (int id = 0; id < 3; ++id) {
        const RangeShape& sh = kRangeTiles[id];
        const long long blocks = (long long)((T + sh.bp - 1) / sh.bp) * ((K + sh.bk - 1) / sh.bk);
        for (int sp = 1; sp <= most_sp && (sp == 1 || sp * 8 <= stages); ++sp) {
            const double share = (double)(blocks * sp) / 256.0;            // workgroups per compute unit
            const double most = (double)((blocks * sp + 255) / 256), n = share < 2.0 ? 0.5 * (share + most) : most;
            const double stage = n * sh.each > sh.alone ? n * sh.each : sh.alone;
            double c = 6.0 + (double)((stages + sp - 1) / sp) * stage + (n > 1.0 ? 0.3 + 0.7 * n : 1.0) * sh.ends;
            if (sp > 1) c += 1.5 + (double)sp * K * T * 8.0 / 3e6;
            if (c < cost) { cost = c; best = id; ranges = sp; }
        }
    }
    // outputs stored one by one or in pairs, where that set left short reductions and the 128x128 block to the other kernel
    if (!nhwc && HoWo % 4 != 0) {
        const long long blocks2 = (long long)((T + 127) / 128) * ((K + 127) / 128);
        if (HoWo % 2 != 0 && stages <= 2) return 0;
        if (best == 2 && ((blocks2 < 256 && stages <= 32) || (HoWo % 2 != 0 && stages <= 8))) return 0;
    }
    if (nhwc && K % 4 != 0 && K >= 64 && ranges == 1) return 0;
    return ranges;
}

template <typename E, bool PIX_A>
static hipError_t launch_tile_t(const E* xh, const E* Wr, const float* bias, E* y, float* part, const IgemmTilePlan& plan, const ConvGeom& g,
                                const IgemmPost& post, bool planes, hipStream_t s) {
    switch (plan.id) {
        case 0: return launch_tile_cfg<E, 64, 64, 4, 2, 4, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 1: return launch_tile_cfg<E, 128, 64, 4, 2, 3, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 2: return launch_tile_cfg<E, 128, 96, 4, 2, 2, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 3: return launch_tile_cfg<E, 128, 96, 4, 2, 3, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 4: return launch_tile_cfg<E, 128, 128, 4, 2, 2, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 5: return launch_tile_cfg<E, 64, 32, 2, 2, 4, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        case 6: return launch_tile_cfg<E, 64, 80, 4, 1, 4, PIX_A>(xh, Wr, bias, y, part, plan.split, g, post, planes, s);
        default: return hipErrorInvalidValue;
    }
}

// Lane offsets are 32-bit and a descriptor covers 2 GB: x, with a row and a pixel in front of it, and the filter have to fit; so has the scalar
// offset by itself, two rows, two pixels and the channels of one, which is more than x where that is a single row: beyond the range it
// would not be sure that lanes at kOutside fail the test against what is left of it.
bool igemm_tile_fits(const ConvGeom& g) {
    const unsigned long long row = (unsigned long long)g.Cp * 2u, lim = kRange, ws = (unsigned long long)g.Ws;
    const unsigned long long operand = (unsigned long long)g.N * g.Hs * ws + ws + 1u, scalar = 2u * ws + 3u;
    return (operand > scalar ? operand : scalar) <= lim / row && (unsigned long long)g.R * g.R * g.K <= lim / row;
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

// Implicit-GEMM convolution on 8-bit floating-point operands (E4M3): operands and staging as in conv_igemm.hip (128-byte stages, global
// -> LDS transfers into a ring, XOR-swizzled chunks), 32x32x64 MFMA steps, outputs in a two-byte type.
//
// A stage of 128 reduction elements is two MFMA steps.  The kernel of conv_igemm.hip reads all fragments of a stage behind its barrier
// and multiplies them when the last has arrived; here the fragments of a step are requested one step ahead, across the barrier, and the
// stage after next is requested in the middle of a stage.  The 256x256 block has eight waves of 64x128 instead of sixteen of 64x64: LDS
// feeds a 64x64 piece at exactly the rate at which it is multiplied, and the transfers into LDS come on top; a 64x128 piece needs 3/4
// of that.  256 channels at 512x512: 208 -> 162 us (1.9 PFLOP/s), four rounds of workgroups of 18 stages.  About 30 us of it are start and
// stores, which one workgroup to a unit does not overlap (1x1: 41 us with one stage, 10 more for each further one of the four rounds), the
// rest 1.8 us a stage; a further stage of a long reduction costs 1.4 (1024 channels: 288 stages in 501 us).  Its products alone take 0.85.
//
// Rows of the block are the dimension that is contiguous in y, as in conv_igemm_tile.hip: four consecutive rows leave as one store.
#include "wino_internal.h"
#include "wino_mma.h"
#include "conv_igemm.h"

namespace wino {

namespace {
constexpr int NST = 2;                                   // ring slots (three with a 256x128 block: within 3 % on every shape)

// every LDS read of the wave has arrived (the caller's waits say so); the workgroup barrier
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }
}  // namespace

// RAGGED: Cp is not a whole number of stages.
// BP pixels x BK output channels per workgroup, WP x WK waves, two ring slots.  PIX_A: pixels are the rows (NCHW y), else channels.
template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A, bool RAGGED>
__global__ void __launch_bounds__(WP * WK * 64)
conv_igemm_fp8_kernel(const uint8_t* __restrict__ xq, const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ zero_row,
                      const float* __restrict__ bias, EO* __restrict__ y, ConvGeom g, IgemmPost post, int tiles_p, int tiles_k,
                      int total_blocks, int blocks_per_xcd, int vec_ok, int planes) {
    constexpr int RB = 128, CPR = RB / 16;                // stage bytes (= reduction elements) and 16-byte chunks per row
    constexpr int BM = PIX_A ? BP : BK, BN = PIX_A ? BK : BP, WGM = PIX_A ? WP : WK, WGN = PIX_A ? WK : WP;
    constexpr int ROWS = BM + BN, NW = WP * WK;
    constexpr int LPX = BP / 8 / NW, LPF = BK / 8 / NW;   // 1 KB transfers (8 rows) per wave and stage: pixels, filter
    constexpr int WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 32, FN = WTN / 32;
    constexpr int STAGE_BYTES = ROWS * RB;
    constexpr int PIX0 = PIX_A ? 0 : BM, FIL0 = PIX_A ? BM : 0;            // first stage row of each operand
    static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BP % (8 * NW) == 0 && BK % (8 * NW) == 0, "tile shape");

    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    // after the ring, per pixel row: image offset (pixels) and the top-left input coordinate of its output pixel
    int* rowtab = reinterpret_cast<int*>(lds + NST * STAGE_BYTES);

    const int logical = (int)(blockIdx.x % 8) * blocks_per_xcd + (int)(blockIdx.x / 8);   // one contiguous range per XCD
    if (logical >= total_blocks) return;                  // uniform, before any barrier
    int tp, tk;
    if (tiles_k <= tiles_p) { tk = logical % tiles_k; tp = logical / tiles_k; }
    else { tp = logical % tiles_p; tk = logical / tiles_p; }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int p0 = tp * BP, k0 = tk * BK;
    const int row_a0 = PIX_A ? p0 : k0, row_b0 = PIX_A ? k0 : p0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds;
    const int HoWo = g.Ho * g.Wo;

    for (int r = tid; r < BP; r += NW * 64) {             // pixels beyond the end repeat the last one; never stored
        const int t = min(p0 + r, g.T - 1);
        const int n = t / HoWo, p = t - n * HoWo;
        const int oi = p / g.Wo, oj = p - oi * g.Wo;
        rowtab[3 * r] = n * g.Hs * g.Ws; rowtab[3 * r + 1] = oi * g.st - g.pad; rowtab[3 * r + 2] = oj * g.st - g.pad;
    }
    __syncthreads();

    // Transfers of a wave: rows wave * 8 + 8 * NW * i of either operand.  The chunk a lane fetches is swizzled by the stage row;
    // 8 * NW rows further on the swizzle is the same.
    const int lrow = wave * 8 + (lane >> 3);
    static_assert(PIX0 % 16 == 0 && FIL0 % 16 == 0 && (8 * NW) % 16 == 0, "one swizzle per lane");
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ ((lrow >> 1) & (CPR - 1))) * 16);
    const uint32_t pdst = lds0 + (uint32_t)(PIX0 * RB) + (uint32_t)wave * 1024u, fdst = lds0 + (uint32_t)(FIL0 * RB) + (uint32_t)wave * 1024u;
    uint32_t foff[LPF];
#pragma unroll
    for (int i = 0; i < LPF; ++i) foff[i] = (uint32_t)(min(k0 + lrow + 8 * NW * i, g.K - 1) - k0) * (uint32_t)g.Cp + chunk;
    const uint8_t* fbase = Wq + (size_t)k0 * g.Cp;        // wave-uniform, walks stages and taps

    // The next stage to fetch: prepare() finds its pixel rows (a branch at each tap), issue() is free of branches, so that it and the two
    // steps of a stage are one basic block: across a branch the compiler moves the products of a step behind the transfers.
    const int nkc = (g.Cp + RB - 1) / RB;
    const int total = g.R * g.R * nkc;
    const int tail = g.Cp - (nkc - 1) * RB;               // bytes of a row in the last stage of a tap
    const size_t fstep = (size_t)g.K * g.Cp - (size_t)(nkc - 1) * RB;
    int itap = 0, ikc = 0;
    const uint8_t* src[LPX];
    auto prepare = [&]() __attribute__((always_inline)) {
        if (ikc != 0) return;
        const int r = itap / g.R, s = itap - r * g.R;
#pragma unroll
        for (int i = 0; i < LPX; ++i) {
            const int* e = rowtab + 3 * (lrow + 8 * NW * i);
            const int ii = e[1] + r, jj = e[2] + s;
            const bool in = ii >= 0 && ii < g.H && jj >= 0 && jj < g.W;
            src[i] = (in ? xq + ((size_t)e[0] + (size_t)(ii >> g.up) * g.Ws + (jj >> g.up)) * g.Cp : zero_row) + chunk;
        }
    };
    auto issue = [&](uint32_t at) __attribute__((always_inline)) {         // into the slot at byte `at` of the ring
        const bool past = RAGGED && ikc == nkc - 1 && (int)chunk >= tail;   // chunks beyond Cp come from the row of zeros
#pragma unroll
        for (int i = 0; i < LPX; ++i) { dma_load_1k_v(past ? zero_row : src[i], pdst + at + (uint32_t)(8 * NW * i) * RB); src[i] += RB; }
#pragma unroll
        for (int i = 0; i < LPF; ++i) {
            if constexpr (RAGGED) dma_load_1k_v(past ? zero_row : fbase + foff[i], fdst + at + (uint32_t)(8 * NW * i) * RB);
            else dma_load_1k_s(fbase, foff[i], fdst + at + (uint32_t)(8 * NW * i) * RB);
        }
        const bool wrap = ikc == nkc - 1;
        fbase += wrap ? fstep : (size_t)RB;
        itap += wrap ? 1 : 0;
        ikc = wrap ? 0 : ikc + 1;
    };

    float16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Lane l of a 32x32x64 step holds two neighbouring chunks of row l % 32, the pair l / 32 of the step's two.  Both steps' fragments
    // at once would not fit beside 128 accumulators: the row fragments have two sets, and a column fragment is read into the registers
    // of its predecessor as soon as that has been multiplied - except the last, which has two, so that the last read of a stage is not
    // waited for at once.  Reads of a step, in order: rows, last column, first column ... last but one.
    u32x4_t fa[2][FM][2], fb[FN + 1][2];                  // [step][sub-tile][chunk]; fb[FN]: last column of step 1
    const int frow = lane & 31, fh = lane >> 5;
    const uint32_t swz = (uint32_t)(((2 * fh) ^ ((frow >> 1) & (CPR - 1))) << 4);
    const uint32_t abase = lds0 + (uint32_t)(wm * WTM + frow) * RB + swz, bbase = lds0 + (uint32_t)(BM + wn * WTN + frow) * RB + swz;
    auto read_b = [&](uint32_t b, auto jc, auto rc) __attribute__((always_inline)) {        // sub-tile j into register set r
        constexpr int j = decltype(jc)::value, r = decltype(rc)::value;
        lds_read16_async<j * 32 * RB>(fb[r][0], b);
        lds_read16_async<j * 32 * RB>(fb[r][1], b ^ 16u);
    };
    auto read_first = [&](uint32_t a, uint32_t b, auto hc) __attribute__((always_inline)) { // rows and last column of step h
        constexpr int h = decltype(hc)::value;
        static_for<FM>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            lds_read16_async<i * 32 * RB>(fa[h][i][0], a);
            lds_read16_async<i * 32 * RB>(fa[h][i][1], a ^ 16u);
        });
        read_b(b, std::integral_constant<int, FN - 1>(), std::integral_constant<int, FN - 1 + h>());
    };
    auto pin_first = [&](auto hc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int i = 0; i < FM; ++i) { pin(fa[h][i][0]); pin(fa[h][i][1]); }
        pin(fb[FN - 1 + h][0]); pin(fb[FN - 1 + h][1]);
    };
    auto mma = [&](auto hc, auto jc) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value, j = decltype(jc)::value, r = j == FN - 1 ? FN - 1 + h : j;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < FM; ++i)
            Mma<fp8_t>::run2(__builtin_bit_cast(uint4, fa[h][i][0]), __builtin_bit_cast(uint4, fa[h][i][1]),
                             __builtin_bit_cast(uint4, fb[r][0]), __builtin_bit_cast(uint4, fb[r][1]), acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // step 0 of a stage, whose fragments have been requested; requests step 1
    auto step0 = [&](uint32_t slot_off) __attribute__((always_inline)) {
        const uint32_t a = (abase + slot_off) ^ 64u, b = (bbase + slot_off) ^ 64u;
        lds_wait<2 * (FN - 2)>();
        pin_first(std::integral_constant<int, 0>());
        read_first(a, b, std::integral_constant<int, 1>());
        static_for<FN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j > 0 && j < FN - 1) lds_wait<2 * (FN - 2 - j) + 2 * FM + 2 + 2 * j>();
            if constexpr (j < FN - 1) { pin(fb[j][0]); pin(fb[j][1]); }
            mma(std::integral_constant<int, 0>(), jc);
            if constexpr (j < FN - 1) read_b(b, jc, jc);
        });
    };
    auto pin_step1 = [&]() __attribute__((always_inline)) {
        lds_wait<0>();
        pin_first(std::integral_constant<int, 1>());
#pragma unroll
        for (int j = 0; j < FN - 1; ++j) { pin(fb[j][0]); pin(fb[j][1]); }
    };
    static_assert(2 * FN + 2 * FM <= 15, "lgkmcnt range");

#pragma unroll
    for (int i = 0; i < NST; ++i)
        if (i < total) { prepare(); issue((uint32_t)i * STAGE_BYTES); }
    if (total >= NST) wait_vmcnt<(NST - 1) * (LPX + LPF)>();
    else wait_vmcnt<0>();
    __syncthreads();
    read_first(abase, bbase, std::integral_constant<int, 0>());
    static_for<FN - 1>([&](auto jc) { read_b(bbase, jc, jc); });
    uint32_t at = 0;                                      // byte offset of the stage's slot
    auto stage = [&](auto morec) __attribute__((always_inline)) {          // a stage that is not the last; `more`: its slot is filled again
        constexpr bool more = decltype(morec)::value;
        step0(at);
        wait_vmcnt<more ? (NST - 2) * (LPX + LPF) : 0>();  // the next stage has landed
        pin_step1();                                      // this wave has read all of this one
        block_barrier();
        if constexpr (more) issue(at);
        at = at == (uint32_t)(NST - 1) * STAGE_BYTES ? 0u : at + STAGE_BYTES;
        const uint32_t a = abase + at, b = bbase + at;
        read_first(a, b, std::integral_constant<int, 0>());
        static_for<FN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            mma(std::integral_constant<int, 1>(), jc);
            if constexpr (j < FN - 1) read_b(b, jc, jc);
        });
    };
    int s = 0;
    for (; s < total - NST; ++s) { prepare(); stage(std::true_type()); }
    for (; s < total - 1; ++s) stage(std::false_type());
    step0(at);
    pin_step1();
    static_for<FN>([&](auto jc) { mma(std::integral_constant<int, 1>(), jc); });
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));    // the products stay in front of the branches of the epilogue

    // 32x32 accumulator layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
    const int ra0 = row_a0 + wm * WTM + 4 * fh;
    if constexpr (PIX_A) {
        const int n0 = p0 / HoWo;
        if (vec_ok > 1 && min(p0 + BP, g.T) <= (n0 + 1) * HoWo) {
            // The planes of y are whole 16-byte pieces and the block lies in one image.  Stored from the accumulators, an instruction
            // touches 32 lines with 16 bytes each; the block goes through the ring's LDS as [channel][pixel] in y's type, 16-byte
            // pieces swizzled by the channel, and leaves as pieces of whole lines (256 channels at 512x512: 178 -> 162 us).  Channel-last
            // the same made no difference.
            constexpr int PIECES = BM / 8;                // 16-byte pieces per channel
            static_assert(BM * BN * 2 <= NST * STAGE_BYTES, "the block fits the ring");
            block_barrier();                              // every wave has read the last stage
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int cl = wn * WTN + j * 32 + frow, k = min(row_b0 + cl, g.K - 1);
                const float bb = (bias ? bias[k] : 0.f) + (post.addvec ? post.addvec[(size_t)n0 * g.K + k] : 0.f);
                const EO* ro = static_cast<const EO*>(post.residual) + ((size_t)n0 * g.K + k) * HoWo + (ra0 - n0 * HoWo);
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int d = i * 32 + 8 * q;
                        float v[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r] * post.scale + bb;
                        if (post.residual && ra0 + d < g.T && row_b0 + cl < g.K) {
                            const uint2 w = *reinterpret_cast<const uint2*>(ro + d);
                            v[0] += lo16<EO>(w.x); v[1] += hi16<EO>(w.x); v[2] += lo16<EO>(w.y); v[3] += hi16<EO>(w.y);
                        }
                        const int piece = (wm * WTM + d) / 8;
                        *reinterpret_cast<uint2*>(lds + (cl * PIECES + (piece ^ (cl & (PIECES - 1)))) * 16 + fh * 8) =
                            make_uint2(pack2<EO>(v[0], v[1]), pack2<EO>(v[2], v[3]));
                    }
            }
            __syncthreads();
            const int piece = tid % PIECES, t = row_a0 + 8 * piece;
            if (t >= g.T) return;                         // no barrier follows
            for (int cl = tid / PIECES; cl < BN && row_b0 + cl < g.K; cl += NW * 64 / PIECES)
                *reinterpret_cast<uint4*>(y + ((size_t)n0 * g.K + row_b0 + cl) * HoWo + (t - n0 * HoWo)) =
                    *reinterpret_cast<const uint4*>(lds + (cl * PIECES + (piece ^ (cl & (PIECES - 1)))) * 16);
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                igemm_store4<EO, PIX_A>(f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]},
                                        ra0 + i * 32 + 8 * q, row_b0 + wn * WTN + j * 32 + frow, y, bias, g, post, vec_ok, planes);
}

template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A, bool RAGGED>
static hipError_t launch_fp8_rag(const uint8_t* xq, const uint8_t* Wq, const float* bias, EO* y, const ConvGeom& g, const IgemmPost& post,
                                 bool planes, hipStream_t s) {
    const int tiles_p = (g.T + BP - 1) / BP, tiles_k = (g.K + BK - 1) / BK;
    const long long total = (long long)tiles_p * tiles_k;
    if (total > 0x3fffffffLL) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    constexpr int lds_bytes = NST * (BP + BK) * 128 + 12 * BP;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    auto kern = conv_igemm_fp8_kernel<EO, BP, BK, WP, WK, PIX_A, RAGGED>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    const uint8_t* zero_row = Wq + (size_t)g.R * g.R * g.K * g.Cp;
    // 2: planes of whole 16-byte pieces
    const int vec_ok = igemm_vec_ok<PIX_A>(g, y, post, planes) ? (g.Ho * g.Wo % 8 == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0 ? 2 : 1) : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(WP * WK * 64), lds_bytes, s, xq, Wq, zero_row, bias, y, g, post, tiles_p, tiles_k,
                       (int)total, per_xcd, vec_ok, planes ? 1 : 0);
    return hipGetLastError();
}

template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A>
static hipError_t launch_fp8_cfg(const uint8_t* xq, const uint8_t* Wq, const float* bias, EO* y, const ConvGeom& g, const IgemmPost& post,
                                 bool planes, hipStream_t s) {
    return g.Cp % 128 == 0 ? launch_fp8_rag<EO, BP, BK, WP, WK, PIX_A, false>(xq, Wq, bias, y, g, post, planes, s)
                           : launch_fp8_rag<EO, BP, BK, WP, WK, PIX_A, true>(xq, Wq, bias, y, g, post, planes, s);
}

// Blocks: 256x256 where there is a round of them and K is a whole number, else 128x128 with two workgroups to a compute unit (a whole
// call, NCHW, us, 128x128 / 256x256: 256 channels at 512x512 239 / 222, 512 at 256x256 172 / 151, but 512 at 128x128 46 / 59, 128 at
// 512x512 86 / 113).
static bool fp8_wide(const ConvGeom& g) { return g.K % 256 == 0 && (long long)((g.T + 255) / 256) * (g.K / 256) >= 256; }

// Whole reductions and two-byte y.  Left to conv_igemm.hip: wide blocks with a channel-last y, where its sixteen waves measured 224 us
// against 232 here (256 channels at 512x512), and images too small to give every compute unit a 128x128 block, where its 64x64 blocks are
// faster; but not with so few output channels that its block is as empty as this one (us, here / there, channel-last: 1x1 64 -> 8 at 76x16
// 6.5 / 8.7, 384 -> 8 at 76x72, N=4, 14.7 / 16.9, 3x3 16 -> 8 at 257x74 14.4 / 17.4, 1x1 48 -> 20 at 61x344 8.2 / 9.5; 112 -> 64 at 48x157
// 10.8 / 9.0, and with 22 channels, stored one by one, 320 -> 22 at 141x120, stride 2, 14.6 / 12.3).
// In NCHW, where outputs leave through LDS here if the images are whole 16-byte pieces, half as many blocks are enough, and with no
// more than a dozen stages and more than 16 channels, or where the last stage of a tap is a partial one, which its kernel fills through
// registers, any number (channel-last 1x1 64 -> 128 at 32x32 11.3 / 8.5, 3x3 256 -> 256 at 64x64 23.7 / 18.1, 640 -> 640 at 64x64 40.9 / 38.3,
// but 256 -> 256 at 128x128 27.9 / 34.5; NCHW 3x3 256 -> 256 at 64x64 20.1 / 18.2, 1280 -> 320 at 64x64 61.2 / 57.7, but 256 -> 256 at 96x96
// 22.0 / 24.5, 64 -> 256 at 64x64 15.7 / 17.4, 320 -> 320 25.5 / 28.0, 1x1 1280 -> 128 15.9 / 16.6; at 15x12 128 -> 1024 11.3 / 9.7; 3x3 128 ->
// 8 at 91x152, stride 2, 16.1 / 14.0).  Everything else is faster here (256 channels at 512x512 270 / 222, 512 at 256x256 187 / 151, 128 at
// 512x512 135 / 86, at 1024x1024 channel-last 456 / 353, 192 -> 320 at 312x200 124 / 73, 64 -> 16 at 118x131, N=8, 63 / 48, there / here).
bool igemm_fp8_tile_ok(const ConvGeom& g, int dt, bool nhwc, int nsplit) {
    if (!two_byte(dt) || nsplit != 1 || (size_t)256 * g.Cp >= ((size_t)1 << 31)) return false;       // 32-bit lane offsets
    const long long blocks = (long long)((g.T + 127) / 128) * ((g.K + 127) / 128), outputs = (long long)g.T * g.K;
    if (blocks >= 256) return !(nhwc && fp8_wide(g));
    if (nhwc) return g.K <= 16 || (g.K <= 32 && g.K % 4 == 0);
    if (g.Ho * g.Wo % 8 != 0) return false;
    return outputs >= 136LL * 128 * 128 || g.Cp % 128 != 0 || (g.K > 16 && g.R * g.R * (g.Cp / 128) <= 12);
}

template <typename EO, bool PIX_A>
static hipError_t launch_fp8_t(const uint8_t* xq, const uint8_t* Wq, const float* bias, EO* y, const ConvGeom& g, const IgemmPost& post,
                               bool planes, hipStream_t s) {
    if constexpr (PIX_A)
        if (fp8_wide(g)) return launch_fp8_cfg<EO, 256, 256, 4, 2, true>(xq, Wq, bias, y, g, post, planes, s);
    return launch_fp8_cfg<EO, 128, 128, 2, 2, PIX_A>(xq, Wq, bias, y, g, post, planes, s);
}

hipError_t launch_igemm_fp8_tile(const void* xq, const void* Wq, const float* bias, void* y, const ConvGeom& g, const IgemmPost& post, int dt,
                                 bool nhwc, hipStream_t s) {
    const bool planes = !nhwc && g.Ho * g.Wo % 2 != 0;
    auto run = [&](auto* tag) {
        using EO = std::remove_pointer_t<decltype(tag)>;
        return nhwc || planes ? launch_fp8_t<EO, false>((const uint8_t*)xq, (const uint8_t*)Wq, bias, (EO*)y, g, post, planes, s)
                              : launch_fp8_t<EO, true>((const uint8_t*)xq, (const uint8_t*)Wq, bias, (EO*)y, g, post, false, s);
    };
    return dt == DT_F16 ? run(static_cast<__half*>(nullptr)) : run(static_cast<bf16_t*>(nullptr));
}

}  // namespace wino

// Implicit-GEMM convolution on 8-bit floating-point operands (E4M3): operands and staging as in conv_igemm.hip (128-byte stages, global
// -> LDS transfers into a ring, XOR-swizzled chunks), 32x32x64 MFMA steps, outputs in a two-byte type.
//
// A stage of 128 reduction elements is two MFMA steps.  The kernel of conv_igemm.hip reads all fragments of a stage behind its barrier
// and multiplies them when the last has arrived; here the fragments of a step are requested one step ahead, across the barrier, and the
// stage after next is requested in the middle of a stage.  The 256x256 block has eight waves of 64x128 instead of sixteen of 64x64: LDS
// feeds a 64x64 piece at exactly the rate at which it is multiplied, and the transfers into LDS come on top; a 64x128 piece needs 3/4
// of that.  256 channels at 512x512, a call that the kernel for 3x3 further down takes now: 208 -> 162 us (1.9 PFLOP/s), four rounds of workgroups of 18 stages.  About 30 us of it are start and
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

struct RowsGeom {
    FastDiv w, h, tiles;                   // divisions by W, H, the shorter tile dimension
    int tiles_k_fast, tiles_short;         // the shorter one is that of the output channels
    int total_blocks, blocks_per_xcd;
};
}  // namespace

// The sums of a block, 32x32 tiles of 64-lane accumulators, scaled, added to and stored; every transfer into LDS has landed.
template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A, int LDS_BYTES, int FM, int FN>
__device__ __forceinline__ void fp8_store(float16_t (&acc)[FM][FN], unsigned char* lds, const float* __restrict__ bias, EO* __restrict__ y,
                                          const ConvGeom& g, const IgemmPost& post, int p0, int k0, int vec_ok, int planes) {
    constexpr int BM = PIX_A ? BP : BK, BN = PIX_A ? BK : BP, WGN = PIX_A ? WK : WP, WTM = FM * 32, WTN = FN * 32, NW = WP * WK;
    const int tid = threadIdx.x, lane = tid & 63, frow = lane & 31, fh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WGN, wn = wave % WGN;
    const int row_a0 = PIX_A ? p0 : k0, row_b0 = PIX_A ? k0 : p0, HoWo = g.Ho * g.Wo;
    // 32x32 accumulator layout: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
    const int ra0 = row_a0 + wm * WTM + 4 * fh;
    if constexpr (PIX_A) {
        const int n0 = p0 / HoWo;
        if (vec_ok > 1 && min(p0 + BP, g.T) <= (n0 + 1) * HoWo) {
            // The planes of y are whole 16-byte pieces and the block lies in one image.  Stored from the accumulators, an instruction
            // touches 32 lines with 16 bytes each; the block goes through the stages' LDS as [channel][pixel] in y's type, 16-byte
            // pieces swizzled by the channel, and leaves as pieces of whole lines (256 channels at 512x512: 178 -> 162 us).  Channel-last
            // the same made no difference.
            constexpr int PIECES = BM / 8;                // 16-byte pieces per channel
            static_assert(BM * BN * 2 <= LDS_BYTES, "the block fits the ring");
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
    fp8_store<EO, BP, BK, WP, WK, PIX_A, NST * STAGE_BYTES>(acc, lds, bias, y, g, post, p0, k0, vec_ok, planes);
}

// 3x3, stride 1: the three taps of a filter row read the same pixels, one place apart.  So the pixels of a row of taps - BP of them and their two
// neighbours, in the order of the image - are fetched once per 128 channels and a lane's fragments of tap s are rows s further on; a tap that
// lies beyond the left or right edge reads a row of zeros instead (rows above and below the image arrive as zeros).  A stage, one tap, then
// moves BK rows of the filter and a third of BP + 8 rows of pixels into LDS instead of BK + BP, and the pixels have three stages to arrive.
// The 256x256 block gains little by that: 256 channels at 512x512, in turn in one run, us with random bytes / with zeros for x (which leave the clock
// higher): the kernel above 162.7 / 146.1, here 161.6 / 148.1, 128x128 blocks 157.2 / 137.9; its products alone would take 62.
template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A, bool RAGGED>
__global__ void __launch_bounds__(WP * WK * 64)
conv_rows_fp8_kernel(const uint8_t* __restrict__ xq, const uint8_t* __restrict__ Wq, const float* __restrict__ bias, EO* __restrict__ y,
                     ConvGeom g, IgemmPost post, RowsGeom q, int vec_ok, int planes) {
    constexpr int RB = 128, CPR = RB / 16;                // stage bytes (= reduction elements) and 16-byte chunks per row
    constexpr int BM = PIX_A ? BP : BK, BN = PIX_A ? BK : BP, WGM = PIX_A ? WP : WK, WGN = PIX_A ? WK : WP, NW = WP * WK;
    constexpr int LPX = BP / 8 / NW, LPF = BK / 8 / NW;   // 1 KB transfers (8 rows) per wave: a row of taps' pixels (and one more), a tap's filter
    constexpr int WTM = BM / WGM, WTN = BN / WGN, FM = WTM / 32, FN = WTN / 32, FPX = PIX_A ? FM : FN;
    constexpr uint32_t PIX_BYTES = (BP + 8) * RB, FIL_BYTES = BK * RB, FIL0 = 2 * PIX_BYTES, ASIDE = FIL0 + 2 * FIL_BYTES, ZERO = ASIDE + 1024;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BP % (8 * NW) == 0 && BK % (8 * NW) == 0 && (8 * NW) % 16 == 0, "tile shape");
    constexpr int XBITS = 3 * LPX + LPF;
    static_assert(XBITS + 3 <= 32, "mask bits");

    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    const int logical = (int)(blockIdx.x % 8) * q.blocks_per_xcd + (int)(blockIdx.x / 8);   // one contiguous range per XCD
    if (logical >= q.total_blocks) return;                // uniform, before any barrier
    const int t_hi = (int)divide((uint32_t)logical, q.tiles), t_lo = logical - t_hi * q.tiles_short;
    const int tk = q.tiles_k_fast ? t_lo : t_hi, tp = q.tiles_k_fast ? t_hi : t_lo;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int p0 = tp * BP, k0 = tk * BK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds, row_bytes = (uint32_t)g.Cp;
    if (tid < 32) *reinterpret_cast<uint32_t*>(lds + ZERO + 4 * tid) = 0u;

    // Transfers: LDS row j of the pixels is pixel p0 - 1 + j, one image row up or down with the row of taps; the descriptor starts one image
    // row and one pixel early.  One lane offset per operand, the rest is scalar; a bit per transfer (and row of taps) says whether the lane's row exists.
    const int lrow = wave * 8 + (lane >> 3);
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ ((lrow >> 1) & (CPR - 1))) * 16);     // 8 * NW rows further on the swizzle is the same
    auto row_bits = [&](int t) __attribute__((always_inline)) {          // rows of taps that lie inside the image for pixel t
        const uint32_t tc = (uint32_t)min(max(t, 0), g.T - 1), line = divide(tc, q.w), oi = line - divide(line, q.h) * (uint32_t)g.H;
        return t >= 0 && t < g.T ? (oi > 0 ? 1u : 0u) | 2u | (oi + 1 < (uint32_t)g.H ? 4u : 0u) : 0u;
    };
    uint32_t live = 0;
#pragma unroll
    for (int i = 0; i < LPX; ++i) live |= row_bits(p0 - 1 + lrow + 8 * NW * i) << (3 * i);
#pragma unroll
    for (int i = 0; i < LPF; ++i) live |= (k0 + lrow + 8 * NW * i < g.K ? 1u : 0u) << (3 * LPX + i);
    const uint32_t poff = (uint32_t)(p0 + lrow) * row_bytes + chunk, foff = (uint32_t)(k0 + lrow) * row_bytes + chunk;
    // the last two pixels, by wave 0 (its lane offset again); the others write zeros aside, so that no branch parts a stage
    live |= (wave == 0 && (lane >> 3) < 2 ? row_bits(p0 - 1 + BP + (lane >> 3)) : 0u) << XBITS;
    const uint32_t xdst = lds0 + (wave == 0 ? (uint32_t)(BP * RB) : ASIDE), xstep = wave == 0 ? PIX_BYTES : 0u;
    const uint32_t line_bytes = (uint32_t)g.W * row_bytes, step8 = (uint32_t)(8 * NW) * row_bytes;
    const rsrc_t xr = make_rsrc(xq - line_bytes - row_bytes), wr = make_rsrc(Wq);
    const uint32_t pdst = lds0 + (uint32_t)wave * 1024u, fdst = lds0 + FIL0 + (uint32_t)wave * 1024u;

    const int nkc = (g.Cp + RB - 1) / RB, groups = 3 * nkc;              // rows of taps over all channel chunks, chunk by chunk
    const uint32_t tail = row_bytes - (uint32_t)(nkc - 1) * RB;          // bytes of a row in the last chunk
    const uint32_t tap_bytes = (uint32_t)g.K * row_bytes;
    uint32_t pr = 0, pkc = 0, ftap = 0, fkc = 0;                         // next row of taps, next tap to fetch
    // lanes of chunk kc that lie inside the operands: none beyond the last, and none of its bytes beyond Cp
    const uint32_t whole = chunk < tail ? ~0u : 0u;
    auto past = [&](uint32_t kc) __attribute__((always_inline)) {
        const uint32_t inner = kc < (uint32_t)(nkc - 1) ? ~0u : 0u, any = kc < (uint32_t)nkc ? ~0u : 0u;
        return RAGGED ? (whole | inner) & any : any;
    };
    auto issue_pixels = [&](uint32_t slot) __attribute__((always_inline)) {
        const uint32_t gone = live & past(pkc);
        uint32_t soff = pr * line_bytes + pkc * RB;
#pragma unroll
        for (int i = 0; i < LPX; ++i) {
            dma_buffer_1k(xr, gone >> (3 * i + pr) & 1u ? poff : kOutside, soff, pdst + slot * PIX_BYTES + (uint32_t)(8 * NW * i) * RB);
            soff += step8;
        }
        dma_buffer_1k(xr, gone >> (XBITS + pr) & 1u ? poff : kOutside, pr * line_bytes + pkc * RB + (uint32_t)BP * row_bytes, xdst + slot * xstep);
        pr = pr == 2 ? 0u : pr + 1; pkc += pr == 0 ? 1u : 0u;
    };
    auto issue_filter = [&](uint32_t slot) __attribute__((always_inline)) {
        const uint32_t gone = live & past(fkc);
        uint32_t soff = ftap * tap_bytes + fkc * RB;
#pragma unroll
        for (int i = 0; i < LPF; ++i) {
            dma_buffer_1k(wr, gone >> (3 * LPX + i) & 1u ? foff : kOutside, soff, fdst + slot * FIL_BYTES + (uint32_t)(8 * NW * i) * RB);
            soff += step8;
        }
        ftap = ftap == 8 ? 0u : ftap + 1; fkc += ftap == 0 ? 1u : 0u;
    };

    float16_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // Fragments as in the kernel above.  Pixel rows: an address per 32-pixel sub-tile, that of the row of zeros where the tap is
    // beyond the edge; filter rows: one address.
    u32x4_t fa[2][FM][2], fb[FN + 1][2];                  // [step][sub-tile][chunk]; fb[FN]: last column of step 1
    const int frow = lane & 31, fh = lane >> 5;
    const int prow = (PIX_A ? wm * WTM : wn * WTN) + frow, krow = (PIX_A ? wn * WTN : wm * WTM) + frow;
    uint32_t edge = 0;                                    // bit 2i: left, 2i + 1: right
#pragma unroll
    for (int i = 0; i < FPX; ++i) {
        const uint32_t t = (uint32_t)min(p0 + prow + 32 * i, g.T - 1), oj = t - divide(t, q.w) * (uint32_t)g.W;
        edge |= (oj == 0 ? 1u : 0u) << (2 * i) | (oj + 1 == (uint32_t)g.W ? 2u : 0u) << (2 * i);
    }
    auto swz = [&](int row) __attribute__((always_inline)) { return (uint32_t)(((2 * fh) ^ ((row >> 1) & (CPR - 1))) << 4); };
    const uint32_t pix_row[3] = {lds0 + (uint32_t)prow * RB + swz(prow), lds0 + (uint32_t)(prow + 1) * RB + swz(prow + 1), lds0 + (uint32_t)(prow + 2) * RB + swz(prow + 2)};
    const uint32_t fil_row = lds0 + FIL0 + (uint32_t)krow * RB + swz(krow), zero_row = lds0 + ZERO;
    uint32_t paddr[FPX], faddr;
    auto locate = [&](auto sc, uint32_t pslot, uint32_t fslot) __attribute__((always_inline)) {         // fragment rows of tap s
        constexpr int s = decltype(sc)::value;
#pragma unroll
        for (int i = 0; i < FPX; ++i) {
            paddr[i] = pix_row[s] + pslot * PIX_BYTES + (uint32_t)(i * 32 * RB);
            if constexpr (s != 1) paddr[i] = edge >> (2 * i + (s >> 1)) & 1u ? zero_row : paddr[i];
        }
        faddr = fil_row + fslot * FIL_BYTES;
    };
    auto read_row = [&](u32x4_t (&f)[2], auto px, auto ic, auto hc) __attribute__((always_inline)) {     // both chunks of a sub-tile, step h
        constexpr int i = decltype(ic)::value, h = decltype(hc)::value;
        if constexpr (decltype(px)::value) {
            const uint32_t a = paddr[i] ^ (uint32_t)(64 * h);
            lds_read16_async<0>(f[0], a);
            lds_read16_async<0>(f[1], a ^ 16u);
        } else {
            const uint32_t a = faddr ^ (uint32_t)(64 * h);
            lds_read16_async<i * 32 * RB>(f[0], a);
            lds_read16_async<i * 32 * RB>(f[1], a ^ 16u);
        }
    };
    using PA = std::integral_constant<bool, PIX_A>;
    using PB = std::integral_constant<bool, !PIX_A>;
    auto read_b = [&](auto hc, auto jc, auto rc) __attribute__((always_inline)) { read_row(fb[decltype(rc)::value], PB(), jc, hc); };
    auto read_first = [&](auto hc) __attribute__((always_inline)) {       // rows and last column of step h
        constexpr int h = decltype(hc)::value;
        static_for<FM>([&](auto ic) { read_row(fa[h][decltype(ic)::value], PA(), ic, hc); });
        read_b(hc, std::integral_constant<int, FN - 1>(), std::integral_constant<int, FN - 1 + h>());
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
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    auto step0 = [&]() __attribute__((always_inline)) {   // of a stage whose fragments have been requested; requests step 1
        lds_wait<2 * (FN - 2)>();
        pin_first(I0());
        read_first(I1());
        static_for<FN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j > 0 && j < FN - 1) lds_wait<2 * (FN - 2 - j) + 2 * FM + 2 + 2 * j>();
            if constexpr (j < FN - 1) { pin(fb[j][0]); pin(fb[j][1]); }
            mma(I0(), jc);
            if constexpr (j < FN - 1) read_b(I1(), jc, jc);
        });
    };
    auto pin_step1 = [&]() __attribute__((always_inline)) {
        lds_wait<0>();
        pin_first(I1());
#pragma unroll
        for (int j = 0; j < FN - 1; ++j) { pin(fb[j][0]); pin(fb[j][1]); }
    };
    static_assert(2 * FN + 2 * FM <= 15, "lgkmcnt range");

    issue_pixels(0);
    issue_filter(0);
    issue_filter(1);
    issue_pixels(1);
    wait_vmcnt<LPF + LPX + 1>();
    __syncthreads();
    uint32_t pslot = 0, fslot = 0;
    locate(I0(), 0, 0);
    read_first(I0());
    static_for<FN - 1>([&](auto jc) { read_b(I0(), jc, jc); });
    // Tap s of a row of taps.  In the middle of it the tap's filter slot, and after the last tap the row's pixel slot, are free and filled with
    // the filter two taps on and the pixels two rows on; beyond the end these are zeros, and the fragments of a stage that does not exist are
    // read from whatever the slots hold: without a condition the stages are one basic block.
    auto stage = [&](auto sc) __attribute__((always_inline)) {
        constexpr int s = decltype(sc)::value;
        step0();
        // the next tap's filter has landed; requested after it are at most the next row's pixels, which have until the second tap
        wait_vmcnt<s == 0 ? LPX + 1 : 0>();
        pin_step1();                                      // this wave has read all of this stage
        block_barrier();
        issue_filter(fslot);
        if constexpr (s == 2) { issue_pixels(pslot); pslot ^= 1u; }
        fslot ^= 1u;
        locate(std::integral_constant<int, s == 2 ? 0 : s + 1>(), pslot, fslot);
        read_first(I0());
        static_for<FN>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            mma(I1(), jc);
            if constexpr (j < FN - 1) read_b(I0(), jc, jc);
        });
    };
#pragma unroll 1
    for (int gr = 0; gr < groups; ++gr) { stage(I0()); stage(I1()); stage(I2()); }
    wait_vmcnt<0>();
    lds_wait<0>();
    pin_first(I0());
#pragma unroll
    for (int j = 0; j < FN - 1; ++j) { pin(fb[j][0]); pin(fb[j][1]); }
    block_barrier();
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));    // the products stay in front of the branches of the epilogue
    fp8_store<EO, BP, BK, WP, WK, PIX_A, (int)ZERO>(acc, lds, bias, y, g, post, p0, k0, vec_ok, planes);
}

// 2: planes of whole 16-byte pieces
template <bool PIX_A, typename EO> static int fp8_vec_ok(const ConvGeom& g, const EO* y, const IgemmPost& post, bool planes) {
    return igemm_vec_ok<PIX_A>(g, y, post, planes) ? (g.Ho * g.Wo % 8 == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0 ? 2 : 1) : 0;
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
    const int vec_ok = fp8_vec_ok<PIX_A>(g, y, post, planes);
    const uint8_t* zero_row = Wq + (size_t)g.R * g.R * g.K * g.Cp;
    auto kern = conv_igemm_fp8_kernel<EO, BP, BK, WP, WK, PIX_A, RAGGED>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
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
// call of 3x3, also of those that the kernel above takes now, NCHW, us, 128x128 / 256x256: 256 channels at 512x512 239 / 222, 512 at 256x256 172 / 151, but 512 at 128x128 46 / 59, 128 at
// 512x512 86 / 113).
static bool fp8_wide(const ConvGeom& g) { return g.K % 256 == 0 && (long long)((g.T + 255) / 256) * (g.K / 256) >= 256; }

// How full the rounds of 256x256 blocks are, one to a compute unit, in 128x128 quarters that are not empty; and the share from which on NCHW images of
// an even number of pixels take them.  Such a round takes as long as 15 / 16 of that of four times as many small blocks, and less in long
// reductions with several columns of blocks or with a partial last chunk of channels (us, 128x128 / 256x256 and how full: 704 -> 512 at 349x144 197 / 185, 0.77,
// 704 -> 768 at 316x128 217 / 190, 0.93, 448 -> 768 at 83x672 204 / 191, 0.85, 448 -> 256 at 224x520 165 / 151, 0.89; but 448 -> 512 at 122x400 122 / 130,
// 0.75, 358 -> 512 at 386x199 226 / 252, 0.78).
static double fp8_round_fill(const ConvGeom& g) {
    const long long small = (long long)((g.T + 127) / 128) * ((g.K + 127) / 128), wide = (long long)((g.T + 255) / 256) * ((g.K + 255) / 256);
    return (double)small / (1024.0 * (double)((wide + 255) / 256));
}
static bool fp8_round_full(const ConvGeom& g) {
    const bool early = fp8_wide(g) && g.Cp > 256 && (g.K >= 512 || g.Cp % 128 != 0);
    return fp8_round_fill(g) >= (!early ? 0.9375 : g.Cp > 512 ? 0.75 : 0.84);
}

// 3x3, stride 1, not upsampled, and blocks of 128x128 for most compute units, or for all of them where outputs leave one by one: channels of a
// channel-last y, or fewer than 96 of an NCHW image of an odd number of pixels.  Lane offsets are 32-bit and a descriptor covers 2 GB: x, with a
// row and a pixel in front of it, and the filter have to fit.  Whole calls, us, other kernels / here: 128 channels at 512x512 86.9 / 75.2 (NCHW), 99.2 /
// 88.1 (channel-last), 320 -> 192 at 200x312 71.2 / 56.3 and 79.9 / 69.3, 192 -> 256 at 160x480 channel-last 99 / 73, 512 -> 320 at 120x72 channel-last
// (204 blocks) 36.9 / 35.2; but 555 -> 126 at 155x58, N=2 (141) 51.3 / 54.8, 172 -> 75 at 125x169 (166) 27.8 / 32.1.  Channel-last, one by one: 256 -> 58 at
// 253x104 (206) 23.3 / 32.4, 47 -> 150 at 76x205 (244) 20.4 / 26.7, 192 -> 222 at 220x60 (208) 29.1 / 33.5, but 192 -> 93 at 82x466 (299) 45.0 /
// 41.2, 320 -> 219 at 182x102 (292) 53.1 / 48.6; NCHW 62 -> 64 at 149x87, N=2 (203) 23.7 / 25.5, but 273 -> 253 at 71x181 (202) 41.3 / 38.0.
// Left to the 256x256 blocks of the kernel above: NCHW, full rounds of them, two columns or more, three whole chunks of channels or more, where the
// pixels of the taps are a small part of what it waits for (us, there / 256x256 here / 128x128 here: 512 -> 512 at 256x256 155 / 157 / 160, at 192x320
// 145 / 146 / 153, 1024 -> 512 at 256x256 278 / 285 / 295, 768 -> 512 at 141x232 112 / 115 / 121, 640 -> 768 at 156x224 158 / 166 / 163; but with one
// column 512 -> 256 at 512x512 358 / 357 / 361, 640 -> 256 at 286x352 194 / 191 / 184, with two chunks 256 -> 256 at 512x512 207 / 201 / 197, with a partial
// chunk 448 -> 768 at 566x72 141 / 133 / 149).  Channel-last, one full round, or two with several columns: those of conv_igemm.hip (256 channels at 256x256
// 59.4 / 60.8, 512 at 192x320 163 / 167, at 256x256 169 / 171; but 640 -> 256 at 512x256 242 / 232, in three rounds 512 at 384x256 248.8 / 248.2).  Over 1196
// calls of 180 blocks and more: 0.876 times the other kernels' time, four calls 1 to 2 % slower than there.
bool igemm_fp8_rows_ok(const ConvGeom& g, int dt, bool nhwc, int nsplit) {
    if (!two_byte(dt) || nsplit != 1 || g.R != 3 || g.st != 1 || g.up) return false;
    const unsigned long long lim = kRange / (unsigned long long)g.Cp;
    if ((unsigned long long)g.N * g.H * g.W + g.W + 512u > lim || 9ull * g.K + 512u > lim) return false;
    const long long blocks = (long long)((g.T + 127) / 128) * ((g.K + 127) / 128);
    const bool planes = !nhwc && g.Ho * g.Wo % 2 != 0, whole = g.Cp % 128 == 0;
    if (blocks < (g.K > 32 && (planes ? g.K <= 96 : nhwc && g.K % 4 != 0) ? 256 : 200)) return false;
    if (nhwc) return !(whole && g.Cp > 128 && fp8_wide(g) && (long long)((g.T + 255) / 256) * (g.K / 256) <= (g.K >= 512 ? 512 : 256) && fp8_round_fill(g) >= 0.88);
    return planes || !(whole && g.K >= 512 && g.Cp > 256 && fp8_wide(g) && fp8_round_full(g));
}

template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A, bool RAGGED>
static hipError_t launch_rows_cfg(const uint8_t* xq, const uint8_t* Wq, const float* bias, EO* y, const ConvGeom& g, const IgemmPost& post,
                                  bool planes, hipStream_t s) {
    const int tiles_p = (g.T + BP - 1) / BP, tiles_k = (g.K + BK - 1) / BK;
    const long long total = (long long)tiles_p * tiles_k;
    if (total > 0x3fffffffLL) return hipErrorInvalidValue;
    constexpr int lds_bytes = 2 * (BP + 8 + BK) * 128 + 1024 + 128;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    RowsGeom q;
    q.tiles_k_fast = tiles_k <= tiles_p;
    q.tiles_short = q.tiles_k_fast ? tiles_k : tiles_p;
    q.w = fast_div((uint32_t)g.W); q.h = fast_div((uint32_t)g.H); q.tiles = fast_div((uint32_t)q.tiles_short);
    q.total_blocks = (int)total; q.blocks_per_xcd = (int)((total + 7) / 8);
    auto kern = conv_rows_fp8_kernel<EO, BP, BK, WP, WK, PIX_A, RAGGED>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3((unsigned)(q.blocks_per_xcd * 8)), dim3(WP * WK * 64), lds_bytes, s, xq, Wq, bias, y, g, post, q,
                       fp8_vec_ok<PIX_A>(g, y, post, planes), planes ? 1 : 0);
    return hipGetLastError();
}

// NCHW: 256x256 instead of 128x128, one workgroup to a unit instead of two, where their rounds are full (us, 128x128 / 256x256: 448 -> 192 at 224x576 176 / 158,
// 320 -> 192 at 200x312 61.3 / 56.3, 448 -> 768 at 566x72 149 / 133; but 448 -> 256 at 512x400 275 / 296, 512 channels at 128x128 45 / 65), with at least
// two chunks of channels.
bool igemm_fp8_rows_wide(const ConvGeom& g) { return g.Cp > 128 && fp8_round_full(g); }

template <typename EO, int BP, int BK, int WP, int WK, bool PIX_A>
static hipError_t launch_rows_t(const uint8_t* xq, const uint8_t* Wq, const float* bias, EO* y, const ConvGeom& g, const IgemmPost& post,
                                bool planes, hipStream_t s) {
    return g.Cp % 128 == 0 ? launch_rows_cfg<EO, BP, BK, WP, WK, PIX_A, false>(xq, Wq, bias, y, g, post, planes, s)
                           : launch_rows_cfg<EO, BP, BK, WP, WK, PIX_A, true>(xq, Wq, bias, y, g, post, planes, s);
}

hipError_t launch_igemm_fp8_rows(const void* xq, const void* Wq, const float* bias, void* y, const ConvGeom& g, const IgemmPost& post, int dt,
                                 bool nhwc, hipStream_t s) {
    const bool planes = !nhwc && g.Ho * g.Wo % 2 != 0;
    auto run = [&](auto* tag) {
        using EO = std::remove_pointer_t<decltype(tag)>;
        const uint8_t *x8 = (const uint8_t*)xq, *w8 = (const uint8_t*)Wq;
        if (nhwc || planes) return launch_rows_t<EO, 128, 128, 2, 2, false>(x8, w8, bias, (EO*)y, g, post, planes, s);
        return igemm_fp8_rows_wide(g) ? launch_rows_t<EO, 256, 256, 4, 2, true>(x8, w8, bias, (EO*)y, g, post, false, s)
                                : launch_rows_t<EO, 128, 128, 2, 2, true>(x8, w8, bias, (EO*)y, g, post, false, s);
    };
    return dt == DT_F16 ? run(static_cast<__half*>(nullptr)) : run(static_cast<bf16_t*>(nullptr));
}

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
// 8 at 91x152, stride 2, 16.1 / 14.0).  Everything else is faster here (measured on 3x3 calls, most of which igemm_fp8_rows_ok takes first now: 256 channels at 512x512 270 / 222, 512 at 256x256 187 / 151, 128 at
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

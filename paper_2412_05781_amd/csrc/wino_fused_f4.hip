// Steps (ii) and (iii) in one kernel for F(4x4,3x3) (Section "Techniques"; its second paragraph argues for keeping
// dependent steps local).  As in the F(2x2) kernel of wino_fused.hip, a workgroup owns a block of (output channels x
// tiles) for ALL 36 positions and walks them one after another, so the product M is never stored.  What differs is the
// bookkeeping of step (iii): an output tile has 16 values per (channel, tile), and with the product and the running sums
// a 32x32 MFMA sub-tile per wave would need more vector registers than exist.  So
//   - a wave owns a 16 x 32 piece (two 16x16 MFMA tiles, v_mfma_f32_16x16x32: four accumulator registers per tile), and
//   - step (iii) is taken one dimension at a time.  Positions run xi-major; while nu runs over a row of the
//     transformed tile the product is folded into four row sums  Z[b] += A^T[b][nu] * M[xi,nu]; at the end of the row
//     Y[a][b] += A^T[a][xi] * Z[b].  That is 21 accumulator sets of 8 registers (16 outputs, 4 row sums, the product), all in vector
//     registers, and 180 multiply-adds per accumulator register instead of 324.  They are not hidden: without them 128 channels at 1024x1024
//     take 413 us instead of 457 (a second set for the product, added in front of each, 8 more).
// The price of the small wave tile is traffic: 3 KB of LDS fragments per 32 reduction elements and wave, and a block of
// at most 64 x 64 per compute unit (the register file holds no more accumulators of this kind), so every byte of U and V is
// fetched into LDS by T/64 and K/64 workgroups.  That fill traffic bounds the kernel; it pays on large images with at
// most 256 channels, where the unfused path is bound by writing and re-reading M.  Two-byte storage types only.
//
// Operand staging is that of the batched GEMM kernel: 128-byte stages per row, global -> LDS directly into a ring,
// XOR-swizzled 16-byte chunks, explicit vmcnt waits; one barrier per pair of stages.
// ROWS_K = true : rows of the block are output channels (U), columns are tiles (V); y is NCHW.
// ROWS_K = false: operands swapped, rows are tiles, columns output channels; y is channel-last.
#include "wino_internal.h"
#include "wino_mma.h"

namespace wino {

namespace {

// A^T of F(4x4,3x3): rows (1 1 1 1 1 0), (0 1 -1 2 -2 0), (0 1 1 4 4 0), (0 1 -1 8 -8 1); both arguments wave-uniform
__device__ __forceinline__ float at4(int a, int x) {
    if (x == 0) return a == 0 ? 1.f : 0.f;
    if (x == 5) return a == 3 ? 1.f : 0.f;
    const float sign = (x & 1) ? 1.f : -1.f, mag = x <= 2 ? 1.f : 2.f;
    return a == 0 ? 1.f : (a == 1 ? sign * mag : (a == 2 ? mag * mag : sign * mag * mag * mag));
}

struct Fused4Geom { int N, K, H, W, th, tw, T; FastDiv dth, dtw; };

__device__ const uint4 zero_chunk = {0u, 0u, 0u, 0u};     // source of the chunks beyond Cp

}  // namespace

// Block = (WGM * 16) rows x (WGN * 32) columns, one 16 x 32 piece per wave.
// RAGGED = true: Cp is not a multiple of the stage (64 elements); the chunks beyond Cp of the last stage of every position are zeros.
template <typename E, int NST, int WGM, int WGN, bool ROWS_K, bool RAGGED>
__global__ void __launch_bounds__(WGM * WGN * 64)
wino_fused_f4_kernel(const E* __restrict__ Aop, const E* __restrict__ Bop, const float* __restrict__ bias, E* __restrict__ y,
                     int rowsA, int rowsB, int Cp, Fused4Geom g, int tiles_m, int tiles_n, int total_blocks, int blocks_per_xcd,
                     int vec_ok, PostOp post) {
    static_assert(sizeof(E) == 2, "two-byte storage types");
    constexpr int A2 = 36;                                // positions of F(4x4,3x3)
    constexpr int RB = 128;                               // stage bytes per row
    constexpr int CPR = RB / 16;                          // 16-byte chunks per row per stage
    constexpr int BKE = RB / 2;                           // reduction elements per stage
    constexpr int BM = WGM * 16, BN = WGN * 32;
    constexpr int ROWS = BM + BN;
    constexpr int RPL = 1024 / RB;                        // rows covered by one wave-wide load
    constexpr int NW = WGM * WGN;
    constexpr int LPW = ROWS / RPL / NW;                  // wave-wide loads per wave per stage
    constexpr int LA = BM / (RPL * NW);                   // ... of which from the row operand
    constexpr int STAGE_BYTES = ROWS * RB;
    static_assert(ROWS % (RPL * NW) == 0 && BM % (RPL * NW) == 0, "load i of every wave lies in the same operand");
    static_assert(NST >= 4 && NST % 2 == 0 && LPW * (NST - 1) < 64, "ring depth: pairs of stages, within the vmcnt range");

    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

    // one contiguous range of logical blocks per XCD; the shorter tile dimension runs fastest
    const int bid = blockIdx.x;
    const int logical = (bid % 8) * blocks_per_xcd + bid / 8;
    if (logical >= total_blocks) return;                  // uniform per workgroup, before any barrier
    int tm, tn;
    if (tiles_m <= tiles_n) { tm = logical % tiles_m; tn = logical / tiles_m; }
    else { tn = logical % tiles_n; tm = logical / tiles_n; }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int row0 = tm * BM, col0 = tn * BN;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds;          // LDS byte address of the ring

    // Global side: one scalar base per operand that walks stage by stage through all positions, plus a fixed 32-bit byte
    // offset per lane and load (row inside the block, clamped to the last valid row, and the swizzled chunk).
    const size_t row_bytes = (size_t)Cp * sizeof(E);
    const int lrow = lane / CPR, lchunk = lane % CPR;
    uint32_t goff[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int row = (wave + NW * i) * RPL + lrow;       // row inside the stage, row-operand rows first
        const int chunk = lchunk ^ ((row >> 1) & (CPR - 1));
        int r;
        if (i < LA) { r = row0 + row; r = (r < rowsA ? r : rowsA - 1) - row0; }
        else { r = col0 + (row - BM); r = (r < rowsB ? r : rowsB - 1) - col0; }
        goff[i] = (uint32_t)r * (uint32_t)row_bytes + (uint32_t)chunk * 16u;
    }
    const unsigned char* sA = reinterpret_cast<const unsigned char*>(Aop) + (size_t)row0 * row_bytes;
    const unsigned char* sB = reinterpret_cast<const unsigned char*>(Bop) + (size_t)col0 * row_bytes;
    const size_t planeA = (size_t)rowsA * row_bytes, planeB = (size_t)rowsB * row_bytes;

    const int nk = (Cp + BKE - 1) / BKE;
    const int total = A2 * nk;
    const uint32_t wave_dst = lds0 + (uint32_t)wave * 1024u;

    int issue_kt = 0;
    auto issue_stage = [&](int slot) __attribute__((always_inline)) {                    // the next stage in order, into ring slot `slot`
        const uint32_t dst = wave_dst + (uint32_t)slot * STAGE_BYTES;
        if (RAGGED && issue_kt == nk - 1) {               // chunks beyond Cp come from the line of zeros
            const unsigned char* zero = reinterpret_cast<const unsigned char*>(&zero_chunk);
#pragma unroll
            for (int i = 0; i < LPW; ++i) {
                const int row = (wave + NW * i) * RPL + lrow;
                const int chunk = lchunk ^ ((row >> 1) & (CPR - 1));
                const bool past = (size_t)issue_kt * RB + (size_t)chunk * 16 >= row_bytes;
                dma_load_1k_v(past ? zero : (i < LA ? sA : sB) + goff[i], dst + (uint32_t)(NW * i) * 1024u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < LPW; ++i) dma_load_1k_s(i < LA ? sA : sB, goff[i], dst + (uint32_t)(NW * i) * 1024u);
        }
        if (++issue_kt == nk) {
            issue_kt = 0;
            sA += planeA - (size_t)(nk - 1) * RB;
            sB += planeB - (size_t)(nk - 1) * RB;
        } else {
            sA += RB;
            sB += RB;
        }
    };

    // accumulators of the wave's two 16x16 tiles: the product of the current position, the four row sums, the 16 outputs
    f32x4_t accM[2], accZ[4][2], accY[4][4][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        accM[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            accZ[b][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int a = 0; a < 4; ++a) accY[a][b][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    }

    // A stage holds two MFMA steps of 32 reduction elements (four 16-byte chunks each; lanes 16q..16q+15 hold chunk q of the
    // step).  All six fragments of a stage (one row tile and two column tiles per step) are requested as soon as the stage is
    // visible and used one stage later, so that a whole stage of MFMAs and the next barrier lie between request and use; two
    // fragment sets alternate.  The swizzled chunk of step h is chunk(0) ^ 4h, i.e. the byte address of step 0 with bit 6
    // flipped; the second column tile lies 16 rows further on (same swizzle).
    u32x4_t fa[2][2], fb[2][2][2];                        // [set][step], [set][step][column tile]
    const int frag_row = lane & 15, frag_q = lane >> 4;
    const int rowA = wm * 16 + frag_row, rowB = BM + wn * 32 + frag_row;
    const uint32_t fbaseA = lds0 + (uint32_t)rowA * RB + (uint32_t)((frag_q ^ ((rowA >> 1) & (CPR - 1))) << 4);
    const uint32_t fbaseB = lds0 + (uint32_t)rowB * RB + (uint32_t)((frag_q ^ ((rowB >> 1) & (CPR - 1))) << 4);
    auto read_stage = [&](int slot, auto setc) __attribute__((always_inline)) {
        constexpr int set = decltype(setc)::value;
        const uint32_t a0 = fbaseA + (uint32_t)slot * STAGE_BYTES, b0 = fbaseB + (uint32_t)slot * STAGE_BYTES;
        lds_read16_async<0>(fa[set][0], a0);
        lds_read16_async<0>(fb[set][0][0], b0);
        lds_read16_async<16 * RB>(fb[set][0][1], b0);
        lds_read16_async<0>(fa[set][1], a0 ^ 64u);
        lds_read16_async<0>(fb[set][1][0], b0 ^ 64u);
        lds_read16_async<16 * RB>(fb[set][1][1], b0 ^ 64u);
    };
    // every fragment read but the `newer` youngest has arrived
    auto await_stage = [&](auto setc, auto newerc) __attribute__((always_inline)) {
        constexpr int set = decltype(setc)::value;
        lds_wait<decltype(newerc)::value>();
#pragma unroll
        for (int h = 0; h < 2; ++h) { pin(fa[set][h]); pin(fb[set][h][0]); pin(fb[set][h][1]); }
    };
    auto mma_stage = [&](auto setc) __attribute__((always_inline)) {
        constexpr int set = decltype(setc)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            Mma16<E>::run(fa[set][h], fb[set][h][0], accM[0]);
            Mma16<E>::run(fa[set][h], fb[set][h][1], accM[1]);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

#pragma unroll
    for (int s = 0; s < NST; ++s)
        if (s < total) issue_stage(s);
    if (NST - 2 >= total) wait_vmcnt<0>();
    else wait_vmcnt<(NST - 2) * LPW>();                    // the first pair has landed
    __syncthreads();
    read_stage(0, I0());

    int kt = 0, xi = 0, nu = 0;
    // after the last MFMA of a stage: at the end of a position the product is folded into the row sums and cleared; at the
    // end of a row of the transformed tile the row sums are folded into the outputs and cleared
    auto end_of_stage = [&]() __attribute__((always_inline)) {
        if (++kt < nk) return;
        kt = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const float c = at4(b, nu);                   // wave-uniform
            if (c != 0.f) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) accZ[b][j][r] = fmaf(c, accM[j][r], accZ[b][j][r]);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) accM[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (++nu < 6) return;
        nu = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float c = at4(a, xi);
            if (c != 0.f) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) accY[a][b][j][r] = fmaf(c, accZ[b][j][r], accY[a][b][j][r]);
            }
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int j = 0; j < 2; ++j) accZ[b][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        ++xi;
    };

    // Stages are taken in pairs (36 * nk is even), one barrier per pair: on entry the pair is visible and the fragments of its first stage
    // have been requested.  The transfers bound the kernel, so this gains little over a barrier per stage and half the ring (whole calls:
    // 256 channels at 512x512 334 -> 327 us, 512 at 256x256 channel-last 238 -> 236, 128 at 1024x1024 channel-last 494 -> 491).  Blocks
    // of 32 tiles x 128 channels, which fetch V half as often and U twice, are slower (349, 268 and 530).  The figures are of the 64x64
    // block, one workgroup to a compute unit with either ring; for the 32x64 block see launch_fused4_t.
    const int pairs = total / 2;
    auto first_half = [&](int slot) __attribute__((always_inline)) {
        read_stage(slot + 1, I1());
        await_stage(I0(), std::integral_constant<int, 6>());
        __builtin_amdgcn_sched_barrier(0);
        mma_stage(I0());
        __builtin_amdgcn_sched_barrier(0);
        end_of_stage();
    };
    int slot = 0;
    for (int p = 0; p < pairs - 1; ++p) {
        const int next = slot + 2 == NST ? 0 : slot + 2;
        first_half(slot);
        // the next pair has landed once no more transfers are outstanding than were issued after it
        if (p + NST / 2 >= pairs) wait_vmcnt<0>();
        else wait_vmcnt<(NST - 4) * LPW>();
        await_stage(I1(), I0());        // this wave has read all of the pair
        __syncthreads();                // the next pair visible to all waves; every wave has read all of this one
        if (p + NST / 2 < pairs) { issue_stage(slot); issue_stage(slot + 1); }
        read_stage(next, I0());
        __builtin_amdgcn_sched_barrier(0);
        mma_stage(I1());
        __builtin_amdgcn_sched_barrier(0);
        end_of_stage();
        slot = next;
    }
    first_half(slot);
    await_stage(I1(), I0());
    mma_stage(I1());
    end_of_stage();

    // ---- epilogue: bias (+ vector, + residual), crop, round once, store ---------------------------------------
    // 16x16 accumulator layout: register r of lane l holds row 4*(l/16) + r, column l%16 of the tile
    const int H = g.H, W = g.W, K = g.K;
    const E* res = static_cast<const E*>(post.residual);
    // tile t (clamped): image, first output row and column
    auto locate = [&](int t, int& n, int& i0, int& j0) __attribute__((always_inline)) {
        const uint32_t tc = (uint32_t)min(t, g.T - 1), q = divide(tc, g.dtw);
        n = (int)divide(q, g.dth);
        j0 = 4 * (int)(tc - q * (uint32_t)g.tw);
        i0 = 4 * ((int)q - n * g.th);
    };
    if constexpr (ROWS_K) {
        // columns are tiles: a lane owns one tile per column tile, its four registers run over output channels; the four
        // pixels of an output row of the tile are stored together, neighbouring lanes hold neighbouring tiles of a tile row
        const int k0 = row0 + wm * 16 + 4 * frag_q;
        float bk[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) bk[r] = bias ? bias[min(k0 + r, K - 1)] : 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = col0 + wn * 32 + j * 16 + frag_row;
            int n, i0, j0;
            locate(t, n, i0, j0);
            float bb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) bb[r] = bk[r] + (post.addvec ? post.addvec[(size_t)n * K + min(k0 + r, K - 1)] : 0.f);
            if (t >= g.T) continue;
            const size_t off = (((size_t)n * K + k0) * H + i0) * W + j0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (k0 + r >= K) continue;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    if (i0 + a >= H) continue;
                    const size_t o = off + ((size_t)r * H + a) * W;
                    float v[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) v[b] = accY[a][b][j][r] + bb[r];
                    if (vec_ok) {
                        if (res) {
                            const uint2 rr = *reinterpret_cast<const uint2*>(res + o);
                            v[0] += lo16<E>(rr.x); v[1] += hi16<E>(rr.x); v[2] += lo16<E>(rr.y); v[3] += hi16<E>(rr.y);
                        }
                        *reinterpret_cast<uint2*>(y + o) = make_uint2(pack2<E>(v[0], v[1]), pack2<E>(v[2], v[3]));
                    } else {
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            if (j0 + b < W) y[o + b] = from_f32<E>(v[b] + (res ? to_f32<E>(res[o + b]) : 0.f));
                    }
                }
            }
        }
    } else {
        // Columns are output channels, which are contiguous in a channel-last y - but a lane holds one channel and a 16x16
        // tile only 16 of them, so stores straight from the accumulators would be 32-byte pieces.  The block goes through LDS
        // instead (the ring is free by now): for each output row a of the tile, every wave parks its sums for the four pixels
        // (a, b) at [b][tile][channel], and a thread then takes eight channels of one tile, always the same, finds its place in y once, adds
        // bias, vector and residual before the one rounding, as everywhere, and writes 16-byte pieces, eight lanes to a 128-byte line.  (With
        // the tile's place found for every value parked and every piece stored, the end of a block took 15 us, and a sixth of that now:
        // 128 channels at 1024x1024, eight rounds of blocks, 488 -> 457 us a call.)
        constexpr int PSTRIDE = BN * 4 + 16;              // bytes per (pixel, tile) row in LDS; the pad spreads the rows over the banks
        constexpr int PIECES = BN / 8;                    // pieces of eight channels per row
        static_assert(4 * BM * PSTRIDE <= NST * STAGE_BYTES, "the parked rows fit the ring's LDS");
        static_assert(BM * PIECES == NW * 64, "a thread keeps its tile and piece");
        const int piece = tid % PIECES, tl = tid / PIECES, t = row0 + tl, k0 = col0 + piece * 8;
        int n, i0, j0;
        locate(t, n, i0, j0);
        float bb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = min(k0 + e, K - 1);
            bb[e] = (bias ? bias[k] : 0.f) + (post.addvec ? post.addvec[(size_t)n * K + k] : 0.f);
        }
        const bool whole = K % 8 == 0 && k0 + 8 <= K;     // a pixel's channel vector starts on a 16-byte boundary
        const size_t base = (((size_t)n * H + i0) * W + j0) * K + k0;
        unsigned char* park = lds + (size_t)(wm * 16 + 4 * frag_q) * PSTRIDE + (size_t)(wn * 32 + frag_row) * 4;
        const unsigned char* take = lds + (size_t)tl * PSTRIDE + (size_t)piece * 32;
#pragma unroll
        for (int a = 0; a < 4; ++a) {                     // unrolled: the accumulators are registers, a must be a constant
            __syncthreads();                              // nobody reads the ring (or the previous rows) any more
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<float*>(park + (b * BM + r) * PSTRIDE + j * 64) = accY[a][b][j][r];
            __syncthreads();
            if (t >= g.T || k0 >= K || i0 + a >= H) continue;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (j0 + b >= W) continue;
                const size_t o = base + ((size_t)a * W + b) * K;
                const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(take + b * BM * PSTRIDE), hi = *reinterpret_cast<const f32x4_t*>(take + b * BM * PSTRIDE + 16);
                float v[8] = {lo[0] + bb[0], lo[1] + bb[1], lo[2] + bb[2], lo[3] + bb[3], hi[0] + bb[4], hi[1] + bb[5], hi[2] + bb[6], hi[3] + bb[7]};
                if (whole) {
                    if (res) {
                        const uint4 w = *reinterpret_cast<const uint4*>(res + o);
                        v[0] += lo16<E>(w.x); v[1] += hi16<E>(w.x); v[2] += lo16<E>(w.y); v[3] += hi16<E>(w.y);
                        v[4] += lo16<E>(w.z); v[5] += hi16<E>(w.z); v[6] += lo16<E>(w.w); v[7] += hi16<E>(w.w);
                    }
                    *reinterpret_cast<uint4*>(y + o) = make_uint4(pack2<E>(v[0], v[1]), pack2<E>(v[2], v[3]), pack2<E>(v[4], v[5]), pack2<E>(v[6], v[7]));
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (k0 + e < K) y[o + e] = from_f32<E>(v[e] + (res ? to_f32<E>(res[o + e]) : 0.f));
                }
            }
        }
    }
}

template <typename E, int NST, int WGM, int WGN, bool ROWS_K, bool RAGGED = false>
static hipError_t launch_fused4_cfg(const void* Aop, const void* Bop, int rowsA, int rowsB, const float* bias, void* y,
                                    const Geom& g, const PostOp& post, hipStream_t s) {
    constexpr int BM = WGM * 16, BN = WGN * 32;
    const int tiles_m = (rowsA + BM - 1) / BM, tiles_n = (rowsB + BN - 1) / BN;
    const long long total = (long long)tiles_m * tiles_n;
    if (total > 0x3fffffffLL) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    constexpr int lds_bytes = (BM + BN) * 128 * NST;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    // lane offsets are 32-bit: a block's rows must span less than 2 GB
    if ((size_t)g.Cp * sizeof(E) * (size_t)(BM > BN ? BM : BN) >= ((size_t)1 << 31)) return hipErrorInvalidValue;
    auto kern = wino_fused_f4_kernel<E, NST, WGM, WGN, ROWS_K, RAGGED>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    Fused4Geom fg{g.N, g.K, g.H, g.W, g.th, g.tw, g.T, fast_div((uint32_t)g.th), fast_div((uint32_t)g.tw)};
    // four-pixel stores of a tile's output row need W % 4 == 0 (the group then never straddles the row end) and 8-byte alignment
    const int vec_ok = (g.W % 4 == 0) && ((reinterpret_cast<uintptr_t>(y) & 7u) == 0) && ((reinterpret_cast<uintptr_t>(post.residual) & 7u) == 0);
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(WGM * WGN * 64), lds_bytes, s,
                       (const E*)Aop, (const E*)Bop, bias, (E*)y, rowsA, rowsB, g.Cp, fg, tiles_m, tiles_n, (int)total, per_xcd, vec_ok, post);
    return hipGetLastError();
}

// Block shapes on offer (rows x columns of the block): 0 = 64x64 with eight waves (4 x 2), 1 = 32x64 with four waves (2 x 2).
int fused4_pick_shape(int rows, int cols) {
    const long long big = (long long)((rows + 63) / 64) * ((cols + 63) / 64);
    return big >= 200 ? 0 : 1;
}

// The ring of the 32x64 block has six slots, 72 KB, because two workgroups then share a compute unit; with eight only one fits, with four
// the next pair is waited for as soon as it is requested.  Whole calls, us, four / six / eight slots: 352 channels at 160x160 (N=4) 336 /
// 323 / 453, 96 -> 128 at 512x512 131 / 128 / 199, 64 -> 896 at 49x234 48 / 48 / 76, 512 -> 256 at 64x64 97 / 89 / 89.
// The chunks beyond Cp come by the same transfers as the rest, from a line of zeros: filled in through registers, the stage waits for
// every transfer in front of it (352 channels 390 us instead of 323, 96 -> 128 159 instead of 128).
template <typename E, bool ROWS_K>
static hipError_t launch_fused4_t(const void* Aop, const void* Bop, int rowsA, int rowsB, const float* bias, void* y,
                                  const Geom& g, const PostOp& post, int shape, hipStream_t s) {
    if (g.Cp % 64 != 0)       // a reduction length that is not a whole number of stages
        return launch_fused4_cfg<E, 6, 2, 2, ROWS_K, true>(Aop, Bop, rowsA, rowsB, bias, y, g, post, s);
    switch (shape) {
        case 0: return launch_fused4_cfg<E, 8, 4, 2, ROWS_K>(Aop, Bop, rowsA, rowsB, bias, y, g, post, s);
        case 1: return launch_fused4_cfg<E, 6, 2, 2, ROWS_K>(Aop, Bop, rowsA, rowsB, bias, y, g, post, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fused4_gemm_output(const void* U, const void* V, const float* bias, void* y, const Geom& g, int dt, bool nhwc,
                                     const PostOp* postp, int shape, hipStream_t s) {
    if (g.m != 4 || !two_byte(dt) || dt == DT_I8) return hipErrorInvalidValue;
    if (shape < -1 || shape > 1) return hipErrorInvalidValue;
    const PostOp post = postp ? *postp : PostOp();
    auto run = [&](auto* tag) {
        using E = std::remove_pointer_t<decltype(tag)>;
        if (nhwc) return launch_fused4_t<E, false>(V, U, g.T, g.K, bias, y, g, post, shape < 0 ? fused4_pick_shape(g.T, g.K) : shape, s);
        return launch_fused4_t<E, true>(U, V, g.K, g.T, bias, y, g, post, shape < 0 ? fused4_pick_shape(g.K, g.T) : shape, s);
    };
    return dt == DT_F16 ? run(static_cast<__half*>(nullptr)) : run(static_cast<bf16_t*>(nullptr));
}

}  // namespace wino

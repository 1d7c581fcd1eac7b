// All three steps in one kernel for F(4x4,3x3) with few input channels and fp32 storage (Section "Techniques"): the first
// convolution of the UNet (4 -> 320 channels).  With a reduction of 4...16 the three-kernel chain is three launches around
// next to no arithmetic: it writes and re-reads V and M (4 and 9 bytes per byte of y) and every launch costs its 2-3 us.
//
// A workgroup owns 16 tiles x 16 output channels.  Three of its waves take two rows of the transformed tile each, 0 and 5, 1 and 2, 3 and 4: twelve
// positions.  The reduction is taken eight channels at a time, as two steps of v_mfma_f32_16x16x4_f32: lane (i = l % 16, q = l / 16) holds
// channels c0 + 2q and c0 + 2q + 1 of row i, in both operands (which channel sits in which step does not matter as long as both agree).
// So a lane transforms the windows of its own tile's two channels and the result is its operand of 24 MFMAs: V exists only in
// registers.  Step (iii) along nu is lane-local; the row sums go through LDS and wave a makes row a of the output tiles.  The activation
// transform is repeated by the K/16 workgroups of a tile group: at eight channels that is 100 vector instructions a wave, less than the
// launch it replaces.
// Loads that put 64 lanes on 64 places cost 64 clocks each however few bytes they fetch.  So a lane loads only the four columns its tile owns,
// one 16-byte load per row in NCHW, and takes the two border columns from its neighbours' registers; the four waves share the
// window's rows through LDS, and the filter block comes in as 1 KB transfers.
// Bound by latency on small images - the chain from load to store, 320 workgroups on 256 units for 4 -> 320 at 64x64 - and by writing y and the
// number of workgroups that a unit holds on large ones: four, by registers (128, which is why the channels are transformed one after the other) and by LDS;
// with three, calls of more than three and up to four to a unit took a second round (us: 16 -> 448 at 41x208 19.7 -> 14.7, 4 -> 160 at 66x360 13.0 -> 10.2, 4 -> 560
// at 282x9, N=2, channel-last 15.5 -> 12.5).  One wave for all 36 positions had 1100 instructions and 72 MFMAs in a row (us, NCHW / channel-last, before -> now: 4 -> 320 at
// 64x64 9.6 / 11.4 -> 7.3 / 9.3, N=2 at 128x128 27.6 / 40.6 -> 21.4 / 29.3, at 47x91 18.2 / 11.5 -> 10.8 / 9.4, 16 -> 320 at 64x64 13.2 / 16.7 -> 10.0 / 13.6).
#include "wino_internal.h"
#include "wino_mma.h"
#include "wino_transforms.h"

namespace wino {

namespace {

struct FewcGeom { int N, C, H, W, K, Cp, th, tw, T; };

// value of the lane before / after this one inside its group of 16 (the first / last lane keeps `edge`)
__device__ __forceinline__ uint32_t from_left(uint32_t edge, uint32_t v) { return __builtin_amdgcn_update_dpp(edge, v, 0x111, 0xf, 0xf, false); }
__device__ __forceinline__ uint32_t from_right(uint32_t edge, uint32_t v) { return __builtin_amdgcn_update_dpp(edge, v, 0x101, 0xf, 0xf, false); }

}  // namespace

// NHWC: x and y channel-last.  ROWVEC: x NCHW, not upsampled, rows of whole 16-byte pieces: the four owned columns are one load.
template <bool NHWC, bool ROWVEC>
__global__ void __launch_bounds__(256, 4)
wino_fewc_f4_kernel(const float* __restrict__ x, const float* __restrict__ U, const float* __restrict__ bias, float* __restrict__ y,
                    FewcGeom g, int tiles_t, int vec_ok, int up, PostOp post) {
    // of each wave: the filter block of a chunk, [position][channel][8], and in its place the row sums, [row][b][lane]
    __shared__ __attribute__((aligned(1024))) f32x4_t part[3][2 * 4 * 64];
    __shared__ uint4 xs[2][6][64];                                          // windows, [channel][row][lane]: the four owned columns
    __shared__ uint32_t es[2][6][64];                                       // ... and the border column of the outer lanes
    static_assert(4 * (sizeof(part) + sizeof(xs) + sizeof(es)) <= 160 * 1024, "four workgroups to a unit");
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int kb = (int)(blockIdx.x / (unsigned)tiles_t) * 16, tb = (int)(blockIdx.x % (unsigned)tiles_t) * 16;
    const int H = g.H, W = g.W, Hs = H >> up, Ws = W >> up;

    // this lane's tile (clamped to the last one; its results are then never stored)
    const int t = min(tb + i, g.T - 1);
    const int tj = t % g.tw, tq = t / g.tw, ti = tq % g.th, n = tq / g.th;

    // the wave's rows of the transformed tile: 0 and 5, 1 and 2, 3 and 4; the fourth wave only helps to load
    const int xi0 = wave == 0 ? 0 : 2 * wave - 1, xi1 = wave == 0 ? 5 : 2 * wave;
    // filter transfers: 32 lanes per position, two 16-byte halves per row of eight channels; rows beyond K repeat the last one
    const uint32_t plane = (uint32_t)g.K * (uint32_t)g.Cp * 4u;
    const uint32_t uoff = (uint32_t)(lane >> 5) * plane + (uint32_t)(min(kb + ((lane & 31) >> 1), g.K - 1) - kb) * (uint32_t)g.Cp * 4u + (uint32_t)(lane & 1) * 16u;
    const unsigned char* ubase = reinterpret_cast<const unsigned char*>(U) + (size_t)kb * g.Cp * 4;
    const float* uw = reinterpret_cast<const float*>(part[wave < 3 ? wave : 0]);       // the wave's twelve positions, row xi0 first
    const uint32_t ulds = (uint32_t)(uintptr_t)(lds_byte_t*)reinterpret_cast<const unsigned char*>(uw);
    auto fetch_filter = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 6; ++p)
            dma_load_1k_s(ubase + (size_t)((p < 3 ? xi0 : xi1) * 6 + 2 * (p % 3)) * plane + (size_t)c0 * 4, uoff, ulds + (uint32_t)p * 1024u);
    };
    if (wave < 3) fetch_filter(0);

    // Windows.  Addresses are clamped into the image and what lies outside is masked afterwards, so that every load is issued unconditionally.
    // Columns 1..4 of a window are the tile's own; column 0 is the left neighbour's column 4 and column 5 the right neighbour's column 1:
    // consecutive tiles of a tile row sit in consecutive lanes, and at the ends of a tile row the border column lies outside the image.
    // Only the first and last of 16 lanes load one.  Wave w loads window rows w and w + 4 for all.
    uint32_t cmask[6];
    int coff[4];
    const int pix = NHWC ? g.C : 1;                         // distance of neighbouring pixels / of neighbouring channels in x
    const size_t chan = NHWC ? 1 : (size_t)Hs * Ws;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        const int c = 4 * tj - 1 + a;
        cmask[a] = (c >= 0 && c < W) ? 0xffffffffu : 0u;
        if (a >= 1 && a <= 4) coff[a - 1] = (min(c, W - 1) >> up) * pix;
    }
    const int ecol = i == 0 ? 4 * tj - 1 : 4 * tj + 4;
    const int eoff = (min(max(ecol, 0), W - 1) >> up) * pix;
    const uint32_t emask = i == 0 ? cmask[0] : cmask[5];
    const float* xn = x + (size_t)n * g.C * Hs * Ws;
    auto load_rows = [&](int c0) __attribute__((always_inline)) {
        uint4 own[2][2];
        uint32_t edge[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = 4 * ti - 1 + wave + 4 * h;
            const int roff = (min(max(r, 0), H - 1) >> up) * Ws * pix;
            if (wave + 4 * h >= 6) continue;                // wave-uniform
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float* xc = xn + (size_t)min(c0 + 2 * q + j, g.C - 1) * chan + roff;
                if constexpr (ROWVEC) own[h][j] = *reinterpret_cast<const uint4*>(xc + coff[0]);
                else own[h][j] = make_uint4(__float_as_uint(xc[coff[0]]), __float_as_uint(xc[coff[1]]), __float_as_uint(xc[coff[2]]), __float_as_uint(xc[coff[3]]));
                if (i == 0 || i == 15) edge[h][j] = __float_as_uint(xc[eoff]);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int a = wave + 4 * h, r = 4 * ti - 1 + a;
            if (a >= 6) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t m = r >= 0 && r < H && c0 + 2 * q + j < g.C ? 0xffffffffu : 0u;
                uint4 o = own[h][j];
                o.x &= m; o.y &= m; o.z &= m; o.w &= m;
                if constexpr (!ROWVEC) { o.y &= cmask[2]; o.z &= cmask[3]; o.w &= cmask[4]; }
                xs[j][a][lane] = o;
                if (i == 0 || i == 15) es[j][a][lane] = edge[h][j] & m & emask;
            }
        }
    };

    f32x4_t acc[12];
#pragma unroll
    for (int p = 0; p < 12; ++p) acc[p] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < g.Cp; c0 += 8) {
        if (c0 > 0) {
            __syncthreads();                                // every wave has read the previous channels
            if (wave < 3) fetch_filter(c0);
        }
        load_rows(c0);
        __syncthreads();
        if (wave == 3) continue;
        // channel by channel: the twelve values of one are gone before those of the next are made (registers for four workgroups to a unit)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float d[6][6], tmp[2][6], v[2][6];              // v: [row xi0 / xi1][nu]
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                const uint4 o = xs[j][a][lane];
                const uint32_t e = es[j][a][lane];          // of the first and last of 16 lanes only
                d[a][0] = __uint_as_float(from_left(e, o.w) & cmask[0]);
                d[a][5] = __uint_as_float(from_right(e, o.x) & cmask[5]);
                d[a][1] = __uint_as_float(o.x); d[a][2] = __uint_as_float(o.y); d[a][3] = __uint_as_float(o.z); d[a][4] = __uint_as_float(o.w);
            }
            // B^T: row 0 = P and row 5 = Q of 4 d0 - 5 d2 + d4, 4 d1 - 5 d3 + d5; rows 1, 2 = P +- Q of d4 - 4 d2, d3 - 4 d1; rows 3, 4 of d4 - d2, 2 (d3 - d1)
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                if (wave == 0) {
                    tmp[0][b] = 4.f * d[0][b] - 5.f * d[2][b] + d[4][b];
                    tmp[1][b] = 4.f * d[1][b] - 5.f * d[3][b] + d[5][b];
                } else {
                    const float P = wave == 1 ? d[4][b] - 4.f * d[2][b] : d[4][b] - d[2][b];
                    const float Q = wave == 1 ? d[3][b] - 4.f * d[1][b] : 2.f * (d[3][b] - d[1][b]);
                    tmp[0][b] = P + Q;
                    tmp[1][b] = P - Q;
                }
            }
            bt_1d<4>(tmp[0], v[0]);
            bt_1d<4>(tmp[1], v[1]);
            if (j == 0) wait_vmcnt<0>();                    // the wave's filter has landed (its own transfers: no barrier)
#pragma unroll
            for (int p = 0; p < 12; ++p)
                acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(uw[p * 128 + i * 8 + q * 2 + j], v[p / 6][p % 6], acc[p], 0, 0, 0);
        }
        lds_wait<0>();                                      // every read of the block has returned
    }
    if (wave < 3) {
        // along nu: row sums of the wave's two rows
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4_t z[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float in[6], o[4];
#pragma unroll
                for (int nu = 0; nu < 6; ++nu) in[nu] = acc[h * 6 + nu][r];
                at_1d<4>(in, o);
#pragma unroll
                for (int b = 0; b < 4; ++b) z[b][r] = o[b];
            }
#pragma unroll
            for (int b = 0; b < 4; ++b) part[wave][(h * 4 + b) * 64 + lane] = z[b];
        }
    }
    __syncthreads();

    // Along xi: wave a makes row a of the output tiles.  16x16 accumulator layout: register r of lane l holds output channel 4*(l/16) + r of tile l%16.
    const int k0 = kb + 4 * q, ii = 4 * ti + wave;
    if (tb + i >= g.T || ii >= H || k0 >= g.K) return;
    f32x4_t out[4], bb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int kk = min(k0 + r, g.K - 1);
        bb[r] = (bias ? bias[kk] : 0.f) + (post.addvec ? post.addvec[(size_t)n * g.K + kk] : 0.f);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        f32x4_t z[6];
#pragma unroll
        for (int xi = 0; xi < 6; ++xi) z[xi] = part[xi % 5 == 0 ? 0 : (xi + 1) / 2][((xi == 0 || xi % 2 == 1) && xi != 5 ? b : 4 + b) * 64 + lane];
        const f32x4_t p = z[1] + z[2], m = z[1] - z[2], r = z[3] + z[4], s = z[3] - z[4];
        out[b] = (wave == 0 ? z[0] + p + r : (wave == 1 ? m + 2.f * s : (wave == 2 ? p + 4.f * r : m + 8.f * s + z[5]))) + bb;
    }
    const float* res = static_cast<const float*>(post.residual);
    if constexpr (NHWC) {
        // a lane's four channels are adjacent: one 16-byte store per pixel, four lanes to a 64-byte run
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int jj = 4 * tj + b;
            if (jj >= W) continue;
            const size_t o = (((size_t)n * H + ii) * W + jj) * g.K + k0;
            if (vec_ok) {                                   // K is a multiple of 4 here
                f32x4_t w = out[b];
                if (res) w += *reinterpret_cast<const f32x4_t*>(res + o);
                *reinterpret_cast<f32x4_t*>(y + o) = w;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (k0 + r < g.K) y[o + r] = out[b][r] + (res ? res[o + r] : 0.f);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (k0 + r >= g.K) continue;
            const size_t o = (((size_t)n * g.K + k0 + r) * H + ii) * W + 4 * tj;
            if (vec_ok) {
                f32x4_t w = {out[0][r], out[1][r], out[2][r], out[3][r]};
                if (res) w += *reinterpret_cast<const f32x4_t*>(res + o);
                *reinterpret_cast<f32x4_t*>(y + o) = w;
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (4 * tj + b < W) y[o + b] = out[b][r] + (res ? res[o + b] : 0.f);
            }
        }
    }
}

// fp32 storage, F(4x4), at most 16 (padded) input channels and no GroupNorm on the way in.  Against the three-kernel chain (us, NCHW / channel-last):
// 4 -> 320 at 64x64 7.3 / 9.3 against 21.4 / 20.7, N=2 at 128x128 21 / 29 against 61 / 59; 16 -> 320 at 64x64 10.0 / 13.6 against 20.6 / 20.4.
// Where two chunks of eight channels are left to the chain the line was drawn with one wave to a block, whose serial chain took 12-13 us
// however small the call was, 20 element by element (that kernel / the chain, NCHW: 16 -> 320 at 16x16 12.2 / 11.1, -> 8 at 64x64 12.5 / 11.6, ->
// 64 12.3 / 12.4; at 78x43 -> 64 20.7 / 16.7, -> 320 21.8 / 22.8; channel-last with a number of output channels that is no multiple of four,
// whose stores are single words, 4 -> 5 at 16x16 15.7 / 9.8); it has not been drawn again for this one.
bool fewc_conv_ok(const Geom& g, int dt, bool nhwc, const PreOp* pre) {
    if (!(dt == DT_F32 && g.m == 4 && g.Cp <= 16 && !(pre && pre->stats))) return false;
    if ((size_t)g.C * g.H * g.W >= ((size_t)1 << 30) || (size_t)g.K * g.Cp >= ((size_t)1 << 28)) return false;       // lane offsets are 32-bit
    const bool element = !nhwc && (g.W % 4 != 0 || (pre && pre->up));
    const long long size = (long long)g.T * (g.K + 64LL);
    if (nhwc && g.K % 4 != 0) return size >= 131072;
    return g.Cp <= 8 || size >= (element ? 81920 : 32768);
}

hipError_t launch_fewc_conv(const void* x, const void* U, const float* bias, void* y, const Geom& g, bool nhwc, const PreOp* pre,
                            const PostOp* postp, hipStream_t s) {
    const PostOp post = postp ? *postp : PostOp();
    const int tiles_t = (g.T + 15) / 16;
    const long long blocks = (long long)tiles_t * ((g.K + 15) / 16);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const FewcGeom fg{g.N, g.C, g.H, g.W, g.K, g.Cp, g.th, g.tw, g.T};
    const bool p16 = (reinterpret_cast<uintptr_t>(y) & 15u) == 0 && (reinterpret_cast<uintptr_t>(post.residual) & 15u) == 0;
    const int vec_ok = p16 && (nhwc ? g.K % 4 == 0 : g.W % 4 == 0);
    const int up = pre ? pre->up : 0;
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, (const float*)x, (const float*)U, bias, (float*)y, fg, tiles_t, vec_ok, up, post);
        return hipGetLastError();
    };
    if (nhwc) return run(wino_fewc_f4_kernel<true, false>);
    return !up && g.W % 4 == 0 ? run(wino_fewc_f4_kernel<false, true>) : run(wino_fewc_f4_kernel<false, false>);
}

}  // namespace wino

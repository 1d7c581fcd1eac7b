// All three steps in one kernel for F(4x4,3x3) with few input channels and fp32 storage (Section "Techniques"): the first
// convolution of the UNet (4 -> 320 channels).  With a reduction of 4...16 the three-kernel chain is three launches around
// next to no arithmetic: it writes and re-reads V and M (4 and 9 bytes per byte of y) and every launch costs its 2-3 us.
//
// A wave owns 16 tiles x 16 output channels for all 36 positions.  The reduction is taken eight channels at a time, as two
// steps of v_mfma_f32_16x16x4_f32: lane (i = l % 16, q = l / 16) holds channels c0 + 2q and c0 + 2q + 1 of row i, in both
// operands (which channel sits in which step does not matter as long as both agree).  So a lane transforms the windows
// of its own tile's two channels and the result is its operand of all 72 MFMAs: V exists only in registers.  The accumulators
// of one lane hold the 36 positions of four (channel, tile) pairs, so step (iii) is lane-local too.  The activation
// transform is repeated by the K/16 waves of a tile group: at eight channels that is 300 vector instructions, less than the
// launch it replaces.
// Loads that put 64 lanes on 64 places cost 64 clocks each however few bytes they fetch (first version: 12.7 us for
// 4 -> 320 at 64x64).  So a lane loads only the four columns its tile owns, one 16-byte load per row in NCHW, and takes
// the two border columns from its neighbours' registers; the filter block comes in as 1 KB transfers into LDS.
// Bound by latency on small images, by writing y on large ones.
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
__global__ void __launch_bounds__(64)
wino_fewc_f4_kernel(const float* __restrict__ x, const float* __restrict__ U, const float* __restrict__ bias, float* __restrict__ y,
                    FewcGeom g, int tiles_t, int vec_ok, int up, PostOp post) {
    __shared__ __attribute__((aligned(1024))) float ub[36 * 128];           // filter block of the chunk, [position][channel][8]
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int kb = (int)(blockIdx.x / (unsigned)tiles_t) * 16, tb = (int)(blockIdx.x % (unsigned)tiles_t) * 16;
    const int H = g.H, W = g.W, Hs = H >> up, Ws = W >> up;

    // filter transfers: 32 lanes per position, two 16-byte halves per row of eight channels; rows beyond K repeat the last one
    const uint32_t plane = (uint32_t)g.K * (uint32_t)g.Cp * 4u;
    const uint32_t uoff = (uint32_t)(lane >> 5) * plane + (uint32_t)(min(kb + ((lane & 31) >> 1), g.K - 1) - kb) * (uint32_t)g.Cp * 4u + (uint32_t)(lane & 1) * 16u;
    const unsigned char* ubase = reinterpret_cast<const unsigned char*>(U) + (size_t)kb * g.Cp * 4;
    const uint32_t ulds = (uint32_t)(uintptr_t)(lds_byte_t*)reinterpret_cast<unsigned char*>(ub);
    auto fetch_filter = [&](int c0) {
#pragma unroll
        for (int p = 0; p < 18; ++p) dma_load_1k_s(ubase + (size_t)(2 * p) * plane + (size_t)c0 * 4, uoff, ulds + (uint32_t)p * 1024u);
    };
    fetch_filter(0);

    // this lane's tile (clamped to the last one; its results are then never stored)
    const int t = min(tb + i, g.T - 1);
    const int tj = t % g.tw, tq = t / g.tw, ti = tq % g.th, n = tq / g.th;

    // Window addresses, clamped into the image, and masks (as in the channel-last activation transform: every load is
    // issued unconditionally and masked afterwards, so that they all overlap).  Columns 1..4 are the tile's own; column 0 is the left
    // neighbour's column 4 and column 5 the right neighbour's column 1: consecutive tiles of a tile row sit in consecutive
    // lanes, and at the ends of a tile row the border column lies outside the image.  Only the first and last of 16 lanes load one.
    int roff[6], coff[4];
    uint32_t rmask[6], cmask[6];
    const int pix = NHWC ? g.C : 1;                         // distance of neighbouring pixels / of neighbouring channels in x
    const size_t chan = NHWC ? 1 : (size_t)Hs * Ws;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        const int r = 4 * ti - 1 + a, c = 4 * tj - 1 + a;
        roff[a] = (min(max(r, 0), H - 1) >> up) * Ws * pix;
        rmask[a] = (r >= 0 && r < H) ? 0xffffffffu : 0u;
        cmask[a] = (c >= 0 && c < W) ? 0xffffffffu : 0u;
        if (a >= 1 && a <= 4) coff[a - 1] = (min(c, W - 1) >> up) * pix;
    }
    const int ecol = i == 0 ? 4 * tj - 1 : 4 * tj + 4;
    const int eoff = (min(max(ecol, 0), W - 1) >> up) * pix;
    const float* xn = x + (size_t)n * g.C * Hs * Ws;

    f32x4_t acc[36];
#pragma unroll
    for (int p = 0; p < 36; ++p) acc[p] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int c0 = 0; c0 < g.Cp; c0 += 8) {
        uint32_t own[2][6][4], edge[2][6];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float* xc = xn + (size_t)min(c0 + 2 * q + j, g.C - 1) * chan;
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                if constexpr (ROWVEC) {
                    const uint4 w = *reinterpret_cast<const uint4*>(xc + roff[a] + coff[0]);
                    own[j][a][0] = w.x; own[j][a][1] = w.y; own[j][a][2] = w.z; own[j][a][3] = w.w;
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b) own[j][a][b] = *reinterpret_cast<const uint32_t*>(xc + roff[a] + coff[b]);
                }
                edge[j][a] = 0u;
            }
            if (i == 0 || i == 15) {
#pragma unroll
                for (int a = 0; a < 6; ++a) edge[j][a] = *reinterpret_cast<const uint32_t*>(xc + roff[a] + eoff);
            }
        }
        float v[2][6][6];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t live = c0 + 2 * q + j < g.C ? 0xffffffffu : 0u;
            float d[6][6], tmp[6][6];
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                const uint32_t m = rmask[a] & live;
                d[a][0] = __uint_as_float(from_left(edge[j][a], own[j][a][3]) & m & cmask[0]);
                d[a][5] = __uint_as_float(from_right(edge[j][a], own[j][a][0]) & m & cmask[5]);
#pragma unroll
                for (int b = 0; b < 4; ++b) d[a][b + 1] = __uint_as_float(own[j][a][b] & (ROWVEC ? m : m & cmask[b + 1]));
            }
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                float in[6], out[6];
#pragma unroll
                for (int a = 0; a < 6; ++a) in[a] = d[a][b];
                bt_1d<4>(in, out);
#pragma unroll
                for (int a = 0; a < 6; ++a) tmp[a][b] = out[a];
            }
#pragma unroll
            for (int xi = 0; xi < 6; ++xi) bt_1d<4>(tmp[xi], v[j][xi]);
        }
        wait_vmcnt<0>();                                    // the filter block has landed (one wave per workgroup: no barrier)
#pragma unroll
        for (int p = 0; p < 36; ++p) {
            const float2 u = *reinterpret_cast<const float2*>(ub + p * 128 + i * 8 + q * 2);
            acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.x, v[0][p / 6][p % 6], acc[p], 0, 0, 0);
            acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.y, v[1][p / 6][p % 6], acc[p], 0, 0, 0);
        }
        if (c0 + 8 < g.Cp) {
            lds_wait<0>();                                  // every read of the block has returned
            fetch_filter(c0 + 8);
        }
    }

    // 16x16 accumulator layout: register r of lane l holds output channel 4*(l/16) + r of tile l%16
    if (tb + i >= g.T) return;
    const float* res = static_cast<const float*>(post.residual);
    float out[4][4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float tmp[4][6];
#pragma unroll
        for (int nu = 0; nu < 6; ++nu) {
            float in[6], o[4];
#pragma unroll
            for (int xi = 0; xi < 6; ++xi) in[xi] = acc[xi * 6 + nu][r];
            at_1d<4>(in, o);
#pragma unroll
            for (int a = 0; a < 4; ++a) tmp[a][nu] = o[a];
        }
        const int kk = min(kb + 4 * q + r, g.K - 1);
        const float bb = (bias ? bias[kk] : 0.f) + (post.addvec ? post.addvec[(size_t)n * g.K + kk] : 0.f);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            at_1d<4>(tmp[a], out[r][a]);
#pragma unroll
            for (int b = 0; b < 4; ++b) out[r][a][b] += bb;
        }
    }
    const int k0 = kb + 4 * q;
    if constexpr (NHWC) {
        // a lane's four channels are adjacent: one 16-byte store per pixel, four lanes to a 64-byte run
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int ii = 4 * ti + a, jj = 4 * tj + b;
                if (ii >= H || jj >= W) continue;
                const size_t o = (((size_t)n * H + ii) * W + jj) * g.K + k0;
                if (vec_ok) {
                    if (k0 >= g.K) continue;                // K is a multiple of 4 here
                    float4 w = make_float4(out[0][a][b], out[1][a][b], out[2][a][b], out[3][a][b]);
                    if (res) { const float4 rr = *reinterpret_cast<const float4*>(res + o); w.x += rr.x; w.y += rr.y; w.z += rr.z; w.w += rr.w; }
                    *reinterpret_cast<float4*>(y + o) = w;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (k0 + r < g.K) y[o + r] = out[r][a][b] + (res ? res[o + r] : 0.f);
                }
            }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (k0 + r >= g.K) continue;
            const size_t off = (((size_t)n * g.K + k0 + r) * H + 4 * ti) * W + 4 * tj;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                if (4 * ti + a >= H) continue;
                const size_t o = off + (size_t)a * W;
                if (vec_ok) {
                    float4 w = make_float4(out[r][a][0], out[r][a][1], out[r][a][2], out[r][a][3]);
                    if (res) { const float4 rr = *reinterpret_cast<const float4*>(res + o); w.x += rr.x; w.y += rr.y; w.z += rr.z; w.w += rr.w; }
                    *reinterpret_cast<float4*>(y + o) = w;
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (4 * tj + b < W) y[o + b] = out[r][a][b] + (res ? res[o + b] : 0.f);
                }
            }
        }
    }
}

// fp32 storage, F(4x4), at most 16 (padded) input channels and no GroupNorm on the way in.  Measured against the three-kernel chain (us,
// NCHW / channel-last): 4 -> 320 at 64x64 10.9 / 12.4 against 21.4 / 20.7, N=2 at 128x128 30 / 43 against 61 / 59; 16 -> 320 at 64x64
// 14.5 / 18.1 against 20.6 / 20.4, N=2 at 128x128 43 / 58 against 62 / 59; with 24 channels level, with 32 slower (22.5 / 28.7 against 20.5 / 21.0).
// With two chunks of eight channels a wave's chain takes 12-13 us however small the call is, 20 element by element (NCHW rows that are no
// whole 16-byte pieces, and upsampling); the chain's kernels back to back take less where there are few tiles and output channels (here / there,
// NCHW: 16 -> 320 at 16x16 12.2 / 11.1, -> 8 at 64x64 12.5 / 11.6, -> 64 12.3 / 12.4, -> 320 13.4 / 19.5, -> 8 at 96x96 (N=2) 12.6 / 14.1;
// at 78x43 -> 64 20.7 / 16.7, -> 320 21.8 / 22.8, at 128x125 -> 8 19.9 / 17.4, -> 64 21.0 / 22.3).  Channel-last with a number of output
// channels that is no multiple of four, stores are single words (4 -> 5 at 16x16 15.7 / 9.8, at 96x96 15.9 / 11.5).
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
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64), 0, s, (const float*)x, (const float*)U, bias, (float*)y, fg, tiles_t, vec_ok, up, post);
        return hipGetLastError();
    };
    if (nhwc) return run(wino_fewc_f4_kernel<true, false>);
    return !up && g.W % 4 == 0 ? run(wino_fewc_f4_kernel<false, true>) : run(wino_fewc_f4_kernel<false, false>);
}

}  // namespace wino

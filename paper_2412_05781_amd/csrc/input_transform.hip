// Step (i), activation side (Section "Techniques"): V = B^T d B for every
// overlapping alpha x alpha window d of the zero-padded image, per channel.
//
// x is NCHW (W contiguous) but the GEMM stage wants the reduction index c
// contiguous, V[alpha^2][T][Cp].  A workgroup therefore stages a patch of
// CB channels x alpha rows x (m*TJ+2) columns in LDS with loads that run along
// W, then each lane takes one channel of one tile, transforms it in fp32 and
// stores with lanes running along c.  Out-of-image taps and channels >= C are
// staged as zeros, so V's padded reduction columns are exact zeros.
// Four kernels: a scalar one for any row length, the chunked strip kernel, the
// sliding-window kernel for long rows, and the channel-last kernel, which needs no
// transposition.  All of them can apply SiLU(GroupNorm(.)) to what they load and
// read x through a 2x nearest-neighbour upsampling.
// Bound by HBM/L2 traffic: reads x once (plus the 2-row/2-column halo), writes V.
#include "wino_internal.h"
#include "wino_transforms.h"

namespace wino {

// These kernels are bound by the vector ALU and by LDS reads as much as by memory: windows are read from LDS as 32-bit words, shared
// columns of neighbouring tiles are read, normalised and transformed once, and SiLU takes the hardware's exponential and reciprocal.
// 512 channels at 256x256 with GroupNorm 87 -> 71 us, 1280 at 16x16 channel-last 9.0 -> 5.7, 320 at 64x64 11.4 -> 10.2.
//
// The transforms of NT neighbouring tiles of a tile row for one channel.  get(a, b): element (a, b) of the (m+2) x (m*NT+2) window;
// put(u, xi, nu, value): position (xi, nu) of tile u.  Columns that two windows share are transformed once.
template <int M, int NT, typename Get, typename Put>
__device__ __forceinline__ void transform_tiles(Get&& get, Put&& put) {
    constexpr int A = M + 2, NC = M * NT + 2;
    float tmp[A][NC];                                    // tmp[:, b] = B^T d[:, b]
#pragma unroll
    for (int b = 0; b < NC; ++b) {
        float in[A], out[A];
#pragma unroll
        for (int a = 0; a < A; ++a) in[a] = get(a, b);
        bt_1d<M>(in, out);
#pragma unroll
        for (int a = 0; a < A; ++a) tmp[a][b] = out[a];
    }
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int xi = 0; xi < A; ++xi) {
            float out[A];
            bt_1d<M>(tmp[xi] + M * u, out);              // rows: (B^T d) B = (B^T (B^T d)^T)^T
#pragma unroll
            for (int nu = 0; nu < A; ++nu) put(u, xi, nu, out[nu]);
        }
}

// element h (0 or 1) of a 32-bit word of storage elements; fp32: the word itself
template <typename E> __device__ __forceinline__ float unpack(uint32_t w, int h) {
    if constexpr (sizeof(E) == 4) return __uint_as_float(w);
    const uint16_t e = (uint16_t)(h ? w >> 16 : w & 0xffffu);
    return to_f32<E>(*reinterpret_cast<const E*>(&e));
}

// two neighbouring two-byte elements at an address of any element
struct __attribute__((packed, aligned(2))) pair_t { uint32_t w; };

// PAIRS: two-byte types and stored rows of at least two elements: the patch is fetched in pairs of columns.
template <int M, typename E, int CB, int TJ, bool PRE, bool PAIRS>
__global__ void __launch_bounds__(256)
input_transform_nchw_kernel(const E* __restrict__ x, E* __restrict__ V,
                            int N, int C, int H, int W, int th, int tw, int T, int Cp, int strips_per_row, PreOp pre) {
    constexpr int A = M + 2;
    constexpr int PW = M * TJ + 2;                       // patch width (elements)
    // channel stride: odd number of 32-bit words so lanes (= channels) hit distinct banks
    constexpr int RAW = A * PW;
    constexpr int EPW = 4 / (int)sizeof(E);              // elements per 32-bit word
    constexpr int CSW = (RAW / EPW) | 1;
    static_assert(PW % EPW == 0 && M % EPW == 0 && CB == 64, "windows start on a word; lane = channel");
    __shared__ uint32_t patch[CB * CSW];

    const int tid = threadIdx.x;
    int sidx = blockIdx.x;
    const int js = sidx % strips_per_row; sidx /= strips_per_row;
    const int ti = sidx % th;
    const int n = sidx / th;
    const int tj0 = js * TJ;
    const int c0 = blockIdx.y * CB;
    const int row0 = M * ti - 1;
    const int col0 = M * tj0 - 1;

    const int cc = tid & 63;
    const int c = c0 + cc;
    PreRaw raw = {0.f, 0.f, 0.f, 0.f};                    // requested here, with the pixels
    if (PRE) raw = pre_request(pre, n, c, C);

    // ---- stage the patch: a lane owns one patch position and walks the channels, so its address and its bounds test are found once;
    // consecutive lanes walk along W.  Loads are issued from clamped addresses and masked: all of a lane's are in flight together.
    // (Element by element over [channel][row][column], each index divided out and tested: 20.2 us against 11.9 for 640 channels, N=2,
    // 52x78 upsampled.)
    const int Hs = H >> pre.up, Ws = W >> pre.up;
    const size_t img = (size_t)Hs * Ws;
    if constexpr (PAIRS) {
        // The window's first column is odd, so a pair of columns is a pair of neighbours in x whether that is read upsampled or not.  At the
        // ends of a row the pair one place further in is fetched and shifted.  (A whole call of 640 channels, N=2, 52x78 upsampled, single
        // elements / pairs: 55.9 / 54.5 us; 960 at 34x50 upsampled 33.6 / 32.7.)
        constexpr int PWW = PW / 2, RAWW = A * PWW, G = 256 / RAWW, LOADS = (CB + G - 1) / G;
        const int rem = tid % RAWW, cg = tid / RAWW;
        const int pr = row0 + rem / PWW, pq = col0 + 2 * (rem % PWW);
        const int s0 = pq >> pre.up, sc = min(max(s0, 0), Ws - 2);
        const int left = s0 < sc ? 16 : 0, right = s0 > sc ? 16 : 0;
        const uint32_t in = pr >= 0 && pr < H ? (pq >= 0 && pq < W ? 0xffffu : 0u) | (pq + 1 >= 0 && pq + 1 < W ? 0xffff0000u : 0u) : 0u;
        // 32-bit lane offsets from the slab's first pixel: the slab spans less than 2 GB
        const unsigned char* xp = reinterpret_cast<const unsigned char*>(x + ((size_t)n * C + c0) * img);
        const uint32_t plane = (uint32_t)img * 2u, last = (uint32_t)min(CB - 1, C - 1 - c0);
        const uint32_t pix = ((uint32_t)(min(max(pr, 0), H - 1) >> pre.up) * (uint32_t)Ws + (uint32_t)sc) * 2u;
        const uint32_t most = pix + last * plane;         // channels beyond the last repeat it, and are staged as zeros
        uint32_t off = pix + (uint32_t)cg * plane, v[LOADS];
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            v[i] = reinterpret_cast<const pair_t*>(xp + min(off, most))->w;
            off += (uint32_t)G * plane;
        }
        if (cg < G) {
            uint32_t* dst = patch + cg * CSW + rem;
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const uint32_t w = v[i] << left >> right & in;
                if (CB % G == 0 || cg + G * i < CB) dst[G * i * CSW] = (uint32_t)(cg + G * i) <= last ? w : 0u;
            }
        }
    } else {
    constexpr int G = 256 / RAW;                         // channels in hand at a time
    constexpr int LOADS = (CB + G - 1) / G;
    const int rem = tid % RAW, cg = tid / RAW;
    const int pr = row0 + rem / PW, pq = col0 + rem % PW;
    const bool in = pr >= 0 && pr < H && pq >= 0 && pq < W;
    const E* xp = x + ((size_t)n * C + c0) * img + (size_t)(min(max(pr, 0), H - 1) >> pre.up) * Ws + (min(max(pq, 0), W - 1) >> pre.up);
    E v[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) v[i] = xp[(size_t)min(cg + G * i, C - 1 - c0) * img];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int ch = cg + G * i;
        if (cg < G && ch < CB) reinterpret_cast<E*>(patch + ch * CSW)[rem] = in && c0 + ch < C ? v[i] : from_f32<E>(0.f);
    }
    }
    __syncthreads();

    // ---- transform: lane = channel, one tile per wave per iteration ----------------------
    PreLane pl = {0.f, 0.f, false};
    if (PRE) pl = pre_finish(raw, c, C);
    if (c >= Cp) return;                                 // no barrier follows
    const size_t plane = (size_t)T * Cp;
    for (int tl = __builtin_amdgcn_readfirstlane(tid >> 6); tl < TJ; tl += 4) {
        const int tj = tj0 + tl;
        if (tj >= tw) break;                             // wave-uniform
        const uint32_t* p = patch + cc * CSW + M * tl / EPW;
        uint32_t w[A][A / EPW];
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int b = 0; b < A / EPW; ++b) w[a][b] = p[a * (PW / EPW) + b];
        const size_t t = ((size_t)n * th + ti) * tw + tj;
        E* dst = V + t * Cp + c;
        transform_tiles<M, 1>(
            [&](int a, int b) __attribute__((always_inline)) {
                float d = unpack<E>(w[a][b / EPW], b % EPW);
                if (PRE) {
                    const int r = M * ti - 1 + a, q = M * tj - 1 + b;
                    d = pre_apply_as<E>(d, pl, r >= 0 && r < H && q >= 0 && q < W);
                }
                return d;
            },
            [&](int, int xi, int nu, float o) __attribute__((always_inline)) { dst[(size_t)(xi * A + nu) * plane] = from_f32<E>(o); });
    }
}

// Fast path for rows that are whole 16-byte chunks (W*sizeof(E) a multiple of 16): the patch is
// fetched as 16-byte chunks, all loads of a lane issued before the first LDS write, so one global
// round trip covers the whole patch.  Patch columns run from m*tj0 - EPC to m*(tj0+TJ) + EPC
// (EPC = elements per chunk); a chunk is either wholly inside the image or wholly outside (zero).
template <int M, typename E, int CB, int TJ, bool PRE, int UP>
__global__ void __launch_bounds__(256)
input_transform_nchw_vec_kernel(const E* __restrict__ x, E* __restrict__ V,
                                int N, int C, int H, int W, int th, int tw, int T, int Cp, int strips_per_row,
                                int total_blocks, int blocks_per_xcd, PreOp pre) {
    constexpr int A = M + 2;
    constexpr int EPC = 16 / (int)sizeof(E);
    static_assert((M * TJ) % EPC == 0, "strip width must be whole chunks");
    constexpr int NCH = (M * TJ) / EPC + 2;              // chunks per patch row
    constexpr int ROWW = NCH * 4;                        // 32-bit words per patch row
    constexpr int CSW = (A * ROWW) | 1;                  // words per channel, odd: lanes = channels hit distinct banks
    __shared__ uint32_t patch[CB * CSW];

    const int tid = threadIdx.x;
    // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of
    // (channel chunk, n, tile row, strip) so neighbours that share halo rows share an L2.
    const int logical = (blockIdx.x % 8) * blocks_per_xcd + blockIdx.x / 8;
    if (logical >= total_blocks) return;                 // uniform, before the barrier
    int sidx = logical;
    const int js = sidx % strips_per_row; sidx /= strips_per_row;
    const int ti = sidx % th; sidx /= th;
    const int n = sidx % N;
    const int c0 = (sidx / N) * CB;
    const int tj0 = js * TJ;
    const int row0 = M * ti - 1;
    const int col0 = M * tj0 - EPC;
    static_assert(CB == 64, "lane = channel");
    const int cc = tid & 63;                              // of the transform
    const int c = c0 + cc;
    PreRaw raw = {0.f, 0.f, 0.f, 0.f};                    // requested here, with the pixels
    if (PRE) raw = pre_request(pre, n, c, C);

    // 32-bit lane offsets against wave-uniform 64-bit bases keep the address arithmetic off the
    // vector ALU (the transform itself is only ~200 operations per tile and channel).
    const int Hs = H >> UP, Ws = W >> UP;                 // the stored image (half size when it is read upsampled)
    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x + ((size_t)n * C + c0) * Hs * Ws);
    // A lane owns one (channel, chunk column) and walks the alpha patch rows.  Loads come from clamped addresses and what lies outside is
    // cleared afterwards: none sits in a branch, where an upsampled row would be waited for before the next one is requested.
    constexpr int ITEMS = CB * NCH;
    constexpr int PASSES = (ITEMS + 255) / 256;
    uint4 reg[PASSES][A];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int item = min(tid + ps * 256, ITEMS - 1);
        const int cc = min(item / NCH, C - 1 - c0), col = min(max(col0 + item % NCH * EPC, 0), W - EPC);
        const unsigned lane0 = (unsigned)((cc * Hs * Ws + (col >> UP)) * (int)sizeof(E));
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const unsigned off = lane0 + (unsigned)((min(max(row0 + a, 0), H - 1) >> UP) * Ws * (int)sizeof(E));
            if constexpr (UP) {                           // 8 source bytes under the 16-byte chunk
                const uint2 h = *reinterpret_cast<const uint2*>(xb + off);
                reg[ps][a].x = h.x; reg[ps][a].y = h.y;
            } else reg[ps][a] = *reinterpret_cast<const uint4*>(xb + off);
        }
    }
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int item = tid + ps * 256, cc = item / NCH, col = col0 + (item - cc * NCH) * EPC;
        const bool ok = c0 + cc < C && col >= 0 && col + EPC <= W;
#pragma unroll
        for (int a = 0; a < A; ++a) {
            if constexpr (UP) reg[ps][a] = dup_elements<E>(make_uint2(reg[ps][a].x, reg[ps][a].y));        // every element twice
            const uint32_t m = ok && row0 + a >= 0 && row0 + a < H ? ~0u : 0u;
            reg[ps][a].x &= m; reg[ps][a].y &= m; reg[ps][a].z &= m; reg[ps][a].w &= m;
        }
    }
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int item = tid + ps * 256;
        if (item < ITEMS) {
            const int cc = item / NCH, ch = item - cc * NCH;
            uint32_t* dst = patch + cc * CSW + ch * 4;
#pragma unroll
            for (int a = 0; a < A; ++a) {
                dst[a * ROWW + 0] = reg[ps][a].x; dst[a * ROWW + 1] = reg[ps][a].y;
                dst[a * ROWW + 2] = reg[ps][a].z; dst[a * ROWW + 3] = reg[ps][a].w;
            }
        }
    }
    __syncthreads();

    // one tile per wave per iteration (lane = channel), so the tile index is wave-uniform
    const size_t plane = (size_t)T * Cp;
    constexpr int EPW = 4 / (int)sizeof(E);
    constexpr int W0 = EPC - EPW, NWD = (A - 1 + EPW - 1) / EPW + 1;       // first word of tile 0's window (its last element), words per row
    PreLane pl = {0.f, 0.f, false};
    if (PRE) pl = pre_finish(raw, c, C);
    if (c >= Cp) return;                                  // no barrier follows
    for (int tl = __builtin_amdgcn_readfirstlane(tid >> 6); tl < TJ; tl += 4) {
        const int tj = tj0 + tl;
        if (tj >= tw) break;                              // wave-uniform
        const uint32_t* p = patch + cc * CSW + (W0 + M * tl) / EPW;
        uint32_t w[A][NWD];
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int b = 0; b < NWD; ++b) w[a][b] = p[a * ROWW + b];
        const size_t t = ((size_t)n * th + ti) * tw + tj;  // wave-uniform
        unsigned char* base = reinterpret_cast<unsigned char*>(V + t * Cp);      // wave-uniform; the lane's offset is just c
        const unsigned coff = (unsigned)c * (unsigned)sizeof(E);
        const size_t plane_bytes = plane * sizeof(E);
        transform_tiles<M, 1>(
            [&](int a, int b) __attribute__((always_inline)) {
                float d = unpack<E>(w[a][(b + EPW - 1) / EPW], (b + EPW - 1) % EPW);
                if (PRE) {
                    const int r = M * ti - 1 + a, q = M * tj - 1 + b;
                    d = pre_apply_as<E>(d, pl, r >= 0 && r < H && q >= 0 && q < W);
                }
                return d;
            },
            [&](int, int xi, int nu, float o) __attribute__((always_inline)) {
                *reinterpret_cast<E*>(base + (size_t)(xi * A + nu) * plane_bytes + coff) = from_f32<E>(o);
            });
    }
}

// Long rows: a workgroup slides along one tile row.  The row is cut into 64-byte bodies (TJ tiles
// wide); LDS keeps the last two bodies of every (channel, patch row), and step s transforms the
// TJ tiles that straddle the seam between bodies s-1 and s, whose windows lie wholly inside those
// two bodies.  Every body is therefore fetched from memory once per workgroup, as aligned 64-byte
// runs, instead of once per strip plus halo chunks on either side; body s+1 is in flight while
// step s computes and stores.  Tiles outside [0, tw) are replaced by the nearest tile inside, which
// the same step computes anyway: the duplicate writes the same values, and every wave issues the
// same number of stores per step, so the wait for the prefetched body leaves those stores pending.
// Needs Cp % 64 == 0 (no lane is idle) and rows of whole 16-byte chunks.
template <int M, typename E, int TJ, bool PRE>
__global__ void __launch_bounds__(256)
input_transform_nchw_slide_kernel(const E* __restrict__ x, E* __restrict__ V,
                                  int N, int C, int H, int W, int th, int tw, int T, int Cp, int steps_per_row,
                                  int spb, int total_blocks, int blocks_per_xcd, PreOp pre) {
    constexpr int A = M + 2;
    constexpr int EPC = 16 / (int)sizeof(E);             // elements per 16-byte chunk
    constexpr int BODYE = 64 / (int)sizeof(E);           // elements per body
    constexpr int EPW = 4 / (int)sizeof(E);              // elements per 32-bit word
    static_assert(TJ * M == BODYE && TJ % 4 == 0, "a body is TJ tiles wide, TJ/4 tiles per wave");
    constexpr int ROWW = 32;                             // words per patch row: two bodies
    constexpr int CSW = (A * ROWW) | 1;                  // words per channel, odd: lanes = channels hit distinct banks
    constexpr int NT = TJ / 4;                           // tiles per wave and step
    constexpr int NWD = (M * NT + 2 - 1 + EPW - 1) / EPW + 1;      // words per row under their windows, the first from its last element on
    __shared__ uint32_t patch[64 * CSW];

    const int tid = threadIdx.x;
    const int logical = (blockIdx.x % 8) * blocks_per_xcd + blockIdx.x / 8;   // one contiguous range per XCD
    if (logical >= total_blocks) return;                 // uniform, before any barrier
    const int groups_per_row = (steps_per_row + spb - 1) / spb;
    int sidx = logical;
    const int jg = sidx % groups_per_row; sidx /= groups_per_row;
    const int ti = sidx % th; sidx /= th;
    const int n = sidx % N;
    const int c0 = (sidx / N) * 64;
    const int s0 = jg * spb;
    const int s1 = min(s0 + spb, steps_per_row);
    const int row0 = M * ti - 1;

    const int Hs = H >> pre.up, Ws = W >> pre.up;         // the stored image (half size when it is read upsampled)
    const unsigned char* xb = reinterpret_cast<const unsigned char*>(x + ((size_t)n * C + c0) * Hs * Ws);
    // loader role: lane = (channel, chunk of the body), walks the alpha patch rows
    const int lc = tid >> 2, lch = tid & 3;
    const bool lc_ok = (c0 + lc) < C;
    uint4 reg[A];
    auto fetch = [&](int body) {
        const int col = body * BODYE + lch * EPC;
        const bool ok = lc_ok && body >= 0 && col < W;   // W is a multiple of EPC: a chunk is inside or outside as a whole
        const unsigned off0 = (unsigned)(((lc * H + row0) * W + col) * (int)sizeof(E));   // only used when row and col are valid
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int r = row0 + a;
            reg[a] = make_uint4(0, 0, 0, 0);
            if (ok && r >= 0 && r < H) {
                if (pre.up)   // 8 source bytes under the 16-byte chunk, every element twice
                    reg[a] = dup_elements<E>(*reinterpret_cast<const uint2*>(
                        xb + (unsigned)(((lc * Hs + (r >> 1)) * Ws + (col >> 1)) * (int)sizeof(E))));
                else
                    reg[a] = *reinterpret_cast<const uint4*>(xb + (off0 + (unsigned)(a * W * (int)sizeof(E))));
            }
        }
    };
    auto stash = [&](int body) {
        uint32_t* dst = patch + lc * CSW + (body & 1) * 16 + lch * 4;
#pragma unroll
        for (int a = 0; a < A; ++a) {
            dst[a * ROWW + 0] = reg[a].x; dst[a * ROWW + 1] = reg[a].y;
            dst[a * ROWW + 2] = reg[a].z; dst[a * ROWW + 3] = reg[a].w;
        }
    };

    // transform role: lane = channel, TJ/4 tiles per wave and step
    const int cc = tid & 63;
    const int c = c0 + cc;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t plane_bytes = (size_t)T * Cp * sizeof(E);
    const uint32_t* pch = patch + cc * CSW;
    const unsigned coff = (unsigned)c * (unsigned)sizeof(E);
    PreRaw raw = {0.f, 0.f, 0.f, 0.f};                    // requested here, with the pixels
    if (PRE) raw = pre_request(pre, n, c, C);

    fetch(s0 - 1);
    stash(s0 - 1);
    fetch(s0);
    stash(s0);
    __syncthreads();
    PreLane pl = {0.f, 0.f, false};
    if (PRE) pl = pre_finish(raw, c, C);
    for (int s = s0; s < s1; ++s) {
        if (s + 1 < s1) fetch(s + 1);                     // in flight while this step is transformed
        // the wave's tiles, neighbours (wave-uniform); moved inside the row as a group, the duplicates write identical values
        const int tj = min(max(TJ * s - TJ / 2 + wave * NT, 0), tw - NT);
        const int g0 = M * tj - 1;                        // first window column (global), -1 for the left border
        const int w0 = (g0 + 1 - EPW) / EPW;              // its word
        uint32_t w[A][NWD];
#pragma unroll
        for (int b = 0; b < NWD; ++b) {
            const uint32_t* p = pch + ((w0 + b) & (ROWW - 1));
#pragma unroll
            for (int a = 0; a < A; ++a) w[a][b] = p[a * ROWW];
        }
        const size_t t = ((size_t)n * th + ti) * tw + tj;                      // wave-uniform
        unsigned char* base = reinterpret_cast<unsigned char*>(V + t * Cp);
        const size_t row_bytes = (size_t)Cp * sizeof(E);
        transform_tiles<M, NT>(
            [&](int a, int b) __attribute__((always_inline)) {
                float d = unpack<E>(w[a][(b + EPW - 1) / EPW], (b + EPW - 1) % EPW);
                if (PRE) {
                    const int r = M * ti - 1 + a, q = g0 + b;
                    d = pre_apply_as<E>(d, pl, r >= 0 && r < H && q >= 0 && q < W);
                }
                return d;
            },
            [&](int u, int xi, int nu, float o) __attribute__((always_inline)) {
                *reinterpret_cast<E*>(base + (size_t)u * row_bytes + (size_t)(xi * A + nu) * plane_bytes + coff) = from_f32<E>(o);
            });
        if (s + 1 < s1) {
            __syncthreads();                              // everyone is done with body s-1
            stash(s + 1);                                 // overwrites it
            __syncthreads();
        }
    }
}

// NHWC activations (channels contiguous): no transposition is needed, V's rows are channel-
// contiguous too.  One lane owns CPT adjacent channels of one tile, reads its alpha x alpha window
// straight from global memory (neighbouring lanes read neighbouring channels, so every load is
// one contiguous run; the 2.25x / 4x window overlap is served by L1/L2) and stores CPT values
// per transformed position.  Channels in [C, Cp) are written as zeros.
template <int M, typename E, int CPT, bool PRE>
__global__ void __launch_bounds__(256)
input_transform_nhwc_kernel(const E* __restrict__ x, E* __restrict__ V,
                            int N, int C, int H, int W, int th, int tw, int T, int Cp, int per_xcd, PreOp pre) {
    constexpr int A = M + 2;
    const int groups = Cp / CPT;                               // Cp is a multiple of 8
    // workgroups go round-robin to the 8 XCDs: give each XCD one contiguous range of tiles, so
    // that the window overlap between neighbouring tiles is served by that XCD's own L2
    const size_t logical = (size_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const size_t item = logical * 256 + threadIdx.x;
    if (item >= (size_t)T * groups) return;
    const int gidx = (int)(item % groups);
    int t = (int)(item / groups);
    const int c = gidx * CPT;
    const int tj = t % tw; int q = t / tw;
    const int ti = q % th;
    const int n = q / th;
    const bool live = c < C;                                   // CPT divides C on this path
    PreRaw raw[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) { raw[u] = PreRaw{0.f, 0.f, 0.f, 0.f}; if (PRE) raw[u] = pre_request(pre, n, c + u, C); }
    // Every load is issued unconditionally from a clamped (always valid) address and the loaded
    // bits are ANDed with an all-ones / all-zeros mask, so that the alpha^2 loads of a lane are all
    // in flight together.  The masks pass through an empty asm statement: seen as a select on the
    // bounds test, the compiler moves each load into a branch of its own and waits for it there.
    const int us = pre.up;                                      // 1: x is stored at half size and read upsampled
    const E* xb = x + (size_t)n * (H >> us) * (W >> us) * C + (live ? c : 0);
    uint32_t rmask[A], cmask[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int r = M * ti - 1 + a, col = M * tj - 1 + a;
        rmask[a] = (live && r >= 0 && r < H) ? 0xffffffffu : 0u;
        cmask[a] = (col >= 0 && col < W) ? 0xffffffffu : 0u;
        asm("" : "+v"(rmask[a]));
        asm("" : "+v"(cmask[a]));
    }
    union word_t { uint32_t w; E e[4 / sizeof(E)]; };
    word_t v[A][A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
        const int r = M * ti - 1 + a;
        const E* xr = xb + (size_t)(min(max(r, 0), H - 1) >> us) * (W >> us) * C;
#pragma unroll
        for (int b = 0; b < A; ++b) {
            const int col = M * tj - 1 + b;
            const E* p = xr + (size_t)(min(max(col, 0), W - 1) >> us) * C;
            if constexpr (CPT == 2) v[a][b].w = *reinterpret_cast<const uint32_t*>(p);
            else if constexpr (sizeof(E) == 4) v[a][b].w = *reinterpret_cast<const uint32_t*>(p);
            else v[a][b].w = *reinterpret_cast<const uint16_t*>(p);
        }
    }
    PreLane pl[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) { pl[u] = PreLane{0.f, 0.f, false}; if (PRE) pl[u] = pre_finish(raw[u], c + u, C); }
    float d[CPT][A][A];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < A; ++b) {
            const uint32_t msk = rmask[a] & cmask[b];
            v[a][b].w &= msk;
#pragma unroll
            for (int u = 0; u < CPT; ++u) {
                d[u][a][b] = to_f32<E>(v[a][b].e[u]);
                if (PRE) d[u][a][b] = pre_apply_as<E>(d[u][a][b], pl[u], msk != 0u);
            }
        }
    float o[CPT][A][A];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        float tmp[A][A];
#pragma unroll
        for (int b = 0; b < A; ++b) {
            float in[A], out[A];
#pragma unroll
            for (int a = 0; a < A; ++a) in[a] = d[u][a][b];
            bt_1d<M>(in, out);
#pragma unroll
            for (int a = 0; a < A; ++a) tmp[a][b] = out[a];
        }
#pragma unroll
        for (int xi = 0; xi < A; ++xi) bt_1d<M>(tmp[xi], o[u][xi]);
    }
    const size_t plane = (size_t)T * Cp;
    E* dst = V + (size_t)t * Cp + c;
#pragma unroll
    for (int xi = 0; xi < A; ++xi)
#pragma unroll
        for (int nu = 0; nu < A; ++nu) {
            E v[CPT];
#pragma unroll
            for (int u = 0; u < CPT; ++u) v[u] = from_f32<E>(o[u][xi][nu]);
            E* p = dst + (size_t)(xi * A + nu) * plane;
            if constexpr (CPT == 2) { *reinterpret_cast<uint32_t*>(p) = *reinterpret_cast<const uint32_t*>(v); }
            else { p[0] = v[0]; }
        }
}

template <int M, typename E>
static hipError_t launch_it_nhwc(const void* x, void* V, const Geom& g, const PreOp* pre, hipStream_t s) {
    const PreOp po = pre ? *pre : PreOp();
    const bool gn = po.stats != nullptr;
    // two fp16 channels per lane (4-byte accesses) when channel pairs never straddle C
    const bool pair = sizeof(E) == 2 && g.C % 2 == 0 && (reinterpret_cast<uintptr_t>(x) & 3u) == 0;
    const int cpt = pair ? 2 : 1;
    const size_t items = (size_t)g.T * (g.Cp / cpt);
    const size_t blocks = (items + 255) / 256;
    if (blocks > 0x3fffffffULL) return hipErrorInvalidValue;
    const int per_xcd = (int)((blocks + 7) / 8);
    dim3 block(256), grid((unsigned)per_xcd * 8);
    if (pair) {
        if constexpr (sizeof(E) == 2) {
            if (gn) hipLaunchKernelGGL((input_transform_nhwc_kernel<M, E, 2, true>), grid, block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, per_xcd, po);
            else     hipLaunchKernelGGL((input_transform_nhwc_kernel<M, E, 2, false>), grid, block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, per_xcd, po);
        }
    } else {
        if (gn) hipLaunchKernelGGL((input_transform_nhwc_kernel<M, E, 1, true>), grid, block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, per_xcd, po);
        else     hipLaunchKernelGGL((input_transform_nhwc_kernel<M, E, 1, false>), grid, block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, per_xcd, po);
    }
    return hipGetLastError();
}

template <int M, typename E, int CB, int TJ>
static hipError_t launch_it_cfg(const void* x, void* V, const Geom& g, const PreOp* pre, hipStream_t s) {
    const PreOp po = pre ? *pre : PreOp();
    const bool gn = po.stats != nullptr;
    const int strips = (g.tw + TJ - 1) / TJ;
    dim3 block(256), grid((unsigned)(g.N * g.th * strips), (unsigned)((g.Cp + CB - 1) / CB));
    // fast path: rows are whole 16-byte chunks and a 64-channel slab of x spans < 2 GB (32-bit lane offsets)
    const bool rows_are_chunks = ((size_t)g.W * sizeof(E)) % 16 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0 &&
                                 (size_t)CB * g.H * g.W * sizeof(E) < ((size_t)1 << 31);
    constexpr int STJ = 64 / (int)sizeof(E) / M;          // tiles per 64-byte body
    if (rows_are_chunks && g.Cp % 64 == 0) {
        const int steps = (g.tw + STJ / 2 + STJ - 1) / STJ;
        // Measured over the SD-shaped layers: with fp16 F(2x2) (16 tiles per body) the aligned fetch
        // alone pays from 16 tiles per row on; otherwise the strip kernel wins until a row has
        // eight steps.  Two steps per workgroup keep the grid large and the tail short.
        const bool wide_body = sizeof(E) == 2 && M == 2;
        const bool pays = wide_body ? g.tw >= STJ : steps >= 8;
        const int spb = steps >= 8 ? 2 : 1;
        const long long total = (long long)g.N * g.th * (g.Cp / 64) * ((steps + spb - 1) / spb);
        if (pays && total <= 0x3fffffffLL) {
            const int per_xcd = (int)((total + 7) / 8);
            if (gn) hipLaunchKernelGGL((input_transform_nchw_slide_kernel<M, E, STJ, true>), dim3((unsigned)(per_xcd * 8)), block, 0, s,
                                        (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, steps, spb, (int)total, per_xcd, po);
            else     hipLaunchKernelGGL((input_transform_nchw_slide_kernel<M, E, STJ, false>), dim3((unsigned)(per_xcd * 8)), block, 0, s,
                                        (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, steps, spb, (int)total, per_xcd, po);
            return hipGetLastError();
        }
    }
    if (rows_are_chunks) {
        const long long total = (long long)grid.x * grid.y;
        if (total > 0x3fffffffLL) return hipErrorInvalidValue;
        const int per_xcd = (int)((total + 7) / 8);
        const auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, strips,
                               (int)total, per_xcd, po);
        };
        if (po.up) { if (gn) run(input_transform_nchw_vec_kernel<M, E, CB, TJ, true, 1>); else run(input_transform_nchw_vec_kernel<M, E, CB, TJ, false, 1>); }
        else if (gn) run(input_transform_nchw_vec_kernel<M, E, CB, TJ, true, 0>);
        else run(input_transform_nchw_vec_kernel<M, E, CB, TJ, false, 0>);
    } else {
        const auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, block, 0, s, (const E*)x, (E*)V, g.N, g.C, g.H, g.W, g.th, g.tw, g.T, g.Cp, strips, po);
        };
        if constexpr (sizeof(E) == 2) {
            // (lane offsets of the pairs, of up to CB + 6 channels: 32-bit)
            if (g.W >> po.up >= 2 && (size_t)(CB + 6) * (g.H >> po.up) * (g.W >> po.up) * sizeof(E) < ((size_t)1 << 31)) {
                if (gn) run(input_transform_nchw_kernel<M, E, CB, TJ, true, true>);
                else run(input_transform_nchw_kernel<M, E, CB, TJ, false, true>);
                return hipGetLastError();
            }
        }
        if (gn) run(input_transform_nchw_kernel<M, E, CB, TJ, true, false>);
        else run(input_transform_nchw_kernel<M, E, CB, TJ, false, false>);
    }
    return hipGetLastError();
}

template <int M, typename E>
static hipError_t launch_it(const void* x, void* V, const Geom& g, const PreOp* pre, hipStream_t s) {
    constexpr int Q = 8 / M;      // TJ multiples that keep strips whole 16-byte chunks for fp16
    return launch_it_cfg<M, E, 64, 2 * Q>(x, V, g, pre, s);      // measured best of 1, 2, 4, 8 x Q tiles per strip
}

hipError_t launch_input_transform(const void* x, void* V, const Geom& g, int dt, bool nhwc, const PreOp* pre, hipStream_t s) {
    return with_dtype(dt, [&](auto* tag) {
        using E = std::remove_pointer_t<decltype(tag)>;
        if (nhwc) return g.m == 2 ? launch_it_nhwc<2, E>(x, V, g, pre, s) : launch_it_nhwc<4, E>(x, V, g, pre, s);
        return g.m == 2 ? launch_it<2, E>(x, V, g, pre, s) : launch_it<4, E>(x, V, g, pre, s);
    });
}

}  // namespace wino

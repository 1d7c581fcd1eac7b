// All three steps in one kernel for F(2x2,3x3), two-byte storage types (Section "Techniques"; its second paragraph argues for
// keeping dependent steps local): neither V nor the product M exists in memory.
//
// F(2x2) has 16 positions, so a compute unit's register file holds the product of ALL positions for a block of 32 tiles x
// 160 output channels (16 * 32 * 160 fp32 = 328 KB of 512 KB).  The reduction over channels can then be the OUTER loop:
// per 64 channels the workgroup stages the pixels of its tiles once, transforms them once into V for the 16 positions
// (64 KB of LDS), and multiplies them with the filter; step (iii) runs once at the end.  What this removes is the traffic
// that bounds the other paths, writing V (4x the bytes of x) and fetching it again for every block of output channels; what it costs
// is that every block of output channels repeats the activation transform, which is why the block is wide in that direction.
//
//   waves   eight: wave = (nu, half of the output channels); for each xi it multiplies position (xi, nu), so every wave works on
//           every xi and the sums over xi of step (iii) stay inside a lane
//   filter  1 KB transfers of whole 128-byte rows into a ring of three 2 KB slots private to the wave (no barrier, vmcnt only).
//           Fragments loaded straight into registers would cost 64 clocks per 1 KB: lanes 0..15 of a fragment are 16 different rows,
//           and the address unit takes one place per clock (16 bytes per clock and compute unit measured); 64-byte rows
//           fetch every 128-byte line twice (29 bytes per clock; whole lines 46-54)
//   pixels  fetched a chunk ahead into registers, converted (GroupNorm + SiLU applied once per pixel, fp32) into LDS while the
//           previous chunk is multiplied
// The block is 4 x 8 tiles of one image.  LDS: 46 KB pixels (fp32), 64 KB V, 48 KB filter ring.
#include "wino_internal.h"
#include "wino_mma.h"
#include "wino_transforms.h"

namespace wino {

namespace {

struct OnepassGeom { int N, C, H, W, K, th, tw; };

typedef f32x4_t f32x4_word_t __attribute__((aligned(4)));           // bias and vector need only be aligned to their elements
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// two elements in one word, rounded to nearest even; one instruction for bf16 (pack2 of wino_mma.h rounds alike; its users' code is ordered otherwise with this form)
template <typename E> __device__ __forceinline__ uint32_t convert2(float a, float b);
template <> __device__ __forceinline__ uint32_t convert2<__half>(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{a, b}), half2_t)); }
template <> __device__ __forceinline__ uint32_t convert2<bf16_t>(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{a, b}), bf16x2_t)); }
template <typename E> __device__ __forceinline__ float low16(uint32_t w) { const uint16_t h = (uint16_t)(w & 0xffffu); return to_f32<E>(*reinterpret_cast<const E*>(&h)); }
template <typename E> __device__ __forceinline__ float high16(uint32_t w) { const uint16_t h = (uint16_t)(w >> 16); return to_f32<E>(*reinterpret_cast<const E*>(&h)); }
template <> __device__ __forceinline__ float low16<bf16_t>(uint32_t w) { return __uint_as_float(w << 16); }
template <> __device__ __forceinline__ float high16<bf16_t>(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// LDS reads and writes issued so far have completed, then the workgroup barrier; transfers into LDS stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The same value, but not known to be: address arithmetic on it stays where it is used.  Hoisted out of the loop over the channels
// it would take more registers than the accumulators leave.
__device__ __forceinline__ int here(int v) { asm volatile("" : "+v"(v)); return v; }

// A pointer that is the same in every lane, in scalar registers
__device__ __forceinline__ const unsigned char* uniform(const unsigned char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
}

constexpr int XM_NHWC = 0, XM_NCHW_ROWS = 1, XM_NCHW_ANY = 2;
constexpr int onepass_most(int xm) { return xm == XM_NCHW_ANY ? 4 : 5; }        // element-wise pixel loads leave no registers for five sub-tiles

}  // namespace

// NS = 16-channel sub-tiles per wave: the block has 32 * NS output channels.
// XM: how x is read.  XM_NHWC: channel-last, 16-byte loads along the channels.  XM_NCHW_ROWS: rows of whole 16-byte pieces.
// XM_NCHW_ANY: any row length, and the 2x upsampling; element by element.
template <typename E, int NS, int XM>
__global__ void __launch_bounds__(512)
wino_onepass_f2_kernel(const E* __restrict__ x, const E* __restrict__ U, const float* __restrict__ bias, E* __restrict__ y,
                       OnepassGeom g, int tbh, int tbw, int total_blocks, int blocks_per_xcd, int row_ok, PreOp pre, PostOp post) {
    static_assert(sizeof(E) == 2, "two-byte storage types");
    constexpr int TH = 4, TW = 8, BT = TH * TW;           // tiles of the block
    constexpr int PH = 2 * TH + 2, PW = 2 * TW + 2, PX = PH * PW;      // pixels under them: 10 x 18
    constexpr int BK = 32 * NS;
    constexpr int PS = 66;                                // words per pixel: 64 channels and a shift of two banks per pixel
    constexpr int PATCH_BYTES = (PX * PS * 4 + 1023) / 1024 * 1024, V_BYTES = 16 * BT * 128, RING = 3, SLOT = 2048;
    constexpr int NX = XM == XM_NHWC ? 3 : (XM == XM_NCHW_ROWS ? 5 : 23);
    static_assert(PATCH_BYTES == 47 * 1024, "V and the ring start on a multiple of the swizzle period");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    float* patch = reinterpret_cast<float*>(lds);                      // [pixel][64 channels + 2]
    unsigned char* vbuf = lds + PATCH_BYTES;                           // [position][tile][64 channels], 16-byte chunks swizzled
    float* csc = reinterpret_cast<float*>(lds + PATCH_BYTES + V_BYTES + 8 * RING * SLOT);   // GroupNorm scale, then shift, of the chunk's channels
    float* csh = csc + 64;

    // one contiguous range of logical blocks per XCD; the tiles run fastest, so that the workgroups of an XCD share a filter slice
    const int logical = (int)(blockIdx.x % 8) * blocks_per_xcd + (int)(blockIdx.x / 8);
    if (logical >= total_blocks) return;                  // uniform, before any barrier
    const int ntb = g.N * tbh * tbw;
    const int kb = logical / ntb; int tb = logical - kb * ntb;
    const int bj = tb % tbw; tb /= tbw;
    const int bi = tb % tbh, n = tb / tbh;
    const int k0 = kb * BK, ti0 = bi * TH, tj0 = bj * TW;
    const int row0 = 2 * ti0 - 1, col0 = 2 * tj0 - 1;      // pixel at the corner of the patch

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nu = wave & 3, kh = wave >> 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_t*)lds;
    const int H = g.H, W = g.W, C = g.C, up = pre.up, Hs = H >> up, Ws = W >> up;
    const int nch = C >> 6;

    // ---- pixels: loads of the next chunk (into registers) and their conversion into `patch` ----------------------------
    const E* xn = x + (size_t)n * C * Hs * Ws;
    typedef typename std::conditional<XM == XM_NCHW_ANY, uint16_t, uint4>::type xreg_t;
    xreg_t xr[NX];
    float cg = 0.f, cb = 0.f, cm = 0.f, cr = 0.f;          // GroupNorm parameters of channel `lane` of the chunk (first wave)
    const bool has_pre = pre.stats != nullptr;
    // channel-last: the addresses of a lane's pieces (eight channels of one pixel) do not change from chunk to chunk
    uint32_t xoff[XM == XM_NHWC ? NX : 1];
    uint32_t xin = 0u;                                    // bit j: piece j lies inside the image
    if constexpr (XM == XM_NHWC) {
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int px = min((tid + 512 * j) >> 3, PX - 1);
            const int r = row0 + px / PW, c = col0 + px % PW;
            xoff[j] = (((uint32_t)(min(max(r, 0), H - 1) >> up) * (uint32_t)Ws + (uint32_t)(min(max(c, 0), W - 1) >> up)) * (uint32_t)C +
                       (uint32_t)((tid & 7) * 8)) * 2u;
            xin |= (r >= 0 && r < H && c >= 0 && c < W) ? 1u << j : 0u;
        }
    }
    auto load_pixels = [&](int ch) __attribute__((always_inline)) {
        const int c0 = ch * 64, tid = here(threadIdx.x);
        if constexpr (XM == XM_NHWC) {
#pragma unroll
            for (int j = 0; j < NX; ++j)
                xr[j] = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(xn + c0) + xoff[j]);
        } else if constexpr (XM == XM_NCHW_ROWS) {
            // 4 pieces of a row (8 columns left of the block's 16, the 16, 8 right of them) x 64 channels x 10 rows
            const int cl = (tid >> 2) & 63;
            const uint32_t lane0 = (uint32_t)cl * (uint32_t)(H * W) + (uint32_t)min(max(16 * bj - 8 + 8 * (tid & 3), 0), W - 8);
            const unsigned char* xc = reinterpret_cast<const unsigned char*>(xn + (size_t)c0 * H * W);
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                const int r = min(max(row0 + 2 * j + (tid >> 8), 0), H - 1);
                xr[j] = *reinterpret_cast<const uint4*>(xc + (lane0 + (uint32_t)(r * W)) * 2u);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                const int e = min(tid + 512 * j, 64 * PX - 1);
                const int cl = e / PX, px = e % PX;
                const int r = min(max(row0 + px / PW, 0), H - 1) >> up, c = min(max(col0 + px % PW, 0), W - 1) >> up;
                xr[j] = *reinterpret_cast<const uint16_t*>(reinterpret_cast<const unsigned char*>(xn + (size_t)c0 * Hs * Ws) +
                                                           ((uint32_t)((cl * Hs + r) * Ws) + (uint32_t)c) * 2u);
            }
        }
        if (has_pre && tid < 64) {
            const int c = c0 + tid;
            const float* st = pre.stats + ((size_t)n * pre.groups + c / pre.cpg) * 2;
            cm = st[0]; cr = st[1]; cg = pre.gamma[c]; cb = pre.beta[c];
        }
    };
    auto put_constants = [&]() __attribute__((always_inline)) {          // same arithmetic as pre_lane
        if (has_pre && tid < 64) { const float sc = cg * cr; csc[tid] = sc; csh[tid] = cb - cm * sc; }
    };
    auto silu = [&](float v, float sc, float sh) __attribute__((always_inline)) { return pre_apply_as<E>(v, PreLane{sc, sh, true}, true); };
    auto convert = [&](int j) __attribute__((always_inline)) {
        const int tid = here(threadIdx.x);
        if constexpr (XM == XM_NHWC) {
            const int px = (tid + 512 * j) >> 3;
            const bool in = (xin >> j) & 1u;
            float v[8] = {low16<E>(xr[j].x), high16<E>(xr[j].x), low16<E>(xr[j].y), high16<E>(xr[j].y),
                          low16<E>(xr[j].z), high16<E>(xr[j].z), low16<E>(xr[j].w), high16<E>(xr[j].w)};
            if (has_pre) {
                float sc[8], sh[8];
                *reinterpret_cast<float4*>(sc) = *reinterpret_cast<const float4*>(csc + (tid & 7) * 8);
                *reinterpret_cast<float4*>(sc + 4) = *reinterpret_cast<const float4*>(csc + (tid & 7) * 8 + 4);
                *reinterpret_cast<float4*>(sh) = *reinterpret_cast<const float4*>(csh + (tid & 7) * 8);
                *reinterpret_cast<float4*>(sh + 4) = *reinterpret_cast<const float4*>(csh + (tid & 7) * 8 + 4);
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = silu(v[u], sc[u], sh[u]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = in ? v[u] : 0.f;
            if (px < PX) {
                float* dst = patch + px * PS + (tid & 7) * 8;
#pragma unroll
                for (int u = 0; u < 4; ++u) *reinterpret_cast<float2*>(dst + 2 * u) = make_float2(v[2 * u], v[2 * u + 1]);
            }
        } else if constexpr (XM == XM_NCHW_ROWS) {
            // of the four pieces of a row the middle two are wanted whole and one element of each outer one: the lanes of the outer pieces
            // take over half of their neighbour's elements
            const int cl = (tid >> 2) & 63, pc = tid & 3, pr = 2 * j + (tid >> 8);
            const int r = row0 + pr, cc = pc < 2 ? col0 : col0 + PW - 1;
            const bool rin = r >= 0 && r < H;
            const bool in = rin && (pc < 2 || 16 * bj + 8 < W);           // half of an inner piece
            const bool ein = rin && cc >= 0 && cc < W;                    // border column (lanes 0 and 3)
            const uint32_t border = pc == 0 ? xr[j].w >> 16 : xr[j].x & 0xffffu;
            uint32_t w[4] = {xr[j].x, xr[j].y, xr[j].z, xr[j].w};
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = __builtin_amdgcn_update_dpp(w[u], w[u], 0xa5, 0xf, 0xf, true);      // quad_perm: lanes 1, 1, 2, 2
            const uint32_t w0 = pc & 1 ? w[2] : w[0], w1 = pc & 1 ? w[3] : w[1];
            float v[5] = {low16<E>(w0), high16<E>(w0), low16<E>(w1), high16<E>(w1), low16<E>(border)};
            if (has_pre) {
                const float sc = csc[cl], sh = csh[cl];
#pragma unroll
                for (int u = 0; u < 5; ++u) v[u] = silu(v[u], sc, sh);
            }
            float* dst = patch + (pr * PW + 1 + 4 * pc) * PS + cl;
#pragma unroll
            for (int u = 0; u < 4; ++u) dst[u * PS] = in ? v[u] : 0.f;
            if (pc == 0 || pc == 3) patch[(pr * PW + (pc == 0 ? 0 : PW - 1)) * PS + cl] = ein ? v[4] : 0.f;
        } else {
            const int e = tid + 512 * j;
            const int cl = e / PX, px = e % PX;
            const int r = row0 + px / PW, c = col0 + px % PW;
            const bool in = r >= 0 && r < H && c >= 0 && c < W;
            float v = to_f32<E>(*reinterpret_cast<const E*>(&xr[j]));
            if (has_pre) v = silu(v, csc[cl & 63], csh[cl & 63]);
            if (e < 64 * PX) patch[px * PS + cl] = in ? v : 0.f;
        }
    };

    // ---- step (i): patch -> V.  A lane owns two neighbouring tiles of a tile row and two channels ----------------------
    auto transform = [&]() __attribute__((always_inline)) {
        const int tid = here(threadIdx.x);
        const int cp = tid & 31, tp = tid >> 5;
        const int tr = tp >> 2, tc = (tp & 3) * 2;
        float2 tmp[4][4];                                 // [xi][column % 4]
        const float* src = patch + (2 * tr * PW + 2 * tc) * PS + 2 * cp;
        auto column = [&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value;
            float2 d[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) d[a] = *reinterpret_cast<const float2*>(src + (a * PW + b) * PS);
            tmp[0][b & 3] = make_float2(d[0].x - d[2].x, d[0].y - d[2].y);
            tmp[1][b & 3] = make_float2(d[1].x + d[2].x, d[1].y + d[2].y);
            tmp[2][b & 3] = make_float2(d[2].x - d[1].x, d[2].y - d[1].y);
            tmp[3][b & 3] = make_float2(d[1].x - d[3].x, d[1].y - d[3].y);
        };
        auto tile = [&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            const int t = tr * TW + tc + u;
            unsigned char* dst = vbuf + t * 128 + (((cp >> 2) ^ ((t >> 1) & 7)) << 4) + (cp & 3) * 4;
#pragma unroll
            for (int xi = 0; xi < 4; ++xi) {
                const float2 d0 = tmp[xi][2 * u], d1 = tmp[xi][2 * u + 1], d2 = tmp[xi][(2 * u + 2) & 3], d3 = tmp[xi][(2 * u + 3) & 3];
                uint32_t* p = reinterpret_cast<uint32_t*>(dst + xi * 4 * BT * 128);
                p[0 * BT * 32] = convert2<E>(d0.x - d2.x, d0.y - d2.y);
                p[1 * BT * 32] = convert2<E>(d1.x + d2.x, d1.y + d2.y);
                p[2 * BT * 32] = convert2<E>(d2.x - d1.x, d2.y - d1.y);
                p[3 * BT * 32] = convert2<E>(d1.x - d3.x, d1.y - d3.y);
            }
        };
        static_for<4>(column);
        tile(std::integral_constant<int, 0>());
        __builtin_amdgcn_sched_barrier(0);                // the first tile's columns are done with before the last two are read
        column(std::integral_constant<int, 4>());
        column(std::integral_constant<int, 5>());
        tile(std::integral_constant<int, 1>());
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- filter ring: slot q of a chunk = sub-tile (q % NS) of position (q / NS, nu) -----------------------------------------
    const uint32_t row_bytes = (uint32_t)C * 2u;
    uint32_t uoff[2];                                     // rows 0..7 and 8..15 of a sub-tile, chunk swizzled by the row
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = i * 8 + (lane >> 3);
        uoff[i] = (uint32_t)row * row_bytes + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
    const uint32_t ring0 = lds0 + PATCH_BYTES + V_BYTES + (uint32_t)wave * (RING * SLOT);
    // byte offsets of the sub-tiles; those beyond K repeat the last one (K is a multiple of 16), their results are never stored
    uint32_t koff[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) koff[s] = (uint32_t)(min(k0 + kh * (16 * NS) + s * 16, g.K - 16) - k0) * row_bytes;
    const size_t plane4 = (size_t)4 * g.K * row_bytes;
    const unsigned char* ucur = reinterpret_cast<const unsigned char*>(U) + ((size_t)nu * g.K + k0) * row_bytes;     // position (xi, nu) of the slot being issued
    // the next slot in order (q = its number in the chunk), into ring slot `slot`
    auto issue = [&](auto qc, int slot) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, s = q % NS;
        const unsigned char* base = uniform(ucur + koff[s]);
        const uint32_t dst = ring0 + (uint32_t)slot * SLOT;
        dma_load_1k_s(base, uoff[0], dst);
        dma_load_1k_s(base, uoff[1], dst + 1024u);
        if constexpr (s == NS - 1) ucur += q == 4 * NS - 1 ? 128 - (ptrdiff_t)(3 * plane4) : (ptrdiff_t)plane4;
    };
    constexpr int NQ = 4 * NS;                            // slots per chunk

    f32x4_t acc[4][NS][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[a][s][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int frow = lane & 15, fq = lane >> 4;
    const uint32_t ufrag = ring0 + (uint32_t)frow * 128u + (uint32_t)((fq ^ ((frow >> 1) & 7)) << 4);          // step 1: chunk + 4, i.e. ^ 64
    const uint32_t vfrag = lds0 + PATCH_BYTES + (uint32_t)(nu * BT + frow) * 128u + (uint32_t)((fq ^ ((frow >> 1) & 7)) << 4);
    u32x4_t uf[3][2], vf[2][2];                           // filter [set][step]; activation [tile sub-tile][step]
    auto read_filter = [&](int slot, auto setc) __attribute__((always_inline)) {
        constexpr int set = decltype(setc)::value;
        const uint32_t a = ufrag + (uint32_t)slot * SLOT;
        lds_read16_async<0>(uf[set][0], a);
        lds_read16_async<0>(uf[set][1], a ^ 64u);
    };
    auto read_v = [&](auto xic) __attribute__((always_inline)) {
        constexpr int xi = decltype(xic)::value;
        lds_read16_async<xi * 4 * BT * 128>(vf[0][0], vfrag);
        lds_read16_async<xi * 4 * BT * 128>(vf[0][1], vfrag ^ 64u);
        lds_read16_async<xi * 4 * BT * 128 + 16 * 128>(vf[1][0], vfrag);
        lds_read16_async<xi * 4 * BT * 128 + 16 * 128>(vf[1][1], vfrag ^ 64u);
    };

    load_pixels(0);
    static_for<3>([&](auto qc) { issue(qc, decltype(qc)::value); });
    put_constants();
    lds_barrier();
#pragma unroll
    for (int j = 0; j < NX; ++j) convert(j);
    lds_barrier();

    int slot = 0;                                         // ring slot of the chunk's slot 0
    for (int ch = 0; ch < nch; ++ch) {
        const bool more = ch + 1 < nch;
        if (more) load_pixels(ch + 1);
        transform();
        put_constants();
        lds_barrier();                                    // V and the constants are complete; `patch` is free
        // The pixels of the next chunk have arrived from here on (the compiler would otherwise wait for them, and with them for
        // every transfer of the ring, in front of each conversion).
        if (more) {
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                if constexpr (XM == XM_NCHW_ANY) asm volatile("" : "+v"(xr[j]));
                else asm volatile("" : "+v"(xr[j].x), "+v"(xr[j].y), "+v"(xr[j].z), "+v"(xr[j].w));
            }
        }
        // Slot q multiplies fragments requested two slots earlier.  Meanwhile slot q+2, whose transfer has to have landed, is read
        // and, once the fragments of slot q+1 have arrived, that slot is refilled with slot q+4.  Transfers land in order, so
        // slot q+2 is complete when only the two transfers of slot q+3 are outstanding.
        wait_vmcnt<4>();
        read_filter(slot, std::integral_constant<int, 0>());
        read_v(std::integral_constant<int, 0>());
        wait_vmcnt<2>();
        read_filter(slot + 1 >= RING ? slot + 1 - RING : slot + 1, std::integral_constant<int, 1>());
        lds_wait<2>();
        pin(uf[0][0]); pin(uf[0][1]); pin(vf[0][0]); pin(vf[0][1]); pin(vf[1][0]); pin(vf[1][1]);
        issue(std::integral_constant<int, 3>(), slot);
        static_for<NQ>([&](auto qc) {
            constexpr int q = decltype(qc)::value, xi = q / NS, s = q % NS, set = q % 3;
            const int next = slot + 1 == RING ? 0 : slot + 1, next2 = next + 1 == RING ? 0 : next + 1;
            if constexpr (q + 2 < NQ) {
                if constexpr (q + 3 >= NQ) {              // slot q+3 exists only if another chunk follows
                    if (more) wait_vmcnt<2>(); else wait_vmcnt<0>();
                } else wait_vmcnt<2>();
                read_filter(next2, std::integral_constant<int, (q + 2) % 3>());
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                Mma16<E>::run(uf[set][h], vf[0][h], acc[xi][s][0]);
                Mma16<E>::run(uf[set][h], vf[1][h], acc[xi][s][1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (q + 1 < NQ) {
                constexpr bool turn = (q + 1) % NS == 0;  // the next slot belongs to the next xi
                if constexpr (turn) read_v(std::integral_constant<int, (q + 1) / NS>());
                // a share of the next chunk's conversion
                constexpr int per = XM == XM_NCHW_ANY ? (NX + NQ - 2) / (NQ - 1) : 1;
                if constexpr (q * per < NX) {
                    if (more) {
#pragma unroll
                        for (int u = 0; u < per; ++u) if (q * per + u < NX) convert(q * per + u);
                    }
                }
                // everything but the two youngest reads (slot q+2); conversions and V are younger than those: wait for all then
                if constexpr (turn || q * per < NX || q + 2 >= NQ) lds_wait<0>();
                else lds_wait<2>();
                pin(uf[(q + 1) % 3][0]); pin(uf[(q + 1) % 3][1]);
                if constexpr (turn) { pin(vf[0][0]); pin(vf[0][1]); pin(vf[1][0]); pin(vf[1][1]); }
                if constexpr (q + 4 < NQ) issue(std::integral_constant<int, q + 4>(), next);
                else if (more) issue(std::integral_constant<int, q + 4 - NQ>(), next);
                slot = next;
            }
        });
        slot = slot + 1 == RING ? 0 : slot + 1;
        lds_barrier();                                    // `patch` holds the next chunk; V is free
    }

    // ---- step (iii): the sums over xi inside the lane, the sums over nu through LDS, one row of the 2x2 outputs at a time.  A lane
    // then owns 16 bytes of y: eight channels of a pixel (channel-last) or eight pixels of an image row (four tiles).
    constexpr int ZS = XM == XM_NHWC ? BK + 4 : BT + 4;   // words per row of the exchanged sums, [nu][tile][k] or [nu][k][tile]
    constexpr int ZN = (XM == XM_NHWC ? BT : BK) * ZS;    // words per nu
    float* z = reinterpret_cast<float*>(lds);
    static_assert(4 * ZN * 4 <= PATCH_BYTES + V_BYTES + 8 * RING * SLOT, "the exchanged sums fit");
    const E* res = static_cast<const E*>(post.residual);
    const int K = g.K;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (a) lds_barrier();
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const f32x4_t v = a == 0 ? acc[0][s][t] + acc[1][s][t] + acc[2][s][t] : acc[1][s][t] - acc[2][s][t] - acc[3][s][t];
                const int kl = kh * (16 * NS) + s * 16 + 4 * fq, tl = t * 16 + frow;
                if constexpr (XM == XM_NHWC) {
                    *reinterpret_cast<f32x4_t*>(z + nu * ZN + tl * ZS + kl) = v;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) z[nu * ZN + (kl + r) * ZS + tl] = v[r];
                }
            }
        lds_barrier();
        constexpr int ITEMS = BK * BT / (XM == XM_NHWC ? 8 : 4);
        for (int idx = tid; idx < ITEMS; idx += 512) {
            if constexpr (XM == XM_NHWC) {
                const int kl = idx % (BK / 8) * 8, t = idx / (BK / 8);
                const int k = k0 + kl, i = 2 * (ti0 + t / TW) + a, j = 2 * (tj0 + t % TW);
                if (k >= K || i >= H || j >= W) continue;              // K is a multiple of 16: the eight channels are all inside
                float o0[8], o1[8];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float* zp = z + t * ZS + kl + 4 * h;
                    const f32x4_t s0 = *reinterpret_cast<const f32x4_t*>(zp), s1 = *reinterpret_cast<const f32x4_t*>(zp + ZN);
                    const f32x4_t s2 = *reinterpret_cast<const f32x4_t*>(zp + 2 * ZN), s3 = *reinterpret_cast<const f32x4_t*>(zp + 3 * ZN);
                    f32x4_t bb = {0.f, 0.f, 0.f, 0.f};
                    if (bias) bb = *reinterpret_cast<const f32x4_word_t*>(bias + k + 4 * h);
                    if (post.addvec) bb += *reinterpret_cast<const f32x4_word_t*>(post.addvec + (size_t)n * K + k + 4 * h);
                    *reinterpret_cast<f32x4_t*>(o0 + 4 * h) = s0 + s1 + s2 + bb;
                    *reinterpret_cast<f32x4_t*>(o1 + 4 * h) = s1 - s2 - s3 + bb;
                }
                const size_t o = (((size_t)n * H + i) * W + j) * K + k;
                auto put = [&](const float* v, size_t at) __attribute__((always_inline)) {
                    uint4 w = make_uint4(0u, 0u, 0u, 0u);
                    if (res) w = *reinterpret_cast<const uint4*>(res + at);
                    w.x = convert2<E>(v[0] + low16<E>(w.x), v[1] + high16<E>(w.x)); w.y = convert2<E>(v[2] + low16<E>(w.y), v[3] + high16<E>(w.y));
                    w.z = convert2<E>(v[4] + low16<E>(w.z), v[5] + high16<E>(w.z)); w.w = convert2<E>(v[6] + low16<E>(w.w), v[7] + high16<E>(w.w));
                    *reinterpret_cast<uint4*>(y + at) = w;
                };
                put(o0, o);
                if (j + 1 < W) put(o1, o + K);
            } else {
                const int tl = idx % (BT / 4) * 4, kl = idx / (BT / 4);
                const int k = k0 + kl, i = 2 * (ti0 + tl / TW) + a, j = 2 * (tj0 + tl % TW);
                if (k >= K || i >= H || j >= W) continue;
                const float* zp = z + kl * ZS + tl;
                const f32x4_t s0 = *reinterpret_cast<const f32x4_t*>(zp), s1 = *reinterpret_cast<const f32x4_t*>(zp + ZN);
                const f32x4_t s2 = *reinterpret_cast<const f32x4_t*>(zp + 2 * ZN), s3 = *reinterpret_cast<const f32x4_t*>(zp + 3 * ZN);
                const float bb = (bias ? bias[k] : 0.f) + (post.addvec ? post.addvec[(size_t)n * K + k] : 0.f);
                const f32x4_t v0 = s0 + s1 + s2 + bb, v1 = s1 - s2 - s3 + bb;          // even and odd columns of the four tiles
                const size_t o = (((size_t)n * K + k) * H + i) * W + j;
                if (row_ok) {                                                          // eight pixels, 16-byte aligned, inside the row
                    uint4 w = make_uint4(0u, 0u, 0u, 0u);
                    if (res) w = *reinterpret_cast<const uint4*>(res + o);
                    w.x = convert2<E>(v0[0] + low16<E>(w.x), v1[0] + high16<E>(w.x)); w.y = convert2<E>(v0[1] + low16<E>(w.y), v1[1] + high16<E>(w.y));
                    w.z = convert2<E>(v0[2] + low16<E>(w.z), v1[2] + high16<E>(w.z)); w.w = convert2<E>(v0[3] + low16<E>(w.w), v1[3] + high16<E>(w.w));
                    *reinterpret_cast<uint4*>(y + o) = w;
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (j + 2 * u < W) y[o + 2 * u] = from_f32<E>(v0[u] + (res ? to_f32<E>(res[o + 2 * u]) : 0.f));
                        if (j + 2 * u + 1 < W) y[o + 2 * u + 1] = from_f32<E>(v1[u] + (res ? to_f32<E>(res[o + 2 * u + 1]) : 0.f));
                    }
                }
            }
        }
    }
}

template <typename E, int NS, int XM>
static hipError_t launch_onepass_cfg(const void* x, const void* U, const float* bias, void* y, const Geom& g, const PreOp& pre,
                                     const PostOp& post, hipStream_t s) {
    constexpr int lds_bytes = 47 * 1024 + 16 * 32 * 128 + 8 * 3 * 2048 + 64 * 8;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    auto kern = wino_onepass_f2_kernel<E, NS, XM>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    const int tbh = (g.th + 3) / 4, tbw = (g.tw + 7) / 8;
    const long long total = (long long)g.N * tbh * tbw * ((g.K + 32 * NS - 1) / (32 * NS));
    if (total > 0x3fffffffLL) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    const int row_ok = g.W % 8 == 0 && ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(post.residual)) & 15u) == 0;
    const OnepassGeom og{g.N, g.C, g.H, g.W, g.K, g.th, g.tw};
    hipLaunchKernelGGL(kern, dim3((unsigned)(per_xcd * 8)), dim3(512), lds_bytes, s, (const E*)x, (const E*)U, bias, (E*)y, og, tbh, tbw,
                       (int)total, per_xcd, row_ok, pre, post);
    return hipGetLastError();
}

// Microseconds of the kernel with NS sub-tiles per wave, fitted to 548 measured calls (64...1280 channels, 24x24...520x520, both layouts, with
// and without GroupNorm and upsampling; off by 7 % channel-last, 10 % NCHW, 14 % element by element): workgroups come in rounds of 256; a
// round takes start and end, and per chunk of 64 channels a time for pixels, transform and barriers plus one per sub-tile.
struct OnepassTimes { double ends, pixels[2], subtile[2]; };             // [GroupNorm]
static double onepass_us(const Geom& g, int xm, bool gn, int ns) {
    static const OnepassTimes times[3] = {{2.9, {0.52, 1.81}, {1.05, 1.01}}, {2.3, {1.52, 2.15}, {1.12, 1.16}}, {7.8, {3.1, 3.4}, {1.48, 2.0}}};
    const long long wgs = (long long)g.N * ((g.th + 3) / 4) * ((g.tw + 7) / 8) * ((g.K + 32 * ns - 1) / (32 * ns));
    const OnepassTimes& t = times[xm];
    return 3.0 + (double)((wgs + 255) / 256) * (t.ends + (g.C / 64) * (t.pixels[gn] + t.subtile[gn] * ns));
}

// ... and of the paths that store V, fitted the same way, with 200 more calls of up to 540 000 pixels (12 % and 8 %).  Chain: V and M through
// memory, at more per byte where the two are larger than the 256 MB memory-side cache, and the products.  Fused variant: the transform, then
// rounds of its blocks, each a serial chain of 16 positions; block shapes as fused_pick_shape() takes them.  Channel-last, V beyond 100 MB
// costs it more (256 channels at 512x512 379 NCHW, 446 channel-last).  It reads a residual in 2.1 (NCHW) to 3.5 us per million outputs, this
// kernel in 0.5.
static double stored_us(const Geom& g, bool ragged, bool gn, bool nhwc, bool residual, bool fused_variant) {
    const double T = g.T, C = g.C, TC = T * C;
    if (!fused_variant) {
        const double K = g.K < 128 ? 128.0 : (double)g.K, far = T * (32.0 * C + 64.0 * K) - 219e6;
        return (12.5 + T * (8.15e-6 * C + 1.76e-5 * K + 3.6e-8 * C * K) + (gn ? 3.3e-6 * TC : 0.0) + (far > 0.0 ? 7.7e-8 * far : 0.0)) *
               (ragged ? 1.06 : 1.0);
    }
    auto blocks = [&](int bk, int bt) { return (double)((g.K + bk - 1) / bk) * (double)((g.T + bt - 1) / bt); };
    auto rounds = [](double n) { const double most = (double)(((long long)n + 255) / 256), r = 0.3 * n / 256.0 + 0.7 * most; return r < 1.0 ? 1.0 : r; };
    const double stages = 16.0 * (g.C / 64), b128 = blocks(128, 128), b64 = g.K < g.T ? blocks(128, 64) : blocks(64, 128), small = blocks(64, 64) / 512.0;
    const double gemm = b128 >= 160 ? rounds(b128) * (22.9 + 0.542 * stages) : (b64 >= 200 ? rounds(b64) * (16.8 + 0.332 * stages) : (small < 1.0 ? 1.0 : small) * (15.8 + 0.238 * stages));
    const double last = nhwc ? 0.3e-6 * TC + (TC > 3.3e6 ? 5.2e-6 * (TC - 3.3e6) : 0.0) : 0.0;
    return 3.0 + 7.8e-6 * TC * (ragged ? 1.44 : 1.0) + gemm + last + (gn ? (nhwc ? 3.65e-6 : 4.4e-6) * TC : 0.0) +
           (residual ? (nhwc ? 3.0e-6 : 1.7e-6) * g.N * g.H * (double)g.W * g.K : 0.0);
}

// Whether it applies and is taken, and how.  It applies to whole 128-byte reduction stages and whole 16-channel sub-tiles, and is taken
// where it is faster than the paths that store V, by the times above: over the measured calls 0.5 % more than the better one each time.  One
// kernel / the other path (us; chain, and with (f) the fused variant): NCHW 320 channels at 128x128 80 / 111, with GroupNorm 92 / 128, (f)
// 92 / 103; at 64x64 30 / 35, 640 channels at 64x64 with GroupNorm 93 / 88, 512 at 256x256 with GroupNorm 487 / 433; channel-last 320 at
// 64x64 25 / 34, with GroupNorm (f) 36 / 51, 512 at 256x256 337 / 389, 256 at 512x512 (f) 357 / 446, 640 -> 320 at 96x96 110 / 87, 192 -> 320
// at 128x312 with GroupNorm and residual (f) 83 / 119; element by element 64 -> 128 at 250x250
// 47 / 62, (f) 46 / 33, 128 -> 128 at 300x300 93 / 121, (f) 91 / 80, 192 -> 96 at 500x300 (f) 164 / 198, 256 -> 256 at 250x250 with GroupNorm
// 226 / 204, (f) 227 / 126, 320 -> 320 at 52x78 (N=2) with GroupNorm 69 / 46.
OnepassPlan onepass_plan(const void* x, const Geom& g, int dt, bool nhwc, bool fused_variant, const PreOp* pre, bool residual) {
    const OnepassPlan none{0, 0};
    if (!(two_byte(dt) && dt != DT_I8 && g.m == 2 && g.C % 64 == 0 && g.K % 16 == 0)) return none;
    if ((size_t)g.C * g.H * g.W >= ((size_t)1 << 31)) return none;             // byte offsets inside an image are 32-bit
    if ((size_t)g.K * g.C * 2 >= ((size_t)1 << 31)) return none;               // byte offsets inside a position of U too
    const bool gn = pre && pre->stats, up = pre && pre->up, rows = g.W % 8 == 0 && !up && (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    const int xm = nhwc ? XM_NHWC : (rows ? XM_NCHW_ROWS : XM_NCHW_ANY);
    OnepassPlan plan{2, xm};
    for (int ns = 3; ns <= onepass_most(xm); ++ns)
        if (onepass_us(g, xm, gn, ns) < onepass_us(g, xm, gn, plan.ns)) plan.ns = ns;
    return onepass_us(g, xm, gn, plan.ns) < 0.93 * stored_us(g, xm == XM_NCHW_ANY && !up, gn, nhwc, residual, fused_variant) ? plan : none;
}

template <typename E, int XM>
static hipError_t launch_onepass_t(const void* x, const void* U, const float* bias, void* y, const Geom& g, const PreOp& pre,
                                   const PostOp& post, int ns, hipStream_t s) {
    switch (ns) {
        case 2: return launch_onepass_cfg<E, 2, XM>(x, U, bias, y, g, pre, post, s);
        case 3: return launch_onepass_cfg<E, 3, XM>(x, U, bias, y, g, pre, post, s);
        case 4: return launch_onepass_cfg<E, 4, XM>(x, U, bias, y, g, pre, post, s);
        default: break;
    }
    if constexpr (onepass_most(XM) == 5)
        if (ns == 5) return launch_onepass_cfg<E, 5, XM>(x, U, bias, y, g, pre, post, s);
    return hipErrorInvalidValue;
}

hipError_t launch_onepass_conv(const void* x, const void* U, const float* bias, void* y, const Geom& g, int dt, const OnepassPlan& plan,
                               const PreOp* prep, const PostOp* postp, hipStream_t s) {
    const PreOp pre = prep ? *prep : PreOp();
    const PostOp post = postp ? *postp : PostOp();
    auto run = [&](auto* tag) {
        using E = std::remove_pointer_t<decltype(tag)>;
        switch (plan.xm) {
            case XM_NHWC: return launch_onepass_t<E, XM_NHWC>(x, U, bias, y, g, pre, post, plan.ns, s);
            case XM_NCHW_ROWS: return launch_onepass_t<E, XM_NCHW_ROWS>(x, U, bias, y, g, pre, post, plan.ns, s);
            default: return launch_onepass_t<E, XM_NCHW_ANY>(x, U, bias, y, g, pre, post, plan.ns, s);
        }
    };
    return dt == DT_F16 ? run(static_cast<__half*>(nullptr)) : run(static_cast<bf16_t*>(nullptr));
}

}  // namespace wino

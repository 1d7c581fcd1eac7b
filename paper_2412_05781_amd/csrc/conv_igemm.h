// Declarations shared by the implicit-GEMM convolution sources (conv_igemm.hip, conv_igemm_tile.hip).
#pragma once
#include "wino_internal.h"
#include "wino_mma.h"

namespace wino {

typedef int rsrc_t __attribute__((ext_vector_type(4)));
// Descriptor for buffer loads of at most 2 GB from `base` on.  A lane whose offset is kOutside lies beyond its range whatever scalar offset
// is added, and reads zeros; every other lane's offset is inside the operand.
constexpr uint32_t kOutside = 0x80000000u, kRange = 0x7fffffffu;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    rsrc_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = (int)kRange;
    r[3] = 0x00020000;
    return r;
}
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 1 KB to LDS: a wave-uniform descriptor and byte offset, a byte offset per lane; a lane outside the range writes zeros
__device__ __forceinline__ void dma_buffer_1k(rsrc_t r, uint32_t lane_off, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_addr), "v"(lane_off), "s"(r), "s"(__builtin_amdgcn_readfirstlane(off)) : "memory", "m0");
}
#pragma clang diagnostic pop

struct ConvGeom {
    int N, C, Cp, H, W, K, R, st, pad, Ho, Wo, T;      // T = N*Ho*Wo output pixels
    int up, Hs, Ws;                                    // up = 1: x is stored at Hs x Ws = H/2 x W/2 and read upsampled
};
// Optional additions in the epilogue (fp32, before the one rounding): a per-(image, channel) vector and a
// tensor of y's shape and layout.
struct IgemmPost {
    const float* addvec = nullptr;    // [N][K]
    const void* residual = nullptr;   // like y
    float scale = 1.f;                // the accumulated sum is multiplied by this first (quantised operands: 1 / (sx * sw))
};

// The 16x16-tile kernel (conv_igemm_tile.hip): two-byte storage types, Cp a whole number of 128-byte stages.
// igemm_block_plan: its choice of block and of the number of reduction ranges, at most most_sp; id < 0: left to the kernels of conv_igemm.hip.
// igemm_tile_ranges: the number of ranges that a workspace is sized for, 0: igemm_split_rule says.
struct IgemmTilePlan { int id, split; };
IgemmTilePlan igemm_block_plan(int T, int HoWo, int K, int Cp, int R, int dt, bool nhwc, int most_sp);
double igemm_block_time(int id, int T, int HoWo, int K, int Cp, int R, bool nhwc, int split);      // the times it compares
bool igemm_tile_fits(const ConvGeom& g);                               // the operands are small enough for the kernel's offsets
int igemm_split_rule(int T, int K, int Cp, int R, int dt);             // ranges where the 16x16-tile kernel does not apply (conv_igemm.hip)
int igemm_tile_ranges(int T, int HoWo, int K, int Cp, int R, int dt, bool nhwc);
// The blocks of conv_igemm.hip, pixels x output channels.
struct IgemmShape { int tp, tk; };
IgemmShape igemm_shape(int T, int K);
hipError_t launch_igemm_tile(const void* xh, const void* Wr, const float* bias, void* y, float* part, const IgemmTilePlan& plan,
                             const ConvGeom& g, const IgemmPost& post, int dt, bool nhwc, hipStream_t s);

// Shared by the kernels with two-byte outputs whose block rows are the contiguous dimension of y: four consecutive rows ra .. ra+3 of
// column cb.  PIX_A: rows are pixels (NCHW y), else output channels (channel-last y; `planes`: an NCHW y with an odd number of pixels,
// whose outputs are stored one by one).  Additions in fp32, one rounding.
template <typename E, bool PIX_A>
__device__ __forceinline__ void igemm_store4(f32x4_t v, int ra, int cb, E* __restrict__ y, const float* __restrict__ bias, const ConvGeom& g,
                                             const IgemmPost& post, int vec_ok, int planes) {
    const int howo = g.Ho * g.Wo, rows_a = PIX_A ? g.T : g.K;
    if (ra >= rows_a || cb >= (PIX_A ? g.K : g.T)) return;
    if (vec_ok) {                                   // the four outputs are adjacent and 8-byte aligned
        size_t o;
        if constexpr (PIX_A) {
            const int n = ra / howo, k = cb;
            o = ((size_t)n * g.K + k) * howo + (ra - n * howo);
            v = v * post.scale + ((bias ? bias[k] : 0.f) + (post.addvec ? post.addvec[(size_t)n * g.K + k] : 0.f));
        } else {
            const int n = post.addvec ? cb / howo : 0;
            o = (size_t)cb * g.K + ra;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[r] = v[r] * post.scale + ((bias ? bias[ra + r] : 0.f) + (post.addvec ? post.addvec[(size_t)n * g.K + ra + r] : 0.f));
        }
        if (post.residual) {
            const uint2 w = *reinterpret_cast<const uint2*>(static_cast<const E*>(post.residual) + o);
            v[0] += lo16<E>(w.x); v[1] += hi16<E>(w.x); v[2] += lo16<E>(w.y); v[3] += hi16<E>(w.y);
        }
        *reinterpret_cast<uint2*>(y + o) = make_uint2(pack2<E>(v[0], v[1]), pack2<E>(v[2], v[3]));
    } else if (PIX_A && howo % 2 == 0) {                 // an even number of pixels per image: pairs are adjacent and aligned
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            const int t = ra + r, k = cb;
            if (t >= rows_a) continue;
            const int n = t / howo;
            const size_t o = ((size_t)n * g.K + k) * howo + (t - n * howo);
            const float bb = (bias ? bias[k] : 0.f) + (post.addvec ? post.addvec[(size_t)n * g.K + k] : 0.f);
            float f0 = v[r] * post.scale + bb, f1 = v[r + 1] * post.scale + bb;
            if (post.residual) {
                const uint32_t w = *reinterpret_cast<const uint32_t*>(static_cast<const E*>(post.residual) + o);
                f0 += lo16<E>(w); f1 += hi16<E>(w);
            }
            *reinterpret_cast<uint32_t*>(y + o) = pack2<E>(f0, f1);
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (ra + r >= rows_a) continue;
            const int t = PIX_A ? ra + r : cb, k = PIX_A ? cb : ra + r;
            const int n = t / howo;
            const size_t o = PIX_A || planes ? ((size_t)n * g.K + k) * howo + (t - n * howo) : (size_t)t * g.K + k;
            float f = v[r] * post.scale + (bias ? bias[k] : 0.f);
            if (post.addvec) f += post.addvec[(size_t)n * g.K + k];
            if (post.residual) f += to_f32<E>(static_cast<const E*>(post.residual)[o]);
            y[o] = from_f32<E>(f);
        }
    }
}

// four adjacent outputs share an image and are 8-byte aligned
template <bool PIX_A, typename E> inline int igemm_vec_ok(const ConvGeom& g, const E* y, const IgemmPost& post, bool planes) {
    const int run = PIX_A ? g.Ho * g.Wo : g.K;            // the contiguous dimension of y
    return run % 4 == 0 && !planes && ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(post.residual)) & 7u) == 0;
}

// The kernel for 8-bit operands (conv_igemm_fp8.hip), two-byte y: whether it applies, and the launch.
bool igemm_fp8_tile_ok(const ConvGeom& g, int dt, bool nhwc, int nsplit);
// ... and the one for 3x3, stride 1, which is asked first, and whether its NCHW blocks are 256x256.
bool igemm_fp8_rows_ok(const ConvGeom& g, int dt, bool nhwc, int nsplit);
bool igemm_fp8_rows_wide(const ConvGeom& g);
hipError_t launch_igemm_fp8_rows(const void* xq, const void* Wq, const float* bias, void* y, const ConvGeom& g, const IgemmPost& post, int dt,
                                 bool nhwc, hipStream_t s);
hipError_t launch_igemm_fp8_tile(const void* xq, const void* Wq, const float* bias, void* y, const ConvGeom& g, const IgemmPost& post, int dt,
                                 bool nhwc, hipStream_t s);

}  // namespace wino

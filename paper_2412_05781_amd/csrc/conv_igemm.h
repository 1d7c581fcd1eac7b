// Declarations shared by the implicit-GEMM convolution sources (conv_igemm.hip, conv_igemm_tile.hip).
#pragma once
#include "wino_internal.h"

namespace wino {

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
// Its choice of block and of the number of reduction ranges; id < 0: it does not apply or another block of conv_igemm.hip is better.
struct IgemmTilePlan { int id, split; };
IgemmTilePlan igemm_tile_plan(int T, int K, int Cp, int R, int dt, bool nhwc);
hipError_t launch_igemm_tile(const void* xh, const void* Wr, const float* bias, void* y, float* part, const IgemmTilePlan& plan,
                             const ConvGeom& g, const IgemmPost& post, int dt, bool nhwc, hipStream_t s);

}  // namespace wino

// Mean and 1/sqrt(var + eps) per (image, channel group): the statistics that the activation
// transform needs to apply GroupNorm + SiLU while it loads x (the operators next to the 3x3
// convolution inside a residual block; the paper's Section "Techniques" argues for keeping such
// dependent steps local).  Partial (sum, sum of squares) per slice of a group: fp32 over at most 32
// elements of a lane, fp64 from there on; then one wave per group merges the slices.  (Channel-last a
// lane adds all its pixels of a slab in fp32, see there.)  Where a group is
// small enough for one workgroup (NCHW, at most kWholeGroupBytes) that workgroup writes the
// statistics itself and the second launch is saved.
// Deterministic (fixed reduction trees, no atomics).  Bound by reading x once from HBM, and for the
// small tensors of the UNet by the latency of the launches.
#include "wino_internal.h"

namespace wino {

// Slices per group.  The buffer's size follows from it and the call is not told that size: 32 is what the buffer has always held, and a
// caller may have kept the number of bytes.
constexpr int kMaxSplit = 32;
// A second launch costs 2-3 us and as much again on the host: a group of up to 128 KB is read as fast by one workgroup (fp16, 64
// groups: 82 KB each 5.4 us against 5.8 in two launches, 128 KB 5.5 against 7.0; 184 KB stay with slices, 6.5 us).
constexpr size_t kWholeGroupBytes = (size_t)128 << 10;
// Channel-last: the least bytes of a pixel that a workgroup reads.  Pieces shorter than a 128-byte line fetch the line several times out
// of L2, longer ones leave compute units idle (fp16, 32 groups, us: 128 channels at 1024x1024, pieces of 32 / 64 / 128 bytes = 256 / 128 /
// 64 workgroups: 53 / 63 / 84; 512 channels at 256x256 16.6 with any of them).
constexpr size_t kMinPiece = 32;

size_t groupnorm_stats_bytes(int N, int groups) {
    const size_t ng = (size_t)N * groups;
    return ((ng * 2 * sizeof(float) + 255) / 256) * 256 + ng * kMaxSplit * 2 * sizeof(double);
}

__device__ __forceinline__ void write_stats(float* stats, int ng, double s, double q, double inv_count, float eps) {
    const double mean = s * inv_count;
    double var = q * inv_count - mean * mean;
    var = var > 0.0 ? var : 0.0;
    stats[(size_t)ng * 2 + 0] = (float)mean;
    stats[(size_t)ng * 2 + 1] = (float)(1.0 / sqrt(var + (double)eps));
}

// Sum over the wave, valid in its last lane: four shifts inside the rows of 16 lanes, then rows 0 and 2 to rows 1 and 3, then the lower
// half to the upper.  Shuffles through LDS take 0.1-0.4 us more.
template <int CTRL, int ROWS> __device__ __forceinline__ double add_lanes(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)u, CTRL, ROWS, 0xf, false), hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(u >> 32), CTRL, ROWS, 0xf, false);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = add_lanes<0x111, 0xf>(v); v = add_lanes<0x112, 0xf>(v); v = add_lanes<0x114, 0xf>(v); v = add_lanes<0x118, 0xf>(v);
    v = add_lanes<0x142, 0xa>(v);
    return add_lanes<0x143, 0xc>(v);
}

// block reduction of (s, q); the total is valid in thread 0
template <int WAVES>
__device__ __forceinline__ void block_reduce(double s, double q, double& ts, double& tq) {
    s = wave_sum(s); q = wave_sum(q);
    __shared__ double ws[WAVES], wq[WAVES];
    if ((threadIdx.x & 63) == 63) { ws[threadIdx.x >> 6] = s; wq[threadIdx.x >> 6] = q; }
    __syncthreads();
    ts = 0.0; tq = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { ts += ws[w]; tq += wq[w]; }
    }
}

// NCHW fast path: a group is one contiguous run of cpg*H*W elements; 16-byte loads, four in flight per lane
// (512 channels at 256x256: 18.4 -> 16.2 us = 4.1 TB/s; 320 channels at 128x128, N=2: 11.2 -> 8.6).
// WHOLE: one workgroup per group (split = 1), which writes the statistics; otherwise one per slice, which writes partial sums.
template <typename E, int THREADS, bool WHOLE>
__global__ void __launch_bounds__(THREADS)
groupnorm_vec_kernel(const E* __restrict__ x, double* __restrict__ partial, float* __restrict__ stats, size_t group_elems, int split,
                     size_t per_slice, double inv_count, float eps) {
    constexpr int EPC = 16 / (int)sizeof(E);
    const int ng = blockIdx.x, sl = blockIdx.y;
    const E* base = x + (size_t)ng * group_elems;          // groups of all images are laid end to end
    const size_t lo = (size_t)sl * per_slice;
    size_t hi = lo + per_slice; hi = hi < group_elems ? hi : group_elems;
    double ds = 0.0, dq = 0.0;
    for (size_t e0 = lo + (size_t)threadIdx.x * EPC; e0 < hi; e0 += (size_t)4 * THREADS * EPC) {
        float s = 0.f, q = 0.f;
        uint4 raw[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t e = e0 + (size_t)u * THREADS * EPC;
            raw[u] = *reinterpret_cast<const uint4*>(base + (e < hi ? e : e0));      // clamped, so that the four loads stay together
            const uint32_t m = e < hi ? 0xffffffffu : 0u;
            raw[u].x &= m; raw[u].y &= m; raw[u].z &= m; raw[u].w &= m;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const E* v = reinterpret_cast<const E*>(&raw[u]);
#pragma unroll
            for (int i = 0; i < EPC; ++i) { const float f = to_f32<E>(v[i]); s += f; q = fmaf(f, f, q); }
        }
        ds += (double)s; dq += (double)q;
    }
    double ts, tq;
    block_reduce<THREADS / 64>(ds, dq, ts, tq);
    if (threadIdx.x == 0) {
        if (WHOLE) write_stats(stats, ng, ts, tq, inv_count, eps);
        else { double* dst = partial + ((size_t)ng * split + sl) * 2; dst[0] = ts; dst[1] = tq; }
    }
}

// Channel-last, C a multiple of 8: a workgroup reads the channels of `gpb` groups of a slab of pixels, a lane the same eight channels of
// every PX-th pixel (16-byte loads that run along the channels), added in fp32: 1/32 of the pixels over 4096 / (channels of the workgroup)
// lanes, 128 elements for 128 channels at 1024x1024.  (fp64 after 32 of them costs 20 % of the time, 16.6 -> 19.9 us for 512 channels at
// 256x256, and changes the largest error of a standard deviation from 6.0e-8 to 6.0e-8.)  Lane sums are added per channel over the pixel
// lanes and then per group in fp64, rounded to fp32 in between.  Read group by group instead, a group of 10...40 channels is a 20...80-byte piece of every pixel
// (N=2, 1280 channels at 16x16: 10.7 -> 6.8 us; 512 channels at 256x256: 66 -> 17 us = 3.9 TB/s).
// The workgroups of a slab, which share the lines of its pixels, are neighbours in one XCD's range.  (All channels to a workgroup and 256
// slabs would take eight times the buffer; 128 channels at 1024x1024 in 43 us instead of 53, 320 at 64x64 in 8.7 instead of 7.7.)
template <typename E, int THREADS>
__global__ void __launch_bounds__(THREADS)
groupnorm_partial_nhwc_vec_kernel(const E* __restrict__ x, double* __restrict__ partial, int C, int HW, int groups, int cpg,
                                  int split, int pixels_per_slab, int gpb, int gblocks, int total_blocks, int blocks_per_xcd) {
    constexpr int EPC = 16 / (int)sizeof(E);
    __shared__ float ls[THREADS * EPC], lq[THREADS * EPC];
    const int logical = (int)(blockIdx.x % 8) * blocks_per_xcd + (int)(blockIdx.x / 8);
    if (logical >= total_blocks) return;                    // uniform, before any barrier
    const int gb = logical % gblocks, sl = logical / gblocks % split, n = logical / gblocks / split;
    const int g0 = gb * gpb, ng = min(gpb, groups - g0), c0 = g0 * cpg, CW = ng * cpg;      // groups and channels of the workgroup
    const int octs = CW / EPC, px = THREADS / octs;         // pixel lanes; lanes beyond px * octs are idle
    const int oct = threadIdx.x % octs, pl = threadIdx.x / octs;
    float s[EPC], q[EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) { s[i] = 0.f; q[i] = 0.f; }
    const int p0 = sl * pixels_per_slab, p1 = min(p0 + pixels_per_slab, HW);
    if (pl < px) {
        const E* base = x + (size_t)n * HW * C + c0 + (size_t)oct * EPC;
        for (int p = p0 + pl; p < p1; p += 4 * px) {
            uint4 raw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int pu = p + u * px;
                raw[u] = *reinterpret_cast<const uint4*>(base + (size_t)(pu < p1 ? pu : p) * C);
                const uint32_t m = pu < p1 ? 0xffffffffu : 0u;
                raw[u].x &= m; raw[u].y &= m; raw[u].z &= m; raw[u].w &= m;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const E* v = reinterpret_cast<const E*>(&raw[u]);
#pragma unroll
                for (int i = 0; i < EPC; ++i) { const float f = to_f32<E>(v[i]); s[i] += f; q[i] = fmaf(f, f, q[i]); }
            }
        }
#pragma unroll
        for (int i = 0; i < EPC; ++i) { ls[pl * CW + oct * EPC + i] = s[i]; lq[pl * CW + oct * EPC + i] = q[i]; }
    }
    __syncthreads();
    // over the pixel lanes, fixed order; many of them in two steps (256 pixel lanes over 16 channels left 16 lanes with 256 pairs of LDS reads each:
    // 64 channels at 256x256 12.6 -> 9.3 us)
    int rows = px;
    if (px > 16) {
        rows = min(16, THREADS / CW);
        const int part = threadIdx.x / CW, c = threadIdx.x - part * CW;
        if (part < rows) {
            double a = 0.0, b = 0.0;
            for (int k = part; k < px; k += rows) { a += (double)ls[k * CW + c]; b += (double)lq[k * CW + c]; }
            ls[part * CW + c] = (float)a; lq[part * CW + c] = (float)b;     // only this lane touches rows part, part + rows, ... of column c
        }
        __syncthreads();
    }
    for (int c = threadIdx.x; c < CW; c += THREADS) {
        double a = 0.0, b = 0.0;
        for (int k = 0; k < rows; ++k) { a += (double)ls[k * CW + c]; b += (double)lq[k * CW + c]; }
        ls[c] = (float)a; lq[c] = (float)b;                 // only this lane touches column c
    }
    __syncthreads();
    auto put = [&](int g, double a, double b) {
        double* dst = partial + (((size_t)n * groups + g0 + g) * split + sl) * 2;
        dst[0] = a; dst[1] = b;
    };
    // A wave to a group where a lane would add many channels or there are no more groups than waves, else a lane (us, lane / wave: N=2, 2560
    // channels at 16x16 in one group 52.7 / 8.4, 960 at 64x64, four groups to a workgroup, 7.8 / 7.1; 1280 at 16x16, all 32 groups, 7.5 / 7.9)
    if (cpg <= 16 || (cpg <= 64 && ng > THREADS / 64)) {
        for (int g = threadIdx.x; g < ng; g += THREADS) {
            double a = 0.0, b = 0.0;
            for (int j = 0; j < cpg; ++j) { a += (double)ls[g * cpg + j]; b += (double)lq[g * cpg + j]; }
            put(g, a, b);
        }
    } else {
        for (int g = threadIdx.x >> 6; g < ng; g += THREADS / 64) {
            double a = 0.0, b = 0.0;
            for (int j = threadIdx.x & 63; j < cpg; j += 64) { a += (double)ls[g * cpg + j]; b += (double)lq[g * cpg + j]; }
            a = wave_sum(a); b = wave_sum(b);
            if ((threadIdx.x & 63) == 63) put(g, a, b);
        }
    }
}

template <typename E, bool NHWC>
__global__ void __launch_bounds__(256)
groupnorm_partial_kernel(const E* __restrict__ x, double* __restrict__ partial, int C, int HW, int groups, int cpg,
                         int split, size_t per_slice) {
    const int ng = blockIdx.x, sl = blockIdx.y;
    const int n = ng / groups, g = ng % groups;
    const size_t elems = (size_t)cpg * HW;
    const size_t lo = (size_t)sl * per_slice;
    size_t hi = lo + per_slice; hi = hi < elems ? hi : elems;
    double ds = 0.0, dq = 0.0;
    for (size_t eb = lo + threadIdx.x; eb < hi; eb += 32 * 256) {
        float s = 0.f, q = 0.f;
        for (size_t e = eb; e < hi && e < eb + 32 * 256; e += 256) {
            size_t idx;
            if (NHWC) { const size_t p = e / cpg; const int j = (int)(e - p * cpg); idx = ((size_t)n * HW + p) * C + (size_t)g * cpg + j; }
            else idx = ((size_t)n * C + (size_t)g * cpg) * HW + e;
            const float v = to_f32<E>(x[idx]);
            s += v; q = fmaf(v, v, q);
        }
        ds += (double)s; dq += (double)q;
    }
    double ts, tq;
    block_reduce<4>(ds, dq, ts, tq);
    if (threadIdx.x == 0) { double* dst = partial + ((size_t)ng * split + sl) * 2; dst[0] = ts; dst[1] = tq; }
}

// One wave per group: the slices are loaded side by side and added in a fixed tree.
__global__ void __launch_bounds__(64)
groupnorm_finalize_kernel(const double* __restrict__ partial, float* __restrict__ stats, int split, double inv_count, float eps) {
    const int ng = blockIdx.x, lane = threadIdx.x;
    const double2* src = reinterpret_cast<const double2*>(partial) + (size_t)ng * split;
    double s = 0.0, q = 0.0;
    for (int i = lane; i < split; i += 64) { const double2 v = src[i]; s += v.x; q += v.y; }
    s = wave_sum(s); q = wave_sum(q);
    if (lane == 63) write_stats(stats, ng, s, q, inv_count, eps);
}

hipError_t launch_groupnorm_stats(const void* x, float* stats, int N, int C, int H, int W, int groups, float eps,
                                  int dt, bool nhwc, hipStream_t s) {
    const int cpg = C / groups, HW = H * W, total = N * groups;
    const size_t elems = (size_t)cpg * HW;
    const size_t esz = two_byte(dt) ? 2 : 4, epc = 16 / esz;
    const double inv_count = 1.0 / (double)elems;
    double* partial = reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(stats) +
                                                (((size_t)total * 2 * sizeof(float) + 255) / 256) * 256);
    const bool x16 = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    const bool vec = !nhwc && (elems * esz) % 16 == 0 && x16;
    if (vec && elems * esz <= kWholeGroupBytes) {
        (void)with_dtype(dt, [&](auto* tag) {
            using E = std::remove_pointer_t<decltype(tag)>;
            hipLaunchKernelGGL((groupnorm_vec_kernel<E, 1024, true>), dim3((unsigned)total, 1), dim3(1024), 0, s,
                               (const E*)x, partial, stats, elems, 1, elems, inv_count, eps);
            return hipSuccess;
        });
        return hipGetLastError();
    }
    // channel-last with whole 16-byte channel octets, all of them within one workgroup's lanes; tensors of less than about 100 000 elements per
    // image are faster group by group (64 channels at 8x8 4.9 us against 6.8, 1280 at 8x8 6.7 against 7.4, 128 at 32x32 8.1 against 7.2)
    constexpr int NT = 512;
    if (nhwc && (size_t)HW * C >= 98304 && C % (int)epc == 0 && C / (int)epc <= NT && x16) {
        // about 16 KB per workgroup and at most 256 per image: 32 slabs of pixels, then blocks of groups, of whole 16-byte pieces and at
        // least kMinPiece bytes of a pixel
        const size_t bytes = (size_t)HW * C * esz;
        const int want = (int)(bytes / (16 << 10) < 1 ? 1 : (bytes / (16 << 10) > 256 ? 256 : bytes / (16 << 10)));
        int split = want > kMaxSplit ? kMaxSplit : want;
        split = split > HW ? HW : split;
        const int pps = (HW + split - 1) / split;
        split = (HW + pps - 1) / pps;
        int unit = 1;                                                                     // groups
        while ((unit * cpg) % (int)epc != 0 || ((size_t)unit * cpg * esz < kMinPiece && unit < groups)) ++unit;
        const int units = (groups + unit - 1) / unit, blocks = want / split < units ? (want / split < 1 ? 1 : want / split) : units;
        const int gpb = (units + blocks - 1) / blocks * unit;
        const int gblocks = (groups + gpb - 1) / gpb;
        const long long all = (long long)N * split * gblocks;
        if (all > 0x3fffffffLL) return hipErrorInvalidValue;
        const int per_xcd = (int)((all + 7) / 8);
        (void)with_dtype(dt, [&](auto* tag) {
            using E = std::remove_pointer_t<decltype(tag)>;
            hipLaunchKernelGGL((groupnorm_partial_nhwc_vec_kernel<E, NT>), dim3((unsigned)(per_xcd * 8)), dim3(NT), 0, s,
                               (const E*)x, partial, C, HW, groups, cpg, split, pps, gpb, gblocks, (int)all, per_xcd);
            return hipSuccess;
        });
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(groupnorm_finalize_kernel, dim3((unsigned)total), dim3(64), 0, s, (const double*)partial, stats, split, inv_count, eps);
        return hipGetLastError();
    }
    // slices are whole numbers of block-wide 16-byte loads (256 lanes x 16 bytes), eight of them per slice with 16-byte loads, two with single elements
    const size_t quantum = 256 * epc;
    const size_t per = (vec ? 8 : 2) * quantum;
    const size_t want = (elems + per - 1) / per;
    const int split0 = want < 1 ? 1 : (want > (size_t)kMaxSplit ? kMaxSplit : (int)want);
    size_t per_slice = (elems + split0 - 1) / split0;
    per_slice = (per_slice + quantum - 1) / quantum * quantum;
    const int split = (int)((elems + per_slice - 1) / per_slice);
    // few groups and long slices: four times the lanes (512x512, 128 channels, 4 groups: 46 -> 15.4 us)
    const bool tall = (long long)total * split < 512 && per_slice >= 16 * quantum;
    dim3 grid((unsigned)total, (unsigned)split), block(256);
    (void)with_dtype(dt, [&](auto* tag) {
        using E = std::remove_pointer_t<decltype(tag)>;
        if (vec && tall) hipLaunchKernelGGL((groupnorm_vec_kernel<E, 1024, false>), grid, dim3(1024), 0, s, (const E*)x, partial, stats, elems, split, per_slice, inv_count, eps);
        else if (vec)  hipLaunchKernelGGL((groupnorm_vec_kernel<E, 256, false>), grid, block, 0, s, (const E*)x, partial, stats, elems, split, per_slice, inv_count, eps);
        else if (nhwc) hipLaunchKernelGGL((groupnorm_partial_kernel<E, true>), grid, block, 0, s, (const E*)x, partial, C, HW, groups, cpg, split, per_slice);
        else           hipLaunchKernelGGL((groupnorm_partial_kernel<E, false>), grid, block, 0, s, (const E*)x, partial, C, HW, groups, cpg, split, per_slice);
        return hipSuccess;
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(groupnorm_finalize_kernel, dim3((unsigned)total), dim3(64), 0, s, (const double*)partial, stats, split, inv_count, eps);
    return hipGetLastError();
}

}  // namespace wino

// tsdf_filter.hip -- the bilateral depth filter of the image preparation
// stage (Sec. 4; Sec. 6 useBilateralFilter) on gfx950.
//
// One workgroup per 16x16 output tile: the tile and its halo of `radius`
// pixels are staged in LDS once (u16 millimetres converted on the way), and
// each thread forms one output pixel's weighted mean from LDS.  The work is a
// small stencil: HBM traffic is one read and one write of the image, and the
// images of a depth camera leave the time to one pixel's chain of taps.  So
// the window is unrolled for each radius: its LDS reads and exponentials
// overlap, the weights come with the arguments, and a tap without depth is
// selected away instead of branched around.  The kernel, against a loop with
// expf: 160x120 radius 4 13.0 -> 6.7 us, 333x251 radius 2 6.8 -> 4.5 (the call
// stays at 8, the host's share); from some 300000 pixels on bound by vector
// instructions, 19 a tap: 1280x720 radius 2 16.5 -> 14.5, radius 3 27.5 -> 25.0,
// radius 5 60.9 -> 54.5; 640x480 radius 7 45.1 -> 36.5; 3000x2000 radius 7
// 586 -> 559 (calls without a gap between them 524 -> 535).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "tsdf_filter.h"

namespace {

constexpr int kTile = 16;
constexpr int taps_of(int r) { return (2 * r + 1) * (2 * r + 1); }

// by value to the kernel, so no longer than the window needs
template <int R>
struct BilArgs {
    float inv2sr2;                 // 1 / (2 sigma_range^2)
    float ws[taps_of(R)];          // spatial weights, row-major over (dy, dx)
};

template <int FMT>
__device__ __forceinline__ float load_depth(const void *src, size_t i)
{
    if (FMT == TF_DEPTH_U16_MM) return (float)((const uint16_t *)src)[i] / 1000.0f;
    return ((const float *)src)[i];
}

// exp(t) for t <= 0: 2^(t log2 e), the product in two parts of which the nearest
// whole number is taken out exactly before the hardware's exponential, and put
// back as the result's exponent.  Over every float from -104 to -1e-9 its error
// is expf's: mean 0.243 to 0.257 ulp, at most 0.857; below -87, among the
// subnormals, mean 0.255 and at most 0.891 (expf 0.273 and 1.0).  What it leaves
// out is expf's way through overflow, which a weight cannot take.
__device__ __forceinline__ float exp_neg(float t)
{
    constexpr float c = 1.44269502162933350f, cl = 1.92596299112661746e-8f;   // log2 e = c + cl
    t = __builtin_elementwise_maximum(t, -1000.0f);   // no infinity below; NaN stays
    const float hi = t * c;
    const float lo = fmaf(t, cl, fmaf(t, c, -hi));
    const float n = rintf(hi);
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((hi - n) + lo), (int)n);
}

// one tap of the window into the sums; a neighbour without depth (0 in the tile)
// leaves them as they are
__device__ __forceinline__ void tap(float dq, float dp, float ws, float inv2sr2, float &sw, float &swd)
{
    const float e = dq - dp;
    const float w = ws * exp_neg(dq > 0.0f ? -(e * e) * inv2sr2 : -1000.0f);   // (2^-1443: none)
    sw += w;
    swd += w * e;
}

template <int FMT, int R>
__global__ __launch_bounds__(256) void k_bilateral(const void *src, int W, int H, BilArgs<R> a, float *out)
{
    constexpr int r = R, side = kTile + 2 * R;
    __shared__ float tile[side * side];
    const int x0 = (int)blockIdx.x * kTile - r, y0 = (int)blockIdx.y * kTile - r;
    for (int i = threadIdx.x; i < side * side; i += 256) {
        const int ty = i / side, tx = i - ty * side;
        const int gx = x0 + tx, gy = y0 + ty;
        // outside the image reads as invalid, which the window skips
        const float d = (gx >= 0 && gx < W && gy >= 0 && gy < H) ? load_depth<FMT>(src, (size_t)gy * W + gx) : 0.0f;
        tile[i] = d > 0.0f ? d : 0.0f;
    }
    __syncthreads();
    const int lx = threadIdx.x & 15, ly = threadIdx.x >> 4;
    const int x = (int)blockIdx.x * kTile + lx, y = (int)blockIdx.y * kTile + ly;
    if (x >= W || y >= H) return;
    const float *c = tile + (ly + r) * side + (lx + r);
    const float dp = c[0];
    float res = 0.0f;
    if (dp > 0.0f) {
        float sw = 0.0f, swd = 0.0f;
#pragma unroll
        for (int k = 0; k < taps_of(R); ++k)
            tap(c[(k / (2 * R + 1) - R) * side + k % (2 * R + 1) - R], dp, a.ws[k], a.inv2sr2, sw, swd);
        res = dp + swd / sw;       // sw >= 1: the centre's own weight
    }
    out[(size_t)y * W + x] = res;
}

template <int FMT, int R>
void launch(dim3 grid, hipStream_t s, const void *src, int W, int H, const tf_bilateral_params &p, float *out)
{
    BilArgs<R> a;
    const double ss = p.sigma_space, sr = p.sigma_range;
    a.inv2sr2 = (float)(1.0 / (2.0 * sr * sr));
    float by_d2[2 * R * R + 1];
    for (int q = 0; q <= 2 * R * R; ++q) by_d2[q] = (float)exp(-(double)q / (2.0 * ss * ss));
    int k = 0;
    for (int dy = -R; dy <= R; ++dy)
        for (int dx = -R; dx <= R; ++dx) a.ws[k++] = by_d2[dx * dx + dy * dy];
    hipLaunchKernelGGL((k_bilateral<FMT, R>), grid, dim3(256), 0, s, src, W, H, a, out);
}

template <int FMT>
void launch_radius(dim3 grid, hipStream_t s, const void *src, int W, int H, const tf_bilateral_params &p, float *out)
{
    static_assert(TF_BILATERAL_MAX_RADIUS == 7, "a kernel for each radius");
    switch (p.radius) {
    case 1: launch<FMT, 1>(grid, s, src, W, H, p, out); break;
    case 2: launch<FMT, 2>(grid, s, src, W, H, p, out); break;
    case 3: launch<FMT, 3>(grid, s, src, W, H, p, out); break;
    case 4: launch<FMT, 4>(grid, s, src, W, H, p, out); break;
    case 5: launch<FMT, 5>(grid, s, src, W, H, p, out); break;
    case 6: launch<FMT, 6>(grid, s, src, W, H, p, out); break;
    default: launch<FMT, 7>(grid, s, src, W, H, p, out); break;
    }
}

}  // namespace

extern "C" int tf_bilateral(const void *d_depth, int depth_format, int32_t width, int32_t height,
                            const tf_bilateral_params *p, float *d_out, tf_stream stream)
{
    if (!d_depth || !d_out || !p) return TF_E_INVAL;
    if (depth_format != TF_DEPTH_F32_M && depth_format != TF_DEPTH_U16_MM) return TF_E_INVAL;
    if (width < 1 || height < 1 || width > 8192 || height > 8192) return TF_E_INVAL;
    if (p->radius < 1 || p->radius > TF_BILATERAL_MAX_RADIUS) return TF_E_INVAL;
    if (!(p->sigma_space > 0.0f) || !(p->sigma_range > 0.0f) || !(p->sigma_space < 1e30f) ||
        !(p->sigma_range < 1e30f))
        return TF_E_INVAL;
    if (((uintptr_t)d_out & 3u) || ((uintptr_t)d_depth & (depth_format == TF_DEPTH_F32_M ? 3u : 1u)))
        return TF_E_INVAL;
    const size_t in_bytes = (size_t)width * height * (depth_format == TF_DEPTH_F32_M ? 4 : 2);
    const uintptr_t a0 = (uintptr_t)d_depth, a1 = a0 + in_bytes;
    const uintptr_t b0 = (uintptr_t)d_out, b1 = b0 + (size_t)width * height * 4;
    if (a0 < b1 && b0 < a1) return TF_E_INVAL;
    const dim3 grid((width + kTile - 1) / kTile, (height + kTile - 1) / kTile);
    if (depth_format == TF_DEPTH_U16_MM)
        launch_radius<TF_DEPTH_U16_MM>(grid, (hipStream_t)stream, d_depth, width, height, *p, d_out);
    else
        launch_radius<TF_DEPTH_F32_M>(grid, (hipStream_t)stream, d_depth, width, height, *p, d_out);
    return hipGetLastError() == hipSuccess ? TF_OK : TF_E_HIP;
}

// nn_kernels.hip -- gfx950 kernels of the learned depth prefilter.
//
// The 3x3 convolutions are implicit GEMMs on the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation):
//   k_conv_fwd          encoder: M = output pixels, N = cout, K = (tap, ci);
//                       the workgroup's input tile is staged in LDS, the
//                       operand reads from it apply the stride
//   k_conv_fwd_up       decoder (nearest 2x upsampling, then 3x3): per output
//                       parity a 2x2 convolution of the source (a tile staged
//                       in LDS) on folded weights split into bf16 high and
//                       low halves, K = (source offset, half, ci)
//   k_conv_bwd_data_s2  stride-2 layers: M = input pixels, N = cin, K = the
//                       taps that reach the input pixel's parity x co
//   k_conv_bwd_data_up  decoder: the adjoint of the folded forward, K = (16
//                       parity x offset, half, co)
//   k_conv_wgrad_s2,    M = cout, N = cin of a tap (or of a parity and source
//   k_conv_wgrad_up     offset), K = pixels of one chunk: staged as they lie,
//                       transposed by the LDS reads; per-chunk partial sums
//                       are reduced in a fixed order
// Bias, skip add / skip gradient and relu (mask) are fused into every
// epilogue, which is staged in LDS and written as 16-byte pixel vectors.
// The 32->1 head, the loss, input packing and Adam are plain VALU kernels.
//
// MFMA 16x16x32 operand layout (per lane l of the wave): A row l%16, k
// (l/16)*8 .. +7; B column l%16, same k; D column l%16, rows (l/16)*4 .. +3.
#include "nn_internal.h"
#include "tsdf.h"

namespace tsdf {
namespace nn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// an int known at compile time, as an argument of a generic lambda
template <int V> struct Const { static constexpr int v = V; };

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;   // NaN
    u += 0x7fffu + ((u >> 16) & 1u);                      // round to nearest even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ u32x4 ld16(const uint16_t *p)
{
    return *(const __attribute__((address_space(1))) u32x4 *)p;
}

__device__ __forceinline__ bf16x8 as_bf(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace

// ============================================================================
// input packing: depth -> metres and (d / 4, valid, hp, 0 x 5) bf16, where
// hp = (d - mean of the valid 3x3 neighbours) / 5 cm on valid pixels
// ============================================================================
template <int FMT>
__device__ __forceinline__ float depth_at(const void *depth, size_t i)
{
    float d;
    if (FMT == TF_DEPTH_U16_MM)
        d = (float)reinterpret_cast<const uint16_t *>(depth)[i] / 1000.0f;
    else
        d = reinterpret_cast<const float *>(depth)[i];
    return d > 0.0f ? d : 0.0f;
}

// One workgroup per 16x16 tile of one image: the tile's depths in metres with
// a one-pixel border (-1 outside the image) are converted once into LDS, then
// each pixel sums its valid 3x3 neighbours from there in row-major order.
template <int FMT>
__global__ __launch_bounds__(256) void k_make_input(const void *depth, int N, int H, int W, uint16_t *x, float *dm)
{
    __shared__ float t[18][18];
    const int tx = (int)blockIdx.x * 16, ty = (int)blockIdx.y * 16, n = (int)blockIdx.z;
    for (int k = (int)threadIdx.x; k < 18 * 18; k += 256) {
        const int iy = ty - 1 + k / 18, ix = tx - 1 + k % 18;
        float v = -1.0f;
        if (iy >= 0 && iy < H && ix >= 0 && ix < W) v = depth_at<FMT>(depth, ((size_t)n * H + iy) * W + ix);
        t[k / 18][k % 18] = v;
    }
    __syncthreads();
    const int lx = (int)threadIdx.x & 15, ly = (int)threadIdx.x >> 4;
    const int xx = tx + lx, y = ty + ly;
    if (xx >= W || y >= H) return;
    const size_t p = ((size_t)n * H + y) * W + xx;
    const float d = t[ly + 1][lx + 1];
    float s = 0.0f, c = 0.0f;
    for (int ky = 0; ky < 3; ++ky)
        for (int kx = 0; kx < 3; ++kx) {
            const float v = t[ly + ky][lx + kx];
            if (v > 0.0f) {
                s += v;
                c += 1.0f;
            }
        }
    const float hp = d > 0.0f ? (d - s / c) / kCorrScale : 0.0f;
    dm[p] = d;
    u32x4 v = {(uint32_t)f2bf(d * 0.25f) | ((uint32_t)(d > 0.0f ? f2bf(1.0f) : 0u) << 16), (uint32_t)f2bf(hp), 0u,
               0u};
    *reinterpret_cast<u32x4 *>(x + p * 8) = v;
}

// ============================================================================
// epilogue of the implicit-GEMM convolutions.  In the MFMA result a lane holds
// 4 pixels of one channel per 16x16 tile, so the per-element bias / skip /
// activation reads and the output writes would be 2-byte accesses.  A wave
// stages each 16-pixel row tile in its own LDS tile instead; every lane then
// handles whole 16-byte vectors (one pixel, 8 channels).  The tile is the
// wave's own, so a wave-scope fence and barrier order the staging writes
// before the other lanes' reads (a wave's LDS instructions execute in order).
// ============================================================================
template <int NT>
struct alignas(16) EpiTile {
    float v[16][NT * 16 + 4];   // +4: the staging writes of one instruction hit distinct banks
};

template <int NT, typename F>
__device__ __forceinline__ void epilogue_tile(EpiTile<NT> &st, const f32x4 (&a)[NT], int lane, F &&emit)
{
    const int r = lane & 15, gq = lane >> 4;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) st.v[gq * 4 + i][j * 16 + r] = a[j][i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int u = 0; u < (32 * NT + 63) / 64; ++u) {
        const int v = lane + 64 * u;   // 16 pixels x 2 NT vectors of 8 channels
        if (v < 32 * NT) {
            const int pix = v / (2 * NT), c8 = (v - pix * 2 * NT) * 8;
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(&st.v[pix][c8]);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(&st.v[pix][c8 + 4]);
            emit(pix, c8, lo, hi);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// two floats to packed bf16 (low half = a) by v_cvt_pk_bf16_f32: round to
// nearest even, the same bits as f2bf for every finite value
__device__ __forceinline__ uint32_t bf2(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

// forward: o[e] = bf16(relu(x[e] + bias[e] (+ skip[e]))), e = 0..7
template <bool SKIP>
__device__ __forceinline__ void fwd_store8(uint16_t *o, f32x4 lo, f32x4 hi, const float *bias, const uint16_t *skip)
{
    const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    u32x4 sk = {0u, 0u, 0u, 0u};
    if (SKIP) sk = ld16(skip);
    u32x4 ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v0 = x[2 * e] + bias[2 * e], v1 = x[2 * e + 1] + bias[2 * e + 1];
        if (SKIP) {
            v0 += bf2f((uint16_t)(sk[e] & 0xffffu));
            v1 += bf2f((uint16_t)(sk[e] >> 16));
        }
        ov[e] = bf2(v0 > 0.0f ? v0 : 0.0f, v1 > 0.0f ? v1 : 0.0f);
    }
    *reinterpret_cast<u32x4 *>(o) = ov;
}

// backward data: o[e] = bf16(x[e] (+ skipg[e])), zero where act[e] <= 0
template <bool SKIP>
__device__ __forceinline__ void bwd_store8(uint16_t *o, f32x4 lo, f32x4 hi, const uint16_t *skipg, const uint16_t *act)
{
    const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    u32x4 sk = {0u, 0u, 0u, 0u};
    if (SKIP) sk = ld16(skipg);
    const u32x4 av = ld16(act);
    u32x4 ov;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v0 = x[2 * e], v1 = x[2 * e + 1];
        if (SKIP) {
            v0 += bf2f((uint16_t)(sk[e] & 0xffffu));
            v1 += bf2f((uint16_t)(sk[e] >> 16));
        }
        if (!(bf2f((uint16_t)(av[e] & 0xffffu)) > 0.0f)) v0 = 0.0f;
        if (!(bf2f((uint16_t)(av[e] >> 16)) > 0.0f)) v1 = 0.0f;
        ov[e] = bf2(v0, v1);
    }
    *reinterpret_cast<u32x4 *>(o) = ov;
}

// ============================================================================
// fp32 master weights -> bf16 GEMM operands of every conv layer
// ============================================================================
// Forward operands are stored in MFMA fragment order: element
// ((step * cout / 16 + tile) * 64 + lane) * 8 + e holds the B value of lane
// lane = gq * 16 + r at K step `step`, i.e. output channel tile * 16 + r and
// k = step * 32 + gq * 8 + e.  The 64 lanes' 16-byte fragments of one (step,
// tile) are contiguous, so a fragment load reads whole cache lines.
__device__ __forceinline__ void frag_coords(int j, int cout, int &co, int &k)
{
    const int e = j & 7, lane = (j >> 3) & 63, st = (j >> 9) / (cout / 16), tile = (j >> 9) - st * (cout / 16);
    co = tile * 16 + (lane & 15);
    k = st * 32 + (lane >> 4) * 8 + e;
}

__device__ __forceinline__ void pack_g(const float *w, int cin, int cinp, int cout, int i, uint16_t *g)
{
    int co, k;
    frag_coords(i, cout, co, k);
    const int tap = k / cinp, ci = k % cinp;
    g[i] = (tap < 9 && ci < cin) ? f2bf(w[(co * 9 + tap) * cin + ci]) : (uint16_t)0;
}

// backward-data operand in the same order: K step tap * cout / 32 + co / 32, the B column is input channel ci
__device__ __forceinline__ void pack_t(const float *w, int cin, int cinp, int cout, int i, uint16_t *t)
{
    int ci, k;
    frag_coords(i, cinp, ci, k);
    const int tap = k / cout, co = k % cout;
    t[i] = ci < cin ? f2bf(w[(co * 9 + tap) * cin + ci]) : (uint16_t)0;
}

// Nearest 2x upsampling followed by a 3x3 convolution, folded by output
// parity: output pixel (2m + py, 2n + px) reads only the 2x2 source pixels
// (m + py - 1 + a, n + px - 1 + b), a, b in {0, 1}.  Tap ky lands on source
// row offset a = ((py + ky - 1) >> 1) + 1 - py (likewise kx -> b): per axis
// one offset receives one tap and the other two, so per parity the four
// offsets receive 1, 2, 2 and 4 of the 9 taps.  The folded weight of an
// offset is s = the fp32 sum of the bf16 taps landing there (ascending ky,
// kx); it is carried as two bf16 numbers, hi = bf16(s) and lo = bf16(s - hi),
// so that a product with a bf16 activation sums the taps' products: hi + lo
// equals s exactly where at most two taps land (the rounding error of a
// two-term sum is representable in the same precision) and within 2^-17 of
// s at the four-tap offset.  The one-tap offset (a, b) = (py, px) has lo = 0.
// Zero padding agrees: a source row is outside the image exactly when every
// tap landing on it is.
__device__ __forceinline__ uint16_t folded_weight(const float *w, int cin, int par, int co, int q, int ci, int lo)
{
    const int py = par >> 1, px = par & 1, a = q >> 1, b = q & 1;
    float s = 0.0f;
    if (ci < cin)
        for (int ky = 0; ky < 3; ++ky) {
            if (((py + ky - 1) >> 1) + 1 - py != a) continue;
            for (int kx = 0; kx < 3; ++kx) {
                if (((px + kx - 1) >> 1) + 1 - px != b) continue;
                s += bf2f(f2bf(w[(co * 9 + ky * 3 + kx) * cin + ci]));
            }
        }
    const uint16_t hi = f2bf(s);
    return lo ? f2bf(s - bf2f(hi)) : hi;
}

// forward operand gu[lo][par][cout x 4 cinp matrix in fragment order], the
// matrix's K index k = q * cinp + ci, q = a * 2 + b
__device__ __forceinline__ void pack_up(const float *w, int cin, int cinp, int cout, int i, uint16_t *gu)
{
    const int k4 = 4 * cinp;
    const int half = 4 * cout * k4;
    const int lo = i / half, j = i - lo * half;
    const int par = j / (cout * k4), rem = j - par * cout * k4;
    int co, k;
    frag_coords(rem, cout, co, k);
    const int q = k / cinp, ci = k - (k / cinp) * cinp;
    gu[i] = folded_weight(w, cin, par, co, q, ci, lo);
}

// backward-data operand of the same folded weights, in fragment order: K step
// st = (par * 4 + q) * cout / 32 + co / 32, the B column is input channel ci
__device__ __forceinline__ void pack_tu(const float *w, int cin, int cinp, int cout, int i, uint16_t *tu)
{
    const int half = cinp * 16 * cout;
    const int lo = i / half, j = i - lo * half;
    int ci, k;
    frag_coords(j, cinp, ci, k);
    const int pq = k / cout, co = k - (k / cout) * cout;
    tu[i] = folded_weight(w, cin, pq >> 2, co, pq & 3, ci, lo);
}

// every conv layer's packed weights in one launch: thread i belongs to the
// layer whose [start, next start) range holds it
__global__ __launch_bounds__(256) void k_pack(PackJobs J)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    int l = 0;
    while (l < kLayers - 1 && i >= J.start[l + 1]) ++l;
    if (l >= kLayers - 1) return;
    const PackJob &p = J.job[l];
    const int li = i - J.start[l];
    if (li < p.n_g) {
        if (p.up)
            pack_up(p.w, p.cin, p.cinp, p.cout, li, p.g);
        else
            pack_g(p.w, p.cin, p.cinp, p.cout, li, p.g);
    }
    if (p.t && li < p.n_t) {
        if (p.up)
            pack_tu(p.w, p.cin, p.cinp, p.cout, li, p.t);
        else
            pack_t(p.w, p.cin, p.cinp, p.cout, li, p.t);
    }
}

// ============================================================================
// Workgroups of the staged forward kernels go round-robin to the 8 XCDs;
// remapped so that XCD x takes the x-th contiguous band of tiles, the
// neighbouring tiles that share input rows share that XCD's L2.  The grid is
// rounded up to a multiple of 8; tiles past the end stage zeros and store
// nothing.
// ============================================================================
__device__ __forceinline__ long xcd_band_tile(long ntiles)
{
    const long per = (ntiles + 7) / 8;
    return (long)(blockIdx.x % 8u) * per + blockIdx.x / 8u;
}

// stage rows iy0 .. iy0 + IR - 1, columns ix0 .. ix0 + IC - 1 of one image's
// NHWC bf16 tensor (CINP channels) in LDS, RS bytes per pixel, zeros outside;
// SPLIT keeps the even columns before the odd ones, so that pixels two apart
// are RS bytes apart (IC even)
template <int CINP, int IR, int IC, int RS, bool SPLIT = false>
__device__ __forceinline__ void stage_tile(unsigned char *tile, const uint16_t *in, int nimg, int Hs, int Ws,
                                           int iy0, int ix0, bool live)
{
    constexpr int CH = CINP / 8;
    for (int i = (int)threadIdx.x; i < IR * IC * CH; i += 256) {
        const int ch = i % CH, pc = i / CH, c = pc % IC, rr = pc / IC;
        const int sy = iy0 + rr, sx = ix0 + c;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (live && sy >= 0 && sy < Hs && sx >= 0 && sx < Ws)
            v = ld16(in + (((size_t)nimg * Hs + sy) * Ws + sx) * CINP + ch * 8);
        const int cs = SPLIT ? (c & 1) * (IC / 2) + (c >> 1) : c;
        *reinterpret_cast<u32x4 *>(tile + (rr * IC + cs) * RS + ch * 16) = v;
    }
    __syncthreads();
}

// ============================================================================
// forward 3x3 convolution (no skip input): a workgroup takes ROWS = 4 R / NS
// output rows x 16 T columns; it stages the input rows and columns those
// reach (with the stride) in LDS with coalesced 16-byte loads, then each
// wave computes 16 T pixels of R rows x COUT / NS channels, A fragments
// from LDS, B fragments (fragment order) from global memory.  The K steps are
// unrolled in full, so that the weight loads of several steps are in flight:
// e4 at 8 x 256 x 256 12.2 -> 8.2 us against steps two at a time.  Two rows
// where the channels are split over the waves stage 5 input rows for 2 outputs
// instead of 3 for 1 (640x480: e2 13.0 -> 11.5 us, e3 8.2 -> 7.8)
// ============================================================================
template <int CINP, int COUT, int STRIDE, int T, int NS, int R>
__global__ __launch_bounds__(256) void k_conv_fwd(const uint16_t *in, int Hs, int Ws, const uint16_t *g,
                                                  const float *bias, uint16_t *out, int N, int Ho, int Wo)
{
    static_assert(NS == 1 || NS == 2 || NS == 4, "channel split must divide the 4 waves of a workgroup");
    constexpr int KP = ((9 * CINP + 31) / 32) * 32;
    constexpr int NT = COUT / 16 / NS;
    constexpr int ROWS = R * (4 / NS);
    constexpr int IR = STRIDE * (ROWS - 1) + 3, IC = STRIDE * (16 * T - 1) + 3;
    constexpr int RS = CINP * 2 + 16;   // +16 bytes: neighbouring pixels' fragments start on different banks
    __shared__ __attribute__((aligned(16))) unsigned char tile[IR * IC * RS];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6, r = lane & 15, gq = lane >> 4;
    const int tx = (Wo + 16 * T - 1) / (16 * T), ty = (Ho + ROWS - 1) / ROWS;
    const long ntiles = (long)N * ty * tx;
    const long wt = xcd_band_tile(ntiles);
    const bool live = wt < ntiles;
    const long gt = live ? wt : 0;
    const int xt = (int)(gt % tx);
    const long nyt = gt / tx;
    const int nimg = (int)(nyt / ty), y0 = (int)(nyt - (long)nimg * ty) * ROWS, x0 = xt * 16 * T;
    stage_tile<CINP, IR, IC, RS>(tile, in, nimg, Hs, Ws, STRIDE * y0 - 1, STRIDE * x0 - 1, live);
    const int yy = w / NS * R, cbase = (w % NS) * (COUT / NS);
    f32x4 acc[R * T][NT];   // [row * T + run of 16 columns]
#pragma unroll
    for (int t = 0; t < R * T; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < KP; k0 += 32) {
        const int k = k0 + gq * 8;
        const int tap = k / CINP, ci = k - (k / CINP) * CINP;
        const int ky = tap / 3, kx = tap - (tap / 3) * 3;
        bf16x8 a[R * T];
#pragma unroll
        for (int t = 0; t < R * T; ++t) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (tap < 9)   // K padding past the 9 taps multiplies zeros
                v = *reinterpret_cast<const u32x4 *>(tile + ((STRIDE * (yy + t / T) + ky) * IC + STRIDE * (t % T * 16 + r) + kx) * RS +
                                                     ci * 2);
            a[t] = as_bf(v);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const bf16x8 b = as_bf(ld16(g + ((size_t)((k0 / 32) * (COUT / 16) + cbase / 16 + j) * 64 + lane) * 8));
#pragma unroll
            for (int t = 0; t < R * T; ++t) acc[t][j] = mfma(a[t], b, acc[t][j]);
        }
    }
    __shared__ EpiTile<NT> st[4];
#pragma unroll
    for (int t = 0; t < R * T; ++t)
        epilogue_tile(st[w], acc[t], lane, [&](int pix, int c8, f32x4 lo, f32x4 hi) {
            const int ox = x0 + t % T * 16 + pix, oy = y0 + yy + t / T;
            if (!live || oy >= Ho || ox >= Wo) return;
            const size_t p = ((size_t)nimg * Ho + oy) * Wo + ox;
            const int co = cbase + c8;
            fwd_store8<false>(out + p * COUT + co, lo, hi, bias + co, nullptr);
        });
}

// Forward of an upsampled layer on the parity-folded weights (split into
// high and low halves; the one-tap offset has no low half: 7 cinp
// multiply-adds per output instead of 9 cinp).  A workgroup = the 4 output
// parities (one per wave) of one (image, band of R source rows, run of 16 T
// source columns) and one of NS shares of the output channels; it stages the
// R + 2 source rows and 16 T + 2 columns that every parity's 2x2 offsets read in
// LDS (a square stages less a pixel than a strip and serves more products with a
// weight load).  The K loop is written out for each parity: which steps have
// a low half is then known, no branch ends a step, and the weight loads (from
// L2, whose latency bounds the loop) of several steps are in flight.  d1, d2,
// d3 at 8 x 256 x 256: 38.7, 24.5 and 17.8 us with the branch, 28.5, 19.1 and 14.6
// without it on strips of one row, 25.0, 15.2 and 11.0 now.
template <int CINP, int COUT, bool SKIP, int T, int NS, int R>
__global__ __launch_bounds__(256) void k_conv_fwd_up(const uint16_t *in, int Hs, int Ws, const uint16_t *gu,
                                                     const float *bias, const uint16_t *skip, uint16_t *out, int N)
{
    constexpr int K4 = 4 * CINP;
    constexpr int NT = COUT / 16 / NS;
    constexpr int TC = 16 * T + 2;
    constexpr int RS = CINP * 2 + 16;
    static_assert(CINP % 32 == 0, "a K step stays inside one source offset");
    __shared__ __attribute__((aligned(16))) unsigned char tile[(R + 2) * TC * RS];
    const int lane = (int)threadIdx.x & 63, r = lane & 15, gq = lane >> 4;
    const int runs = (Ws + 16 * T - 1) / (16 * T);
    const int bands = (Hs + R - 1) / R;
    const long ntiles = (long)N * bands * runs * NS;
    const long wt = xcd_band_tile(ntiles);
    const bool live = wt < ntiles;
    const int cbase = (int)(wt % NS) * (COUT / NS);
    const long gt = live ? wt / NS : 0;
    const int run = (int)(gt % runs);
    const long nm = gt / runs;
    const int nimg = (int)(nm / bands), m0 = (int)(nm - (long)nimg * bands) * R;
    const int c0 = run * 16 * T;
    stage_tile<CINP, R + 2, TC, RS>(tile, in, nimg, Hs, Ws, m0 - 1, c0 - 1, live);
    const int par = (int)threadIdx.x >> 6;
    const int py = par >> 1, px = par & 1;
    const int Ho = 2 * Hs, Wo = 2 * Ws;
    f32x4 acc[R * T][NT];   // [row * T + run of 16 columns]
#pragma unroll
    for (int t = 0; t < R * T; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t *gp = gu + (size_t)par * COUT * K4;
    const uint16_t *gl = gp + (size_t)4 * COUT * K4;   // low halves
    auto contract = [&](auto parity) {
        constexpr int PAR = decltype(parity)::v;
#pragma unroll
        for (int st = 0; st < K4 / 32; ++st) {
            const int q = st / (CINP / 32), ci = (st - q * (CINP / 32)) * 32 + gq * 8;
            bf16x8 av[R * T];
#pragma unroll
            for (int t = 0; t < R * T; ++t)
                av[t] = as_bf(*reinterpret_cast<const u32x4 *>(
                    tile + ((t / T + (PAR >> 1) + (q >> 1)) * TC + t % T * 16 + r + (PAR & 1) + (q & 1)) * RS + ci * 2));
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const size_t wo = ((size_t)(st * (COUT / 16) + cbase / 16 + j) * 64 + lane) * 8;
                const bf16x8 b = as_bf(ld16(gp + wo));
#pragma unroll
                for (int t = 0; t < R * T; ++t) acc[t][j] = mfma(av[t], b, acc[t][j]);
                if (q != PAR) {
                    const bf16x8 bl = as_bf(ld16(gl + wo));
#pragma unroll
                    for (int t = 0; t < R * T; ++t) acc[t][j] = mfma(av[t], bl, acc[t][j]);
                }
            }
        }
    };
    switch (par) {
    case 0: contract(Const<0>{}); break;
    case 1: contract(Const<1>{}); break;
    case 2: contract(Const<2>{}); break;
    default: contract(Const<3>{}); break;
    }
    __shared__ EpiTile<NT> st[4];
#pragma unroll
    for (int t = 0; t < R * T; ++t)
        epilogue_tile(st[par], acc[t], lane, [&](int pix, int c8, f32x4 lo, f32x4 hi) {
            const int nn = c0 + t % T * 16 + pix, m = m0 + t / T;
            if (!live || nn >= Ws || m >= Hs) return;
            const size_t p = ((size_t)nimg * Ho + 2 * m + py) * Wo + 2 * nn + px;
            const int co = cbase + c8;
            fwd_store8<SKIP>(out + p * COUT + co, lo, hi, bias + co, SKIP ? skip + p * COUT + co : nullptr);
        });
}

// ============================================================================
// backward data: gradient at the conv input (the source, for an upsampled
// input), then + skip gradient, then the source's relu mask
// ============================================================================
// backward data of an upsampled layer: the adjoint of the parity-folded
// forward.  Source pixel (m, n) collects, for each output parity (py, px)
// and source offset (a, b), the output pixel (2 m' + py, 2 n' + px) with
// m' = m + 1 - py - a, n' = n + 1 - px - b, on the same split folded
// weights as the forward (high and low halves; 28 COUT multiply-adds per
// source channel instead of 36 COUT).  Then the source's relu mask.
//
// A workgroup takes R = 4 / NS source rows x 16 T columns; it stages the
// (2 R + 2) x (32 T + 2) output pixels those collect from in LDS once (each is
// read by four source pixels), and each wave computes one row x CIN / NS
// channels, the weights in fragment order so that a load reads whole lines.
// Bound by the latency of a K step (weights from L2), so the steps are unrolled
// in full: where the low half is loaded is then known, no branch ends a block,
// and the loads of several steps are in flight.  Layers d1, d2, d3 at
// 8 x 256 x 256: 31, 22 and 20 us; in a loop with that branch 37, 43 and 51;
// gathered from global memory per tap, the 16 rows of a weight fragment apart,
// 72, 77 and 43.
template <int CIN, int COUT, int T, int NS>
__global__ __launch_bounds__(256) void k_conv_bwd_data_up(const uint16_t *gpre, const uint16_t *tu,
                                                          const uint16_t *act, uint16_t *gout, int N, int Hs, int Ws)
{
    static_assert(NS == 1 || NS == 2 || NS == 4, "channel split must divide the 4 waves of a workgroup");
    static_assert(COUT % 32 == 0, "a K step is 32 output channels of one (parity, offset)");
    constexpr int K16 = 16 * COUT;
    constexpr int NT = CIN / 16 / NS, R = 4 / NS;
    constexpr int IR = 2 * R + 2, IC = 32 * T + 2;
    constexpr int RS = COUT * 2 + 16;   // +16 bytes: neighbouring pixels' fragments start on different banks
    __shared__ __attribute__((aligned(16))) unsigned char tile[IR * IC * RS];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6, r = lane & 15, gq = lane >> 4;
    const int Ho = 2 * Hs, Wo = 2 * Ws;
    const int tx = (Ws + 16 * T - 1) / (16 * T), ty = (Hs + R - 1) / R;
    const long ntiles = (long)N * ty * tx;
    const long wt = xcd_band_tile(ntiles);
    const bool live = wt < ntiles;
    const long gt = live ? wt : 0;
    const int xt = (int)(gt % tx);
    const long nyt = gt / tx;
    const int nimg = (int)(nyt / ty), m0 = (int)(nyt - (long)nimg * ty) * R, n0 = xt * 16 * T;
    stage_tile<COUT, IR, IC, RS, true>(tile, gpre, nimg, Ho, Wo, 2 * m0 - 1, 2 * n0 - 1, live);
    const int yy = w / NS, cbase = (w % NS) * (CIN / NS);
    f32x4 acc[T][NT];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t *th = tu + (size_t)cbase / 16 * 512 + lane * 8;
    const uint16_t *tl = th + (size_t)CIN * K16;   // low halves
#pragma unroll
    for (int st = 0; st < K16 / 32; ++st) {
        const int pq = st / (COUT / 32), co = (st - pq * (COUT / 32)) * 32 + gq * 8;
        const int py = pq >> 3, px = (pq >> 2) & 1, a = (pq >> 1) & 1, b = pq & 1;
        const bool split = (pq & 3) != (pq >> 2);   // offset (a, b) != (py, px): two or four taps
        // output row 2 m' + py = 2 m + 2 - py - 2 a of source row m, counted from 2 m0 - 1; columns likewise
        const unsigned char *src = tile + ((2 * yy + 3 - py - 2 * a) * IC + (1 - px) * (IC / 2) + r + 1 - b) * RS + co * 2;
        bf16x8 av[T];
#pragma unroll
        for (int t = 0; t < T; ++t) av[t] = as_bf(*reinterpret_cast<const u32x4 *>(src + 16 * t * RS));
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const size_t wo = (size_t)(st * (CIN / 16) + j) * 512;
            const bf16x8 bv = as_bf(ld16(th + wo));
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t][j] = mfma(av[t], bv, acc[t][j]);
            if (split) {
                const bf16x8 bl = as_bf(ld16(tl + wo));
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t][j] = mfma(av[t], bl, acc[t][j]);
            }
        }
    }
    __shared__ EpiTile<NT> st[4];
    const int m = m0 + yy;
#pragma unroll
    for (int t = 0; t < T; ++t)
        epilogue_tile(st[w], acc[t], lane, [&](int pix, int c8, f32x4 lo, f32x4 hi) {
            const int n = n0 + t * 16 + pix;
            if (!live || m >= Hs || n >= Ws) return;
            const size_t o = (((size_t)nimg * Hs + m) * Ws + n) * CIN + cbase + c8;
            bwd_store8<false>(gout + o, lo, hi, nullptr, act + o);
        });
}

// backward data of a stride-2 layer by input parity: input pixel
// (2m + py, 2n + px) receives gradient only through the taps ky = 1 (py = 0)
// or ky in {0, 2} (py = 1), likewise kx, from output pixel
// ((iy + 1 - ky) / 2, (ix + 1 - kx) / 2) -- 1, 2 or 4 of the 9 taps; so the
// four parities of (m, n) use every tap once, on the gradients of output
// pixels (m, n) to (m + 1, n + 1).  The skip gradient and the relu mask are
// fused into the store.
//
// A workgroup takes R = 4 / NS rows m x 16 T columns n; it stages their
// (R + 1) x (16 T + 1) gradient pixels in LDS once, and each wave computes the
// four parities of one row for CIN / NS channels: a weight fragment (in
// fragment order, whole lines a load) serves T products, a 2 x 2 of input pixels
// leaves one wave.  Layers e2, e3, e4 at 8 x 256 x 256: 30, 15 and 11 us
// (per parity and from global memory, the 16 rows of a weight fragment apart:
// 66, 22 and 15); e2 moves 117 MB, 23 us at a copy's rate.
template <int CIN, int COUT, bool SKIP, int T, int NS>
__global__ __launch_bounds__(256) void k_conv_bwd_data_s2(const uint16_t *gpre, int Ho, int Wo, const uint16_t *tw,
                                                          const uint16_t *skipg, const uint16_t *act, uint16_t *gout,
                                                          int N, int Hq, int Wq)
{
    static_assert(NS == 1 || NS == 2 || NS == 4, "channel split must divide the 4 waves of a workgroup");
    static_assert(COUT % 32 == 0, "a K step is 32 output channels of one tap");
    constexpr int NT = CIN / 16 / NS, R = 4 / NS;
    constexpr int IR = R + 1, IC = 16 * T + 1;
    constexpr int RS = COUT * 2 + 16;   // +16 bytes: neighbouring pixels' fragments start on different banks
    __shared__ __attribute__((aligned(16))) unsigned char tile[IR * IC * RS];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6, r = lane & 15, gq = lane >> 4;
    const int Hh = (Hq + 1) >> 1, Wh = (Wq + 1) >> 1;
    const int tx = (Wh + 16 * T - 1) / (16 * T), ty = (Hh + R - 1) / R;
    const long ntiles = (long)N * ty * tx;
    const long wt = xcd_band_tile(ntiles);
    const bool live = wt < ntiles;
    const long gt = live ? wt : 0;
    const int xt = (int)(gt % tx);
    const long nyt = gt / tx;
    const int nimg = (int)(nyt / ty), m0 = (int)(nyt - (long)nimg * ty) * R, n0 = xt * 16 * T;
    stage_tile<COUT, IR, IC, RS>(tile, gpre, nimg, Ho, Wo, m0, n0, live);
    const int yy = w / NS, cbase = (w % NS) * (CIN / NS);
    f32x4 acc[4][T][NT];   // [py * 2 + px]
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[p][t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned char *src = tile + (yy * IC + r) * RS + gq * 16;
    const uint16_t *tf = tw + (size_t)cbase / 16 * 512 + lane * 8;
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const int par = (ky != 1) * 2 + (kx != 1);
            const int off = ((ky == 0) * IC + (kx == 0)) * RS;   // tap 0 reads the next output row / column
#pragma unroll
            for (int c = 0; c < COUT / 32; ++c) {
                bf16x8 av[T];
#pragma unroll
                for (int t = 0; t < T; ++t)
                    av[t] = as_bf(*reinterpret_cast<const u32x4 *>(src + off + c * 64 + 16 * t * RS));
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const size_t wo = (size_t)(((ky * 3 + kx) * (COUT / 32) + c) * (CIN / 16) + j) * 512;
                    const bf16x8 bv = as_bf(ld16(tf + wo));
#pragma unroll
                    for (int t = 0; t < T; ++t) acc[par][t][j] = mfma(av[t], bv, acc[par][t][j]);
                }
            }
        }
    __shared__ EpiTile<NT> st[4];
#pragma unroll
    for (int py = 0; py < 2; ++py) {
        const int iy = 2 * (m0 + yy) + py;
        const size_t prow = ((size_t)nimg * Hq + iy) * Wq;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int px = 0; px < 2; ++px)
                epilogue_tile(st[w], acc[py * 2 + px][t], lane, [&](int pix, int c8, f32x4 lo, f32x4 hi) {
                    const int ix = 2 * (n0 + t * 16 + pix) + px;
                    if (!live || iy >= Hq || ix >= Wq) return;
                    const size_t o = (prow + ix) * CIN + cbase + c8;
                    bwd_store8<SKIP>(gout + o, lo, hi, SKIP ? skipg + o : nullptr, act + o);
                });
    }
}

// ============================================================================
// weight gradients: M = cout, N = cin of a tap, K = pixels of a chunk; each
// chunk leaves a partial sum, summed in a fixed order by k_wgrad_reduce
// ============================================================================
// MFMA operands along pixels from a tile that is kept pixel by pixel, as it
// lies in memory: ds_read_tr16_b64 gives lane i of each 16 column i of four
// rows, whose 8-byte pieces the lanes address (lane i: row i / 4, columns
// 4 (i % 4) .. + 3).  Two reads make the operand: channel r of pixels gq * 8 ..
// + 7, `pitch` bytes apart from `base`.  The pitch is an odd number of 32
// bytes, so the four rows of a read lie on different banks.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 pixel_pieces(const unsigned char *p, int pitch)   // p: this lane's first piece
{
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 4 * pitch));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ bf16x8 pixel_operand(const unsigned char *base, int pitch, int lane)
{
    const int i = lane & 15, gq = lane >> 4;
    return pixel_pieces(base + (gq * 8 + (i >> 2)) * pitch + (i & 3) * 8, pitch);
}

// Past the right and lower border a block's gradient pixels are zeros, but a tap
// still leads from some of them to input pixels of the image, and a zero times
// an infinity or a NaN there would spoil a sum it has no part in.  In blocks
// across a border (`ragged`) the operand keeps the first `left` pixels of its
// row, and rows past the border are left out.
__device__ __forceinline__ bf16x8 first_pixels(bf16x8 b, int left, int lane)
{
    const int n = left - (lane >> 4) * 8;
    u32x4 v = __builtin_bit_cast(u32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] &= n >= 2 * i + 2 ? 0xffffffffu : (n == 2 * i + 1 ? 0xffffu : 0u);
    return as_bf(v);
}

// Weight gradient of an upsampled layer on its parity-folded taps:
// partial[chunk][co][tap][ci], tap = (py * 2 + px) * 4 + a * 2 + b, over source
// pixels (m, n), the gradient at (2m + py, 2n + px) times the source at
// (m + py - 1 + a, n + px - 1 + b).
//
// A workgroup takes one chunk (a run of blocks of 4 rows x 32 columns), one
// output parity and 64 input channels; wave (a, b) takes that offset.  Of a
// block it stages 4 x 32 gradient and 5 x 33 source pixels, which the four
// offsets share, as they lie in memory, and the transposing LDS reads turn them
// into operands along the pixels; the next block's loads are in flight
// meanwhile.  Bound by those loads' latency.  Tap by tap, with 2-byte
// transposed writes to LDS, d1 / d2 / d3 at 8 x 256 x 256 took 84.5, 33.8 and
// 24.2 us; now 26.0, 18.2 and 13.4.  The bias gradient is one more product, with ones.
template <int CIN, int COUT>
__global__ __launch_bounds__(256) void k_conv_wgrad_up(const uint16_t *gpre, const uint16_t *in, int Hs, int Ws, int N,
                                                       float *partial, float *partial_b, int per, int nchunk)
{
    constexpr int R = kWgradRows, C = kWgradCols, MT = COUT / 16, NT = 4, NG = CIN / 64;
    constexpr int GP = COUT * 2 + 32, IP = 64 * 2 + 32;   // bytes per pixel in LDS
    constexpr int GV = R * C * (COUT / 8), IV = (R + 1) * (C + 1) * 8;   // 16-byte vectors of a block
    constexpr int GQ = (GV + 255) / 256, IQ = (IV + 255) / 256;
    __shared__ __attribute__((aligned(16))) unsigned char gt[R * C * GP];
    __shared__ __attribute__((aligned(16))) unsigned char it[(R + 1) * (C + 1) * IP];
    // the parities and channel groups of a chunk get linear indices of one
    // residue mod 8: one XCD, whose L2 they share the chunk's pixels in
    const int id = (int)blockIdx.x, slot = id >> 3;
    const int chunk = (id & 7) + 8 * (slot / (4 * NG)), sub = slot % (4 * NG);
    if (chunk >= nchunk) return;
    const int par = sub & 3, py = par >> 1, px = par & 1, cg = (sub >> 2) * 64;
    const int w = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, r = lane & 15, gq = lane >> 4;
    const int bx = (Ws + C - 1) / C, by = (Hs + R - 1) / R;
    const long nb = (long)N * by * bx, b0 = (long)chunk * per, b1 = b0 + per < nb ? b0 + per : nb;
    u32x4 gv[GQ], iv[IQ];
    int m0 = 0, c0 = 0;   // first row and column of the block loaded last
    auto load = [&](long blk) {
        const int xb = (int)(blk % bx);
        const long yb = blk / bx;
        const int n = (int)(yb / by);
        m0 = (int)(yb - (long)n * by) * R;
        c0 = xb * C;
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q, pix = v / (COUT / 8), cv = (v % (COUT / 8)) * 8;
            const int m = m0 + pix / C, c = c0 + pix % C;
            gv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < GV && m < Hs && c < Ws)
                gv[q] = ld16(gpre + (((size_t)n * 2 * Hs + 2 * m + py) * (2 * (size_t)Ws) + 2 * c + px) * COUT + cv);
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q, pix = v / 8, cv = (v % 8) * 8;
            const int sy = m0 + py - 1 + pix / (C + 1), sx = c0 + px - 1 + pix % (C + 1);
            iv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < IV && sy >= 0 && sy < Hs && sx >= 0 && sx < Ws)
                iv[q] = ld16(in + (((size_t)n * Hs + sy) * Ws + sx) * CIN + cg + cv);
        }
    };
    f32x4 acc[MT][NT], accb[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const u32x4 one2 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bf16x8 ones = as_bf(one2);
    const unsigned char *ip = it + ((w >> 1) * (C + 1) + (w & 1)) * IP;
    if (b0 < b1) load(b0);
    for (long blk = b0; blk < b1; ++blk) {
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q;
            if (v < GV) *reinterpret_cast<u32x4 *>(gt + (v / (COUT / 8)) * GP + (v % (COUT / 8)) * 16) = gv[q];
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q;
            if (v < IV) *reinterpret_cast<u32x4 *>(it + (v / 8) * IP + (v % 8) * 16) = iv[q];
        }
        __syncthreads();
        const int rows = Hs - m0, cols = Ws - c0;
        if (blk + 1 < b1) load(blk + 1);
        auto products = [&](auto ragged) {
#pragma unroll
            for (int y = 0; y < R; ++y) {
                if (decltype(ragged)::v && y >= rows) continue;
                bf16x8 a[MT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = pixel_operand(gt + y * C * GP + i * 32, GP, lane);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    bf16x8 b = pixel_operand(ip + y * (C + 1) * IP + j * 32, IP, lane);
                    if (decltype(ragged)::v) b = first_pixels(b, cols, lane);
#pragma unroll
                    for (int i = 0; i < MT; ++i) acc[i][j] = mfma(a[i], b, acc[i][j]);
                }
                if (w == 0 && cg == 0)
#pragma unroll
                    for (int i = 0; i < MT; ++i) accb[i] = mfma(a[i], ones, accb[i]);
            }
        };
        if (rows >= R && cols >= C)
            products(Const<0>{});
        else
            products(Const<1>{});
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = i * 16 + gq * 4 + e;
            float *o = partial + (((size_t)chunk * COUT + co) * 16 + par * 4 + w) * CIN + cg + r;
#pragma unroll
            for (int j = 0; j < NT; ++j) o[j * 16] = acc[i][j][e];
            if (w == 0 && cg == 0 && r == 0) partial_b[((size_t)chunk * 4 + par) * COUT + co] = accb[i][e];
        }
}

// Weight gradient of a stride-2 layer: partial[chunk][co][tap][ci], the
// gradient at (m, n) times the input at (2m + ky - 1, 2n + kx - 1).
//
// A workgroup of 8 waves takes one chunk (a run of blocks of 4 rows x 32
// columns), 32 input and 64 output channels and all 9 taps.  Of a block it
// stages 4 x 32 gradient and 9 x 65 input pixels, the even columns before the
// odd ones, so that a tap's pixels lie side by side; wave (h, i) takes output
// channels 16 i .. + 15 of rows 2 h and 2 h + 1, and the two halves are added
// at the end.  The next block's loads are in flight meanwhile.  Tap by tap, with
// 2-byte transposed writes to LDS, e2 / e3 / e4 at 8 x 256 x 256 took 33.9,
// 22.6 and 13.5 us; now 19.8, 13.7 and 13.8.  The bias gradient is one more product, with ones.
template <int CIN, int COUT>
__global__ __launch_bounds__(512) void k_conv_wgrad_s2(const uint16_t *gpre, const uint16_t *in, int Hs, int Ws, int N,
                                                       int Ho, int Wo, float *partial, float *partial_b, int per,
                                                       int nchunk)
{
    constexpr int R = kWgradRows, C = kWgradCols, NB = 512;
    constexpr int NGI = CIN / 32, NSUB = NGI * (COUT / 64);
    constexpr int GP = 64 * 2 + 32, IP = 32 * 2 + 32;   // bytes per pixel in LDS
    constexpr int IR = 2 * R + 1, IC = 2 * C + 1, ODD = C + 1;
    constexpr int GV = R * C * 8, IV = IR * IC * 4;     // 16-byte vectors of a block
    constexpr int GQ = (GV + NB - 1) / NB, IQ = (IV + NB - 1) / NB;
    constexpr int NA = 19;   // 9 taps x 2 tiles of input channels, and the bias
    static_assert(R == 4, "two halves of two rows");
    constexpr int TILE = R * C * GP + IR * IC * IP, SUMS = 4 * NA * 64 * 16;
    __shared__ __attribute__((aligned(16))) unsigned char lds[TILE > SUMS ? TILE : SUMS];
    unsigned char *const gt = lds, *const it = lds + R * C * GP;
    const int id = (int)blockIdx.x, slot = id >> 3;
    const int chunk = (id & 7) + 8 * (slot / NSUB), sub = slot % NSUB;
    if (chunk >= nchunk) return;
    const int ci0 = (sub % NGI) * 32, co0 = (sub / NGI) * 64;
    const int w = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, r = lane & 15, gq = lane >> 4;
    const int h = w >> 2, mt = w & 3;
    const int bx = (Wo + C - 1) / C, by = (Ho + R - 1) / R;
    const long nb = (long)N * by * bx, b0 = (long)chunk * per, b1 = b0 + per < nb ? b0 + per : nb;
    u32x4 gv[GQ], iv[IQ];
    int m0 = 0, c0 = 0;   // first row and column of the block loaded last
    auto load = [&](long blk) {
        const int xb = (int)(blk % bx);
        const long yb = blk / bx;
        const int n = (int)(yb / by);
        m0 = (int)(yb - (long)n * by) * R;
        c0 = xb * C;
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + NB * q, pix = v / 8, cv = (v % 8) * 8;
            const int m = m0 + pix / C, c = c0 + pix % C;
            gv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < GV && m < Ho && c < Wo) gv[q] = ld16(gpre + (((size_t)n * Ho + m) * Wo + c) * COUT + co0 + cv);
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + NB * q, pix = v / 4, cv = (v % 4) * 8;
            const int sy = 2 * m0 - 1 + pix / IC, sx = 2 * c0 - 1 + pix % IC;
            iv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < IV && sy >= 0 && sy < Hs && sx >= 0 && sx < Ws)
                iv[q] = ld16(in + (((size_t)n * Hs + sy) * Ws + sx) * CIN + ci0 + cv);
        }
    };
    f32x4 acc[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 one2 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bf16x8 ones = as_bf(one2);
    if (b0 < b1) load(b0);
    for (long blk = b0; blk < b1; ++blk) {
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + NB * q;
            if (v < GV) *reinterpret_cast<u32x4 *>(gt + (v / 8) * GP + (v % 8) * 16) = gv[q];
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + NB * q, pix = v / 4, x = pix % IC;
            if (v < IV)
                *reinterpret_cast<u32x4 *>(it + ((pix / IC) * IC + (x & 1) * ODD + (x >> 1)) * IP + (v % 4) * 16) = iv[q];
        }
        __syncthreads();
        const int rows = Ho - m0, cols = Wo - c0;
        if (blk + 1 < b1) load(blk + 1);
        auto products = [&](auto ragged) {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                if (decltype(ragged)::v && 2 * h + y >= rows) continue;
                const bf16x8 a = pixel_operand(gt + (2 * h + y) * C * GP + mt * 32, GP, lane);
#pragma unroll
                for (int tap = 0; tap < 9; ++tap) {
                    const int ky = tap / 3, kx = tap % 3;
                    const unsigned char *p = it + ((2 * (2 * h + y) + ky) * IC + (kx & 1) * ODD + (kx >> 1)) * IP;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        bf16x8 b = pixel_operand(p + j * 32, IP, lane);
                        if (decltype(ragged)::v) b = first_pixels(b, cols, lane);
                        acc[tap * 2 + j] = mfma(a, b, acc[tap * 2 + j]);
                    }
                }
                if (ci0 == 0) acc[18] = mfma(a, ones, acc[18]);
            }
        };
        if (rows >= R && cols >= C)
            products(Const<0>{});
        else
            products(Const<1>{});
        __syncthreads();
    }
    f32x4 *const sums = reinterpret_cast<f32x4 *>(lds);
    if (h == 1)
#pragma unroll
        for (int j = 0; j < NA; ++j) sums[(mt * NA + j) * 64 + lane] = acc[j];
    __syncthreads();
    if (h == 0) {
#pragma unroll
        for (int j = 0; j < NA; ++j) acc[j] += sums[(mt * NA + j) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = co0 + mt * 16 + gq * 4 + e;
            float *o = partial + ((size_t)chunk * COUT + co) * 9 * CIN + ci0 + r;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                for (int j = 0; j < 2; ++j) o[tap * CIN + j * 16] = acc[tap * 2 + j][e];
            if (ci0 == 0 && r == 0) partial_b[(size_t)chunk * COUT + co] = acc[18][e];
        }
    }
}

// Weight gradient of the first layer (8 padded input channels, stride 1):
// partial[chunk][co][tap][ci].  A workgroup takes blocks of 8 rows x 32
// columns, staged as they lie, and all 9 taps: a tile of 16 columns is two
// taps of 8 channels, whose pixels the lanes of a transposing read address
// each for itself (the tenth tap repeats the ninth and is dropped).  Wave w
// takes rows 2 w and 2 w + 1, and the four sums are added at the end.
// Staged per tap with 2-byte transposed writes to LDS it took 38.3 us at
// 8 x 256 x 256, now 14.9.
template <int COUT>
__global__ __launch_bounds__(256) void k_conv_wgrad_c8(const uint16_t *gpre, const uint16_t *in, int H, int W, int N,
                                                       float *partial, float *partial_b, int per)
{
    constexpr int R = kWgradRows0, C = kWgradCols, MT = COUT / 16, NT = 5;
    constexpr int GP = COUT * 2 + 32;   // bytes per gradient pixel in LDS; an input pixel has 16
    constexpr int IC = C + 2;
    constexpr int GV = R * C * (COUT / 8), IV = (R + 2) * IC;   // 16-byte vectors of a block
    constexpr int GQ = (GV + 255) / 256, IQ = (IV + 255) / 256;
    constexpr int NA = MT * (NT + 1);   // the products and the bias
    static_assert(R == 8, "two rows a wave");
    constexpr int TILE = R * C * GP + IV * 16, SUMS = 4 * NA * 64 * 16;
    __shared__ __attribute__((aligned(16))) unsigned char lds[TILE > SUMS ? TILE : SUMS];
    unsigned char *const gt = lds, *const it = lds + R * C * GP;
    const int w = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, r = lane & 15, gq = lane >> 4;
    const int bx = (W + C - 1) / C, by = (H + R - 1) / R;
    const long nb = (long)N * by * bx, b0 = (long)blockIdx.x * per, b1 = b0 + per < nb ? b0 + per : nb;
    u32x4 gv[GQ], iv[IQ];
    int m0 = 0, c0 = 0;   // first row and column of the block loaded last
    auto load = [&](long blk) {
        const int xb = (int)(blk % bx);
        const long yb = blk / bx;
        const int n = (int)(yb / by);
        m0 = (int)(yb - (long)n * by) * R;
        c0 = xb * C;
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q, pix = v / (COUT / 8), cv = (v % (COUT / 8)) * 8;
            const int m = m0 + pix / C, c = c0 + pix % C;
            gv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < GV && m < H && c < W) gv[q] = ld16(gpre + (((size_t)n * H + m) * W + c) * COUT + cv);
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q;
            const int sy = m0 - 1 + v / IC, sx = c0 - 1 + v % IC;
            iv[q] = u32x4{0u, 0u, 0u, 0u};
            if (v < IV && sy >= 0 && sy < H && sx >= 0 && sx < W) iv[q] = ld16(in + (((size_t)n * H + sy) * W + sx) * 8);
        }
    };
    // where this lane's piece of tile j lies, from a row's first pixel: tap 2 j
    // or 2 j + 1 by its column, 4 channels of it
    int off[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int tp = 2 * j + ((lane >> 1) & 1), tap = tp < 9 ? tp : 8;
        off[j] = ((tap / 3) * IC + tap % 3 + gq * 8 + ((lane & 15) >> 2)) * 16 + (lane & 1) * 8;
    }
    f32x4 acc[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 one2 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bf16x8 ones = as_bf(one2);
    if (b0 < b1) load(b0);
    for (long blk = b0; blk < b1; ++blk) {
#pragma unroll
        for (int q = 0; q < GQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q;
            if (v < GV) *reinterpret_cast<u32x4 *>(gt + (v / (COUT / 8)) * GP + (v % (COUT / 8)) * 16) = gv[q];
        }
#pragma unroll
        for (int q = 0; q < IQ; ++q) {
            const int v = (int)threadIdx.x + 256 * q;
            if (v < IV) *reinterpret_cast<u32x4 *>(it + v * 16) = iv[q];
        }
        __syncthreads();
        const int rows = H - m0, cols = W - c0;
        if (blk + 1 < b1) load(blk + 1);
        auto products = [&](auto ragged) {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int row = 2 * w + y;
                if (decltype(ragged)::v && row >= rows) continue;
                bf16x8 a[MT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = pixel_operand(gt + row * C * GP + i * 32, GP, lane);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    bf16x8 b = pixel_pieces(it + row * IC * 16 + off[j], 16);
                    if (decltype(ragged)::v) b = first_pixels(b, cols, lane);
#pragma unroll
                    for (int i = 0; i < MT; ++i) acc[i * (NT + 1) + j] = mfma(a[i], b, acc[i * (NT + 1) + j]);
                }
#pragma unroll
                for (int i = 0; i < MT; ++i) acc[i * (NT + 1) + NT] = mfma(a[i], ones, acc[i * (NT + 1) + NT]);
            }
        };
        if (rows >= R && cols >= C)
            products(Const<0>{});
        else
            products(Const<1>{});
        __syncthreads();
    }
    f32x4 *const sums = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
    for (int j = 0; j < NA; ++j) sums[(w * NA + j) * 64 + lane] = acc[j];
    __syncthreads();
    for (int j = w; j < NA; j += 4) {
        const f32x4 s = (sums[j * 64 + lane] + sums[(NA + j) * 64 + lane]) +
                        (sums[(2 * NA + j) * 64 + lane] + sums[(3 * NA + j) * 64 + lane]);
        const int i = j / (NT + 1), nt = j % (NT + 1), col = nt * 16 + r;   // col = tap * 8 + ci
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = i * 16 + gq * 4 + e;
            if (nt == NT) {
                if (r == 0) partial_b[(size_t)blockIdx.x * COUT + co] = s[e];
            } else if (col < 72) {
                partial[((size_t)blockIdx.x * COUT + co) * 72 + col] = s[e];
            }
        }
    }
}

// fixed-order sum of the chunk partials into the fp32 gradient vector: a
// workgroup takes 64 consecutive partial entries j (weights with the padded
// input channels, then the biases); wave sl sums chunks sl, sl + 16, ... with
// eight or sixteen loads in flight per lane, and the wave sums are added in
// LDS.  Bound by the latency of those loads, so a workgroup has 16 waves: the
// folded layers at 8 x 256 x 256 9.6 us (with 4 waves, and half the chunks, 12.7).
constexpr int kReduceWaves = 16;
template <bool FOLD>
__global__ __launch_bounds__(64 * kReduceWaves) void k_wgrad_reduce(const float *partial, const float *partial_b, int chunks,
                                                      int cout, int cin, int cinp, float *dw, float *db)
{
    constexpr int S = kReduceWaves;
    __shared__ float red[S][64];
    const int nw = cout * 9 * cinp;
    const int j = (int)blockIdx.x * 64 + ((int)threadIdx.x & 63), sl = (int)threadIdx.x >> 6;
    const bool isw = j < nw, valid = j < nw + cout;
    float s = 0.0f;
    if (valid && !FOLD) {
        const float *src = isw ? partial + j : partial_b + (j - nw);
        const size_t stride = isw ? (size_t)nw : (size_t)cout;
        float a[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = 0.0f;
        int c = sl;
        for (; c + 7 * S < chunks; c += 8 * S)
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] += src[(size_t)(c + S * k) * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (c + S * k < chunks) a[k] += src[(size_t)(c + S * k) * stride];
        s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    } else if (valid) {
        // FOLD: partial[chunk][co][16][cinp] over (output parity, source
        // offset); tap (ky, kx) of parity (py, px) sits at offset
        // a = floor((py + ky - 1) / 2) + 1 - py, likewise b; bias partials
        // [chunk][4 parities][cout]
        int off[4];
        size_t stride;
        const float *src;
        if (isw) {
            const int co = j / (9 * cinp), rem = j - co * 9 * cinp, tap = rem / cinp, ci = rem - (rem / cinp) * cinp;
            const int ky = tap / 3, kx = tap - (tap / 3) * 3;
#pragma unroll
            for (int par = 0; par < 4; ++par) {
                const int py = par >> 1, px = par & 1;
                const int fa = ((py + ky - 1) >> 1) + 1 - py, fb = ((px + kx - 1) >> 1) + 1 - px;
                off[par] = ((co * 16 + par * 4 + fa * 2 + fb) * cinp) + ci;
            }
            src = partial;
            stride = (size_t)cout * 16 * cinp;
        } else {
#pragma unroll
            for (int par = 0; par < 4; ++par) off[par] = par * cout + (j - nw);
            src = partial_b;
            stride = (size_t)4 * cout;
        }
        float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int c = sl;
        for (; c + 3 * S < chunks; c += 4 * S)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float *q = src + (size_t)(c + S * k) * stride;
                a[k] += (q[off[0]] + q[off[1]]) + (q[off[2]] + q[off[3]]);
            }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + S * k < chunks) {
                const float *q = src + (size_t)(c + S * k) * stride;
                a[k] += (q[off[0]] + q[off[1]]) + (q[off[2]] + q[off[3]]);
            }
        s = (a[0] + a[1]) + (a[2] + a[3]);
    }
    red[sl][threadIdx.x & 63] = s;
    __syncthreads();
    if (sl != 0 || !valid) return;
    const int l = (int)threadIdx.x;
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < S; k += 4) t += (red[k][l] + red[k + 1][l]) + (red[k + 2][l] + red[k + 3][l]);
    if (isw) {
        const int co = j / (9 * cinp), rem = j - co * 9 * cinp, tap = rem / cinp, ci = rem - (rem / cinp) * cinp;
        if (ci < cin) dw[(co * 9 + tap) * cin + ci] = t;
    } else {
        db[j - nw] = t;
    }
}

// ============================================================================
// head: delta = conv(d1, 32 -> 1); out = d + 5 cm delta on valid pixels
// ============================================================================
// One workgroup per 16x16 output tile of one image: the tile's d1 with a
// one-pixel halo (zeros outside the image) is staged in LDS once, 80 bytes a
// pixel (at 64 the 16-byte reads of neighbouring pixels met on the same
// banks), and the 288 weights, the same for every lane, are read through the
// scalar cache.  The sum runs tap by tap, channel by channel, from the bias,
// one fused multiply-add (a single rounding) per term; taps outside the image
// are left out, which only tiles on its border test.  The caller's copy of the
// output is stored here too (a copy of 640x480 was 3.9 us).
// 640x480: 11.8 us, with 64-byte pixels and the test in every tile, to 10.7;
// bound by the 576 vector instructions a pixel (unpack and multiply-add).
__global__ __launch_bounds__(256) void k_head_fwd(const uint16_t *d1, const float *__restrict__ w,
                                                  const float *__restrict__ b, const float *dm, float *out,
                                                  float *out2, int N, int H, int W)
{
    constexpr int PS = 5;   // pitch of a pixel in 16-byte vectors
    __shared__ u32x4 tile[18 * 18 * PS];
    const int tx = (int)blockIdx.x * 16, ty = (int)blockIdx.y * 16, n = (int)blockIdx.z;
    for (int k = threadIdx.x; k < 18 * 18 * 4; k += 256) {
        const int pix = k >> 2, q = k & 3;
        const int iy = ty - 1 + pix / 18, ix = tx - 1 + pix % 18;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (iy >= 0 && iy < H && ix >= 0 && ix < W) v = ld16(d1 + (((size_t)n * H + iy) * W + ix) * 32 + 8 * q);
        tile[pix * PS + q] = v;
    }
    __syncthreads();
    const int lx = (int)threadIdx.x & 15, ly = (int)threadIdx.x >> 4;
    const int x = tx + lx, y = ty + ly;
    if (x >= W || y >= H) return;
    float s = b[0];
    auto sum = [&](auto border) {
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int iy = y + tap / 3 - 1, ix = x + tap % 3 - 1;
            if (decltype(border)::v && (iy < 0 || iy >= H || ix < 0 || ix >= W)) continue;
            const u32x4 *src = tile + ((ly + tap / 3) * 18 + lx + tap % 3) * PS;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32x4 v = src[q];
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(w[tap * 32 + 8 * q + e], bf2f((uint16_t)(v[e >> 1] >> (16 * (e & 1)))), s);
            }
        }
    };
    if (tx > 0 && ty > 0 && tx + 16 < W && ty + 16 < H)
        sum(Const<0>{});
    else
        sum(Const<1>{});
    const size_t p = ((size_t)n * H + y) * W + x;
    const float d = dm[p];
    const float o = d > 0.0f ? d + kCorrScale * s : 0.0f;
    out[p] = o;
    if (out2) out2[p] = o;
}

// masked L1 in four fixed-order steps (no atomics; the same sums every run):
// per-workgroup valid counts, their total, per-workgroup |out - target| sums
// with the gradient, then the mean
__global__ __launch_bounds__(256) void k_loss_count(const float *dm, const float *target, int n, unsigned *part)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    const int c = __syncthreads_count(p < n && dm[p] > 0.0f && target[p] > 0.0f);
    if (threadIdx.x == 0) part[blockIdx.x] = (unsigned)c;
}

__global__ __launch_bounds__(256) void k_loss_total(const unsigned *part, int nwg, unsigned *cnt)
{
    __shared__ unsigned red[256];
    unsigned c = 0u;
    for (int i = (int)threadIdx.x; i < nwg; i += 256) c += part[i];
    red[threadIdx.x] = c;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) cnt[0] = red[0];
}

__global__ __launch_bounds__(256) void k_loss_grad(const float *out, const float *dm, const float *target, int n,
                                                   const unsigned *cnt, float *ddelta, float *part)
{
    __shared__ float red[4];
    const int p = blockIdx.x * 256 + threadIdx.x;
    const float inv_n = *cnt ? 1.0f / (float)*cnt : 0.0f;
    float a = 0.0f;
    if (p < n) {
        float g = 0.0f;
        if (dm[p] > 0.0f && target[p] > 0.0f) {
            const float diff = out[p] - target[p];
            g = diff > 0.0f ? inv_n : (diff < 0.0f ? -inv_n : 0.0f);
            a = diff < 0.0f ? -diff : diff;
        }
        ddelta[p] = kCorrScale * g;
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) a += __shfl_xor(a, m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_loss_final(const float *part, int nwg, const unsigned *cnt, float *loss)
{
    __shared__ float red[256];
    float s = 0.0f;
    for (int i = (int)threadIdx.x; i < nwg; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        loss[0] = *cnt ? red[0] / (float)*cnt : 0.0f;
        loss[1] = (float)*cnt;
    }
}

// Backward of the head over one chunk of rows, d1 and ddelta read once for both:
// the gradient at d1, g[p][c] = sum_tap ddelta[p - off(tap)] w[tap][c] with the
// relu mask of d1, and the weight gradient gathered from the input side,
// dw[tap][c] = sum_p ddelta[p] d1[p + off(tap)][c] = sum_q d1[q][c] ddelta[q - off(tap)].
//
// A workgroup takes segments of 64 pixels of a row, their ddelta with the rows
// and columns around in LDS (zeros outside the image), the next segment's loads
// in flight.  Gradient: four lanes a pixel with eight channels each, whose 72
// weights stay in registers; their loads and stores are one run a wave.  Weight
// gradient: on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32: A row l % 16,
// k = l / 16; B column l % 16, same k; D as above): M = tap (rows past 8 are not
// used), K = pixels, N = channels 2 c and 2 c + 1 of the 32 in two products, so
// that a lane's load is the 4 bytes of its column and a wave's the 256 of four
// pixels; wave w takes pixels 16 w .. + 15.
// partial[j * nchunk + chunk]: j = tap * 32 + c, j = 288 the bias, the sum of
// ddelta.  A pixel on the image's border has no part in the taps whose ddelta
// lies outside, zero here.  That zero times an infinity or a NaN would spread
// it, so a chunk whose sums are not all finite is taken again with the terms of
// such activations on the border led past the products.  Bound by the gradient's vector instructions (18 a channel and pixel
// beside the unpacking) and memory; at 8 x 256 x 256 a kernel each, with a pixel
// a lane 64 bytes apart and the weight gradient on the vector units, took 29.7
// and 52.6 us, now 39 together.
__global__ __launch_bounds__(256) void k_head_bwd(const float *ddelta, const float *__restrict__ wt,
                                                  const uint16_t *__restrict__ d1, uint16_t *__restrict__ g_d1, int N,
                                                  int H, int W, float *__restrict__ partial, int per)
{
    constexpr int SP = 64, DW = SP + 2;
    __shared__ float dl[2][3 * DW];
    __shared__ float red[4][289];
    __shared__ float past[288];   // terms of non-finite activations on the border
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6, r = lane & 15, gq = lane >> 4;
    const int bx = (W + SP - 1) / SP;
    const long ns = (long)N * H * bx, s0 = (long)blockIdx.x * per, s1 = s0 + per < ns ? s0 + per : ns;
    const int px = (int)threadIdx.x >> 2, oct = (int)threadIdx.x & 3;
    float ws[9][8];
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) ws[k][e] = wt[k * 32 + 8 * oct + e];
    for (int j = (int)threadIdx.x; j < 288; j += 256) past[j] = 0.0f;
    const int tap = r < 9 ? r : 0;
    const int at = (2 - tap / 3) * DW + 2 - tap % 3 + 16 * w + gq;   // ddelta of q - off(tap), q = 16 w + gq + 4 k
    float dv = 0.0f;
    uint32_t v[4];
    u32x4 av;
    int c0n = 0, yn = 0;   // the segment loaded last: its first column, row, and image * H + row
    long rown = 0;
    auto load = [&](long s) {
        const long row = s / bx;
        const int c0 = (int)(s - row * bx) * SP;
        const int n = (int)(row / H), y = (int)(row - (long)n * H);
        c0n = c0;
        yn = y;
        rown = row;
        dv = 0.0f;
        if ((int)threadIdx.x < 3 * DW) {
            const int oy = y - 1 + (int)threadIdx.x / DW, ox = c0 - 1 + (int)threadIdx.x % DW;
            if (oy >= 0 && oy < H && ox >= 0 && ox < W) dv = ddelta[((size_t)n * H + oy) * W + ox];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int x = c0 + 16 * w + 4 * k + gq;
            v[k] = 0u;
            if (x < W) v[k] = *reinterpret_cast<const uint32_t *>(d1 + ((size_t)row * W + x) * 32 + 2 * r);
        }
        av = u32x4{0u, 0u, 0u, 0u};
        if (c0 + px < W) av = ld16(d1 + ((size_t)row * W + c0 + px) * 32 + 8 * oct);
    };
    f32x4 acc[2];
    float bsum;
    auto pass = [&](auto border) {
        acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        bsum = 0.0f;
        if (s0 < s1) load(s0);
        for (long s = s0; s < s1; ++s) {
            float *const d = dl[s & 1];
            if ((int)threadIdx.x < 3 * DW) d[threadIdx.x] = dv;
            uint32_t u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = v[k];
            const u32x4 act = av;
            __syncthreads();   // two tiles of ddelta, so that this one barrier also guards the one before
            const int c0 = c0n, y = yn;
            const long row = rown;
            if (s + 1 < s1) load(s + 1);
            if (decltype(border)::v) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = 16 * w + 4 * k + gq, x = c0 + q;
                    const bool edge = x < W && (y == 0 || y == H - 1 || x == 0 || x == W - 1);
                    const bool lo = edge && (u[k] & 0x7f80u) == 0x7f80u, hi = edge && (u[k] & 0x7f800000u) == 0x7f800000u;
                    if (!__any(lo || hi)) continue;
#pragma unroll 1
                    for (int t = 0; t < 9; ++t) {
                        const int oy = y - t / 3 + 1, ox = x - t % 3 + 1;
                        if (oy < 0 || oy >= H || ox < 0 || ox >= W) continue;
                        const float a = d[(2 - t / 3) * DW + 2 - t % 3 + q];
                        if (lo) atomicAdd(&past[t * 32 + 2 * r], a * __uint_as_float(u[k] << 16));
                        if (hi) atomicAdd(&past[t * 32 + 2 * r + 1], a * __uint_as_float(u[k] & 0xffff0000u));
                    }
                    u[k] &= (lo ? 0xffff0000u : ~0u) & (hi ? 0xffffu : ~0u);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float a = d[at + 4 * k];
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, __uint_as_float(u[k] << 16), acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, __uint_as_float(u[k] & 0xffff0000u), acc[1], 0, 0, 0);
                bsum += a;   // of use where the tap is the centre
            }
            float g[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = 0.0f;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const float a = d[(2 - k / 3) * DW + 2 - k % 3 + px];
                if (a != 0.0f)   // a gradient of zero is left out, whatever the weight
#pragma unroll
                    for (int e = 0; e < 8; ++e) g[e] += a * ws[k][e];
            }
            u32x4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v0 = bf2f((uint16_t)(act[e] & 0xffffu)) > 0.0f ? g[2 * e] : 0.0f;
                const float v1 = bf2f((uint16_t)(act[e] >> 16)) > 0.0f ? g[2 * e + 1] : 0.0f;
                ov[e] = bf2(v0, v1);
            }
            if (c0 + px < W) *reinterpret_cast<u32x4 *>(g_d1 + ((size_t)row * W + c0 + px) * 32 + 8 * oct) = ov;
        }
    };
    pass(Const<0>{});
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (gq * 4 + i < 9) finite = finite && isfinite(acc[0][i]) && isfinite(acc[1][i]);
    if (__syncthreads_or(!finite)) pass(Const<1>{});
    bsum += __shfl_xor(bsum, 16);
    bsum += __shfl_xor(bsum, 32);
    if (lane == 4) red[w][288] = bsum;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (gq * 4 + i < 9) red[w][(gq * 4 + i) * 32 + 2 * r + j] = acc[j][i];
    __syncthreads();
    for (int j = (int)threadIdx.x; j < 289; j += 256) {
        const float sum = (red[0][j] + red[1][j]) + (red[2][j] + red[3][j]), p = j < 288 ? past[j] : 0.0f;
        partial[(size_t)j * gridDim.x + blockIdx.x] = p != 0.0f ? sum + p : sum;
    }
}

// fixed-order sum of the head partials: workgroup j sums row j of partial
__global__ __launch_bounds__(256) void k_head_reduce(const float *partial, int chunks, float *dw, float *db)
{
    __shared__ float red[256];
    const int j = (int)blockIdx.x;
    float s = 0.0f;
    for (int c = (int)threadIdx.x; c < chunks; c += 256) s += partial[(size_t)j * chunks + c];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (j < 288)
            dw[j] = red[0];
        else
            db[0] = red[0];
    }
}

// Adam (Kingma & Ba, Algorithm 1); c1 = 1 - beta1^t, c2 = 1 - beta2^t
__global__ __launch_bounds__(256) void k_adam(float *p, const float *g, float *m, float *v, int n, float lr,
                                              float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    p[i] = p[i] - lr * mh / (sqrtf(vh) + eps);
}

// ============================================================================
// launchers
// ============================================================================
static dim3 grid1(long n, int per) { return dim3((unsigned)((n + per - 1) / per)); }

hipError_t launch_make_input(const void *depth, int fmt, int N, int H, int W, uint16_t *x, float *dm, hipStream_t s)
{
    const dim3 g((unsigned)((W + 15) / 16), (unsigned)((H + 15) / 16), (unsigned)N);
    if (fmt == TF_DEPTH_U16_MM)
        hipLaunchKernelGGL(k_make_input<TF_DEPTH_U16_MM>, g, dim3(256), 0, s, depth, N, H, W, x, dm);
    else
        hipLaunchKernelGGL(k_make_input<TF_DEPTH_F32_M>, g, dim3(256), 0, s, depth, N, H, W, x, dm);
    return hipGetLastError();
}

hipError_t launch_pack(const Net &net, const float *params, uint16_t *g, uint16_t *t, hipStream_t s)
{
    PackJobs J = {};
    int at = 0;
    for (int l = 0; l < kLayers - 1; ++l) {
        const LayerDesc &L = net.L[l];
        PackJob &p = J.job[l];
        p.w = params + L.w_off;
        p.g = g + L.g_off;
        p.t = L.t_off >= 0 ? t + L.t_off : nullptr;
        p.cin = L.cin;
        p.cinp = L.cinp;
        p.cout = L.cout;
        p.kp = L.kp;
        p.up = L.up;
        p.n_g = L.up ? 2 * 16 * L.cout * L.cinp : L.cout * L.kp;   // up layers: high and low halves
        p.n_t = p.t ? L.cinp * (L.up ? 2 * 16 : 9) * L.cout : 0;
        J.start[l] = at;
        at += p.n_g > p.n_t ? p.n_g : p.n_t;
    }
    J.start[kLayers - 1] = at;
    hipLaunchKernelGGL(k_pack, grid1(at, 256), dim3(256), 0, s, J);
    return hipGetLastError();
}


hipError_t launch_conv_fwd(int layer, const uint16_t *in, int Hs, int Ws, const uint16_t *g, const float *bias,
                           const uint16_t *skip, uint16_t *out, int N, int Ho, int Wo, hipStream_t s)
{
    // encoder tiles: 4 R / NS output rows x 16 T columns per workgroup, the
    // stride-2 layers splitting their output channels over the 4 waves (R
    // output rows per workgroup); decoder tiles: R source rows x 16 T columns,
    // the smaller layers' channels split over NS workgroups (shapes measured
    // at 640x480 and 8 x 256 x 256)
    const dim3 b(256);
    auto enc_grid = [&](int T, int NS, int R) {
        const int rows = R * (4 / NS);
        const long nt = (long)N * ((Ho + rows - 1) / rows) * ((Wo + 16 * T - 1) / (16 * T));
        return dim3((unsigned)((nt + 7) / 8 * 8));
    };
    auto up_grid = [&](int T, int NS, int R) {
        const long nt = (long)N * ((Hs + R - 1) / R) * ((Ws + 16 * T - 1) / (16 * T)) * NS;
        return dim3((unsigned)((nt + 7) / 8 * 8));
    };
    if (layer < 4 && skip) return hipErrorInvalidValue;
    if (layer >= 4 && (Ho != 2 * Hs || Wo != 2 * Ws)) return hipErrorInvalidValue;
    switch (layer) {
    case 0: hipLaunchKernelGGL((k_conv_fwd<8, 32, 1, 2, 1, 1>), enc_grid(2, 1, 1), b, 0, s, in, Hs, Ws, g, bias, out, N, Ho, Wo); break;
    case 1: hipLaunchKernelGGL((k_conv_fwd<32, 64, 2, 2, 4, 2>), enc_grid(2, 4, 2), b, 0, s, in, Hs, Ws, g, bias, out, N, Ho, Wo); break;
    case 2: hipLaunchKernelGGL((k_conv_fwd<64, 64, 2, 1, 4, 2>), enc_grid(1, 4, 2), b, 0, s, in, Hs, Ws, g, bias, out, N, Ho, Wo); break;
    case 3: hipLaunchKernelGGL((k_conv_fwd<64, 128, 2, 1, 4, 1>), enc_grid(1, 4, 1), b, 0, s, in, Hs, Ws, g, bias, out, N, Ho, Wo); break;
    case 4: hipLaunchKernelGGL((k_conv_fwd_up<128, 64, true, 1, 4, 2>), up_grid(1, 4, 2), b, 0, s, in, Hs, Ws, g, bias, skip, out, N); break;
    case 5: hipLaunchKernelGGL((k_conv_fwd_up<64, 64, true, 1, 2, 4>), up_grid(1, 2, 4), b, 0, s, in, Hs, Ws, g, bias, skip, out, N); break;
    case 6: hipLaunchKernelGGL((k_conv_fwd_up<64, 32, true, 1, 1, 4>), up_grid(1, 1, 4), b, 0, s, in, Hs, Ws, g, bias, skip, out, N); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_head_fwd(const uint16_t *d1, const float *w, const float *b, const float *dm, float *out,
                           float *out2, int N, int H, int W, hipStream_t s)
{
    hipLaunchKernelGGL(k_head_fwd, dim3((W + 15) / 16, (H + 15) / 16, N), dim3(256), 0, s, d1, w, b, dm, out, out2, N, H, W);
    return hipGetLastError();
}

// scratch: [0] the valid count (uint32), then loss_scratch_words(n_pix) - 4
// words of per-workgroup counts and sums; loss: [0] mean, [1] count
hipError_t launch_loss(const float *out, const float *dm, const float *target, int n_pix, float *ddelta,
                       float *scratch, float *loss, hipStream_t s)
{
    const int nwg = (n_pix + 255) / 256;
    unsigned *cnt = reinterpret_cast<unsigned *>(scratch);
    unsigned *pc = cnt + 4;
    float *ps = scratch + 4 + nwg;
    hipLaunchKernelGGL(k_loss_count, dim3(nwg), dim3(256), 0, s, dm, target, n_pix, pc);
    hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(256), 0, s, pc, nwg, cnt);
    hipLaunchKernelGGL(k_loss_grad, dim3(nwg), dim3(256), 0, s, out, dm, target, n_pix, cnt, ddelta, ps);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, ps, nwg, cnt, loss);
    return hipGetLastError();
}

hipError_t launch_head_bwd(const float *ddelta, const float *w, const uint16_t *d1, uint16_t *g_d1, int N, int H,
                           int W, float *partial, int chunks, float *dw, float *db, hipStream_t s)
{
    const long segs = (long)N * H * ((W + 63) / 64);
    const int per = (int)((segs + chunks - 1) / chunks);
    const int nc = (int)((segs + per - 1) / per);
    hipLaunchKernelGGL(k_head_bwd, dim3(nc), dim3(256), 0, s, ddelta, w, d1, g_d1, N, H, W, partial, per);
    hipLaunchKernelGGL(k_head_reduce, dim3(289), dim3(256), 0, s, partial, nc, dw, db);
    return hipGetLastError();
}

hipError_t launch_conv_bwd_data(int layer, const uint16_t *gpre, int Ho, int Wo, const uint16_t *t,
                                const uint16_t *skipg, const uint16_t *act, uint16_t *gout, int N, int Hq, int Wq,
                                hipStream_t s)
{
    const dim3 b(256);
    // 4 / NS rows x 16 T columns per workgroup: of source pixels (upsampled layers) or of 2 x 2 input pixels (stride 2)
    auto tiles = [&](int h, int w, int T, int NS) {
        const long nt = (long)N * ((h + 4 / NS - 1) / (4 / NS)) * ((w + 16 * T - 1) / (16 * T));
        return dim3((unsigned)((nt + 7) / 8 * 8));
    };
    auto up_grid = [&](int T, int NS) { return tiles(Hq, Wq, T, NS); };
    auto s2_grid = [&](int T, int NS) { return tiles((Hq + 1) >> 1, (Wq + 1) >> 1, T, NS); };
    if (layer >= 4 && (Ho != 2 * Hq || Wo != 2 * Wq)) return hipErrorInvalidValue;
    switch (layer) {
    // stride-2 layers: only the taps of each input parity
    case 1: hipLaunchKernelGGL((k_conv_bwd_data_s2<32, 64, true, 1, 2>), s2_grid(1, 2), b, 0, s, gpre, Ho, Wo, t, skipg, act, gout, N, Hq, Wq); break;
    case 2: hipLaunchKernelGGL((k_conv_bwd_data_s2<64, 64, true, 1, 2>), s2_grid(1, 2), b, 0, s, gpre, Ho, Wo, t, skipg, act, gout, N, Hq, Wq); break;
    case 3: hipLaunchKernelGGL((k_conv_bwd_data_s2<64, 128, true, 1, 4>), s2_grid(1, 4), b, 0, s, gpre, Ho, Wo, t, skipg, act, gout, N, Hq, Wq); break;
    // upsampled layers: the adjoint of the parity-folded forward (t holds the folded weights)
    case 4: hipLaunchKernelGGL((k_conv_bwd_data_up<128, 64, 1, 4>), up_grid(1, 4), b, 0, s, gpre, t, act, gout, N, Hq, Wq); break;
    case 5: hipLaunchKernelGGL((k_conv_bwd_data_up<64, 64, 1, 2>), up_grid(1, 2), b, 0, s, gpre, t, act, gout, N, Hq, Wq); break;
    case 6: hipLaunchKernelGGL((k_conv_bwd_data_up<64, 32, 2, 2>), up_grid(2, 2), b, 0, s, gpre, t, act, gout, N, Hq, Wq); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_conv_wgrad(int layer, const uint16_t *gpre, const uint16_t *in, int Hs, int Ws, int N, int Ho,
                             int Wo, float *partial, int chunks, float *dw, float *db, hipStream_t s)
{
    // the decoder layers (4-6) run folded: 16 (parity, offset) taps over the
    // source grid
    const bool fold = layer >= 4;
    const long P = wgrad_blocks(layer, N, fold ? Hs : Ho, fold ? Ws : Wo);
    if (fold && (Ho != 2 * Hs || Wo != 2 * Ws)) return hipErrorInvalidValue;
    const int per = (int)((P + chunks - 1) / chunks);
    const int nc = (int)((P + per - 1) / per);
    float *pb = partial;   // bias partials after the weight partials
    const int nc8 = (nc + 7) / 8 * 8;   // chunks padded to a multiple of 8, the XCDs they are dealt to
    const dim3 b(256);
    int cout = 0, cin = 0, cinp = 0;
    switch (layer) {
    case 0: cout = 32; cin = 3; cinp = 8; pb += (size_t)nc * 32 * 9 * 8;   // all taps per workgroup
        hipLaunchKernelGGL((k_conv_wgrad_c8<32>), dim3(nc), b, 0, s, gpre, in, Ho, Wo, N, partial, pb, per); break;
    case 1: cout = 64; cin = cinp = 32; pb += (size_t)nc * 64 * 9 * 32;
        hipLaunchKernelGGL((k_conv_wgrad_s2<32, 64>), dim3(1 * nc8), dim3(512), 0, s, gpre, in, Hs, Ws, N, Ho, Wo, partial, pb, per, nc); break;
    case 2: cout = 64; cin = cinp = 64; pb += (size_t)nc * 64 * 9 * 64;
        hipLaunchKernelGGL((k_conv_wgrad_s2<64, 64>), dim3(2 * nc8), dim3(512), 0, s, gpre, in, Hs, Ws, N, Ho, Wo, partial, pb, per, nc); break;
    case 3: cout = 128; cin = cinp = 64; pb += (size_t)nc * 128 * 9 * 64;
        hipLaunchKernelGGL((k_conv_wgrad_s2<64, 128>), dim3(4 * nc8), dim3(512), 0, s, gpre, in, Hs, Ws, N, Ho, Wo, partial, pb, per, nc); break;
    case 4: cout = 64; cin = cinp = 128; pb += (size_t)nc * 64 * 16 * 128;
        hipLaunchKernelGGL((k_conv_wgrad_up<128, 64>), dim3(8 * nc8), b, 0, s, gpre, in, Hs, Ws, N, partial, pb, per, nc); break;
    case 5: cout = 64; cin = cinp = 64; pb += (size_t)nc * 64 * 16 * 64;
        hipLaunchKernelGGL((k_conv_wgrad_up<64, 64>), dim3(4 * nc8), b, 0, s, gpre, in, Hs, Ws, N, partial, pb, per, nc); break;
    case 6: cout = 32; cin = cinp = 64; pb += (size_t)nc * 32 * 16 * 64;
        hipLaunchKernelGGL((k_conv_wgrad_up<64, 32>), dim3(4 * nc8), b, 0, s, gpre, in, Hs, Ws, N, partial, pb, per, nc); break;
    default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (fold)
        hipLaunchKernelGGL(k_wgrad_reduce<true>, grid1((long)cout * 9 * cinp + cout, 64), dim3(64 * kReduceWaves), 0, s, partial, pb,
                           nc, cout, cin, cinp, dw, db);
    else
        hipLaunchKernelGGL(k_wgrad_reduce<false>, grid1((long)cout * 9 * cinp + cout, 64), dim3(64 * kReduceWaves), 0, s, partial, pb,
                           nc, cout, cin, cinp, dw, db);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int n, float lr, float b1, float b2, float eps,
                       int step, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, grid1(n, 256), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace tsdf

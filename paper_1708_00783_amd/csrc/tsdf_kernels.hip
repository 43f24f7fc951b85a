// tsdf_kernels.hip -- gfx950 kernels of the voxel-hashed TSDF fusion hot path.
//
// Frame pipeline (one launch each, counts stay on the device):
//   k_alloc_rays   one lane per pixel: depth ingest, segment samples, hash probes,
//                  visible marks, de-duplicated insertion requests; workgroups
//                  past the image re-test the previous visible list   (Sec. 4.2, parts 1, 3)
//   k_insert       one lane per request: free-stack pops, bucket claim or excess
//                  chain link, block init                              (Sec. 4.2, part 2)
//   k_visible      16 entries per lane: scan compaction of the marks   (Sec. 4.2, part 3)
//   k_integrate    one wave per visible block, 8 voxels per lane; for the
//                  allocation view also the block's search-range record and
//                  its 16x16-pixel tile bins                           (Sec. 4.3, 4.4)
//   k_range_bin    one lane per block: projected box -> tile bins, for any
//                  other view                                          (Sec. 4.4)
//   k_raycast      one workgroup per 16x16 tile: per-pixel search range from the
//                  tile's bin, then the ray state machine                (Sec. 4.4)
//
// Compiled with -ffp-contract=off and correctly rounded fp32 division and
// square root: every float expression below is evaluated as written, one IEEE
// operation at a time.
#include <type_traits>

#include "tsdf_device.h"

namespace tsdf {

// ============================================================================
// initialisation
// ============================================================================
__global__ __launch_bounds__(256) void k_init(Vol v, uint32_t max_tiles)
{
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = gid; i < v.n_entries; i += stride) {
        int4 e;
        e.x = 0;
        e.y = 0;
        e.z = 0;
        e.w = kPtrEmpty;
        *reinterpret_cast<int4 *>(v.entries + i) = e;
    }
    const size_t nvis = ((size_t)v.n_entries + 15) & ~(size_t)15;
    for (size_t i = gid; i < nvis; i += stride) v.vis[i] = 0;
    for (size_t i = gid; i < v.n_blocks; i += stride) v.free_blocks[i] = (int32_t)i;
    for (size_t i = gid; i < v.n_excess; i += stride) v.free_excess[i] = (int32_t)i;
    for (size_t i = gid; i <= v.reqset_mask; i += stride) v.reqset[i] = 0ull;
    if (v.host_has)
        for (size_t i = gid; i < nvis; i += stride) v.host_has[i] = 0;
    for (size_t i = gid; i < (size_t)kIntegrateGrid; i += stride) v.acc_cols[i] = 0ull;
    for (size_t i = gid; i < max_tiles; i += stride) {
        *bin_counter(v, (int)i) = 0;
        v.acc_hits[i] = 0ull;
    }
    for (size_t i = gid; i < (size_t)(v.n_buckets / 32u); i += stride) v.occ[i] = 0u;
    for (size_t i = gid; i < (size_t)kBrickWords; i += stride) v.brick[i] = 0u;
    if (gid == 0) {
        Ctrl c = {};
        c.free_blocks = (int32_t)v.n_blocks;
        c.free_excess = (int32_t)v.n_excess;
        *v.ctrl = c;
    }
}

// empty every tile's bin and the record list (bins abandoned unread)
__global__ __launch_bounds__(256) void k_clear_bins(Vol v, uint32_t max_tiles)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < max_tiles; i += gridDim.x * blockDim.x)
        *bin_counter(v, (int)i) = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) v.ctrl->n_rec = 0u;
}

// ============================================================================
// allocation (Sec. 4.2) and integration (Sec. 4.3), one volume per launch
// ============================================================================
template <int FMT>
__global__ __launch_bounds__(256) void k_alloc_rays(Vol v, Cam c, const void *din)
{
    alloc_rays_body<FMT>(v, c, din, true);
}

__global__ __launch_bounds__(256) void k_insert(Vol v, Cam c) { insert_body(v, c); }

__global__ __launch_bounds__(256) void k_visible(Vol v) { visible_body(v); }

__global__ __launch_bounds__(256) void k_integrate(Vol v, Cam c, int bin)
{
    __shared__ float rcp_w[260];
    __shared__ uint32_t wg_cols;
    integrate_body<256>(v, c, rcp_w, &wg_cols, false, bin != 0);
}

// ============================================================================
// depth ingest on its own (integration with a depth map other than the last
// allocation's)
// ============================================================================
template <int FMT>
__global__ __launch_bounds__(256) void k_depth_convert(float *dst, const void *src, int n)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    if (FMT == TF_DEPTH_U16_MM)
        dst[p] = (float)reinterpret_cast<const uint16_t *>(src)[p] / 1000.0f;
    else
        dst[p] = reinterpret_cast<const float *>(src)[p];
}


// ============================================================================
// search range (Sec. 4.4): project blocks, bin them by 16x16 tile
// ============================================================================
constexpr int kExpandV = 3;   // voxels added around a block when binning it

// The blocks' records (search-range box and z range of the block itself, key,
// device pointer) go to every tile their cubes cover -- grown by kExpandV
// voxels when every block is binned, so that a tile's bin then holds every
// block any trilinear read of the tile's rays can touch.
//
// Bound: latency of the tile counters' atomics and, over a sparse table, the
// read of its entries.  A workgroup lists the live entries of its strips that
// the view can see in LDS, so that the lanes are full whatever the table's
// load (3 of 64 at 5%); a listed block's records take eight lanes, one per
// corner; the records are reserved with one global atomic per round of up to
// 256 blocks (same-address atomics take 11 ns each: one per wave and 64
// entries cost more than everything else); and the (record, tile) writes are
// spread over the workgroup, four per thread in flight, as a block near the
// camera covers hundreds of tiles.  2^20 + 2^17 entries, 58 k blocks,
// 960x540: 110 us before, 30 us now.
constexpr int kBinStrips = 4;
constexpr int kBinGrid = 512;

struct BinLds {
    int4 live[256 + 256 * kBinStrips];       // {bx | by << 16, bz, ptr}
    Rec rec[256];
    uint32_t excl[257];                      // exclusive tile counts of the round's blocks, and their sum
    int16_t rect[256][3];                    // tx0, ty0, nx
    int tiles[256];                          // tiles of the block's cube (0: it misses the image)
    uint32_t n, wave_n[4], wave_t[4], base;
};

// bin the m <= 256 blocks from live[first] (every thread calls it)
__device__ __forceinline__ void bin_blocks(const Vol &v, const Cam &c, bool all, BinLds &B, uint32_t first, uint32_t m)
{
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const int ntx = (c.W + kTile - 1) / kTile;
    // the records, eight lanes to a block
    for (uint32_t b = threadIdx.x >> 3; b < m; b += 32u) {
        const int4 w = B.live[first + b];
        const int bx = (int16_t)(w.x & 0xffff), by = (int16_t)((uint32_t)w.x >> 16), bz = w.y;
        // bins of every block (foreign views) grow the cubes so that a
        // complete tile table answers every lookup of the tile's rays;
        // bins of the visible list cannot, so they use the plain cube
        Rec r = {}, ex = {};
        int tiles = 0;
        bool in = true, own = false;
#pragma unroll 1
        for (int grown = 1; grown >= 0 && in; --grown) {       // the grown cube, then the block itself
            const int g = grown && all ? kExpandV : 0;
            ex = r;
            const bool ok = cube_record_lanes(c, v.voxel, 8 * bx - g, 8 * by - g, 8 * bz - g, 8 + 2 * g, r);
            in = grown ? ok : true;
            own = ok;
        }
        if (in) {
            if (!own) {
                // only the grown cube reaches the image: a table entry with no range
                r.x0 = 1;
                r.x1 = 0;
                r.y0 = 1;
                r.y1 = 0;
                r.zlo = __builtin_inff();
                r.zhi = -__builtin_inff();
            }
            const int tx0 = ex.x0 / kTile, tx1 = ex.x1 / kTile, ty0 = ex.y0 / kTile, ty1 = ex.y1 / kTile;
            tiles = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
            if ((lane & 7u) == 0u) {
                r.bx = (int16_t)bx;
                r.by = (int16_t)by;
                r.bz = (int16_t)bz;
                r.pad = 0;
                r.ptr = w.z;
                r.pad2 = 0;
                B.rec[b] = r;
                B.rect[b][0] = (int16_t)tx0;
                B.rect[b][1] = (int16_t)ty0;
                B.rect[b][2] = (int16_t)(tx1 - tx0 + 1);
            }
        }
        if ((lane & 7u) == 0u) B.tiles[b] = tiles;
    }
    __syncthreads();
    const uint32_t cnt = threadIdx.x < m ? (uint32_t)B.tiles[threadIdx.x] : 0u;
    const bool emit = cnt != 0u;
    const unsigned long long em = __ballot(emit);
    // exclusive scan of the threads' tile counts
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d);
        if ((int)lane >= d) incl += t;
    }
    if (lane == kWave - 1) {
        B.wave_t[wv] = incl;
        B.wave_n[wv] = (uint32_t)__popcll(em);
    }
    __syncthreads();
    uint32_t before = 0, rank = rank_in(em);
    for (uint32_t k = 0; k < wv; ++k) {
        before += B.wave_t[k];
        rank += B.wave_n[k];
    }
    B.excl[threadIdx.x] = before + incl - cnt;
    uint32_t rec_base = 0u;                  // thread 255: the round's place in the record list, in flight
    if (threadIdx.x == 255) {
        B.excl[256] = before + incl;
        const uint32_t k = rank + (emit ? 1u : 0u);
        if (k) rec_base = atomicAdd(&v.ctrl->n_rec, k);
    }
    __syncthreads();
    // (record, tile) items over all threads, four per thread in flight
    const uint32_t total = B.excl[256];
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 1024u) {
        int own[4], tl[4], sl[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t item = i0 + 256u * (uint32_t)q;
            // owner: the last j with excl[j] <= item (blocks without tiles have empty ranges)
            int j = 0;
#pragma unroll
            for (int b = 128; b; b >>= 1)
                if (B.excl[j + b] <= item) j += b;
            const uint32_t li = item - B.excl[j];
            const int nx = item < total ? B.rect[j][2] : 1;
            own[q] = item < total ? j : -1;
            tl[q] = (B.rect[j][1] + (int)(li / (uint32_t)nx)) * ntx + B.rect[j][0] + (int)(li % (uint32_t)nx);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) sl[q] = own[q] >= 0 ? atomicAdd(bin_counter(v, tl[q]), 1) : kBinCap;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (sl[q] < kBinCap) *bin_record(v, tl[q], sl[q]) = B.rec[own[q]];
    }
    if (threadIdx.x == 255) B.base = rec_base;
    __syncthreads();
    if (emit) v.recs[B.base + rank] = B.rec[threadIdx.x];
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_range_bin(Vol v, Cam c, int all)
{
    __shared__ BinLds B;
    const uint32_t n = all ? v.n_entries : v.ctrl->n_vis;
    const uint32_t strips = (n + 255u) / 256u;
    const Frustum fr = make_frustum(c, v.voxel, kExpandV);
    if (threadIdx.x == 0) B.n = 0u;
    __syncthreads();
    // strips a grid apart: the used slots of the excess list are all at its
    // end, and a workgroup that took them alone finished 40 us after the rest
    for (uint32_t s = blockIdx.x; s < strips; s += kBinStrips * gridDim.x) {
        int4 w[kBinStrips];
#pragma unroll
        for (int k = 0; k < kBinStrips; ++k) {
            const uint32_t i = (s + (uint32_t)k * gridDim.x) * 256u + threadIdx.x;
            w[k] = make_int4(0, 0, 0, -2);
            if (i < n) w[k] = load_entry(v.entries, all ? i : (uint32_t)v.vlist[i]);
        }
#pragma unroll
        for (int k = 0; k < kBinStrips; ++k) {
            const int bx = (int16_t)(w[k].x & 0xffff), by = (int16_t)((uint32_t)w[k].x >> 16),
                      bz = (int16_t)(w[k].y & 0xffff);
            const bool in = w[k].w >= 0 && !outside_frustum(fr, c.M, c, v.voxel, bx, by, bz);
            const unsigned long long m = __ballot(in);
            if (!m) continue;
            const int leader = __ffsll((long long)m) - 1;
            uint32_t at = 0;
            if ((int)lane_id() == leader) at = atomicAdd(&B.n, (uint32_t)__popcll(m));
            at = __shfl(at, leader);
            if (in) B.live[at + rank_in(m)] = make_int4(w[k].x, bz, w[k].w, 0);
        }
        __syncthreads();
        // whole rounds of 256 from the end of the list; the rest waits for
        // the next strips, or goes last
        uint32_t have = B.n;
        while (have >= 256u || (have && s + kBinStrips * gridDim.x >= strips)) {
            const uint32_t m = have < 256u ? have : 256u;
            have -= m;
            bin_blocks(v, c, all != 0, B, have, m);
        }
        if (threadIdx.x == 0) B.n = have;
        __syncthreads();
    }
}

// LDS of a raycast tile: the (block key -> record of the tile's bin) table,
// and, first, the records' pixel boxes and z ranges (their first 16 bytes)
// with each wave's list of those that matter to it, for the per-pixel range;
// then, in the same bytes, the device pointers of every record's block and of
// its neighbours, n = 1..7 at (n & 1, n >> 1 & 1, n >> 2), -1 where absent.
struct TileTable {
    unsigned long long key[kTileTable];   // 0 = empty slot
    union {
        struct {
            uint4 box[kBinCap];            // x0, y0, x1, y1 (int16), zlo, zhi (float)
            uint16_t wlist[4][kBinCap];    // per wave: the staged records whose box meets its pixels
        } r;
        int nb[kBinCap][8];
    };
    uint16_t rec[kTileTable];             // record of the slot's block
    int wcnt[4];
    int complete;                         // the table holds the whole bin
};

// slot hash of the tile's private table: products of the 16-bit coordinates
// (callers have range-checked them) with 23-bit constants, which compile to
// full-rate 24-bit multiplies, folded to the table size
__device__ __forceinline__ uint32_t table_slot(int bx, int by, int bz)
{
    const int x = (int16_t)bx, y = (int16_t)by, z = (int16_t)bz;
    const uint32_t h = (uint32_t)(x * 0x1f1f1f) ^ (uint32_t)(y * 0x3c6ef3) ^ (uint32_t)(z * 0x5a8279);
    return (h ^ (h >> 10)) & (uint32_t)(kTileTable - 1);
}

// the record of a block (coordinates in the 16-bit range) in the tile's table, or -1
__device__ __forceinline__ int table_find(const TileTable *tt, int bx, int by, int bz)
{
    const unsigned long long key = pack_key(bx, by, bz);
    uint32_t sl = table_slot(bx, by, bz);
    for (int k = 0; k < kTileTable; ++k) {
        const unsigned long long kk = tt->key[sl];
        if (kk == key) return (int)tt->rec[sl];
        if (kk == 0ull) break;
        sl = (sl + 1u) & (uint32_t)(kTileTable - 1);
    }
    return -1;
}

// device pointer of a block (coordinates in the 16-bit range; -1 = absent or
// not on the device) from its occupancy brick and its bucket entry, loaded
// together; the chain beyond the bucket only when the entry is another block's
struct MapProbe {
    uint32_t bw;
    int4 w;
};

__device__ __forceinline__ MapProbe map_probe(const Vol &v, int bx, int by, int bz)
{
    MapProbe m;
    m.bw = gload(v.brick + brick_word(bx, by, bz));
    m.w = load_entry(v.entries, hash_index(bx, by, bz, v.n_buckets - 1u));
    return m;
}

__device__ __forceinline__ int map_resolve(const Vol &v, const MapProbe &m, int bx, int by, int bz)
{
    const int4 w = m.w;
    if (!(m.bw & brick_bit(bx, by, bz))) return -1;
    const uint32_t kxy = (uint32_t)(uint16_t)bx | ((uint32_t)(uint16_t)by << 16);
    if ((uint32_t)w.x == kxy && (int16_t)(w.y & 0xffff) == (int16_t)bz && w.w >= 0) return w.w;
    if (w.z < 1 || (uint32_t)(w.z - 1) >= v.n_excess) return -1;
    int ptr = -1;
    const int e = find_entry_from(v.entries, v.n_buckets, v.n_excess, v.n_buckets + (uint32_t)(w.z - 1), bx, by, bz, 0,
                                  &ptr);
    return e >= 0 ? ptr : -1;
}

__device__ __forceinline__ int map_find(const Vol &v, int bx, int by, int bz)
{
    return map_resolve(v, map_probe(v, bx, by, bz), bx, by, bz);
}

// The tile's block table and the search range of pixel (px, py) from the
// tile's bin (all records, in chunks of kBinCap and without a table, if the
// bin overflowed).  The records are staged in LDS, each also listed for the
// waves whose pixels its box meets (wave w's pixels: the 8 x 8 quadrant w of
// the tile when `quads`, else rows 4 w .. 4 w + 3); every thread then takes
// the min / max over its wave's list whose box holds its pixel: the
// per-pixel loop itself, with no atomics, over the records that can matter.
// Every thread of the workgroup calls it; zmin = +inf and zmax = -inf when
// no record covers the pixel.
__device__ __forceinline__ void tile_range(const Vol &v, int tile, int tx0, int ty0, bool quads, int px, int py,
                                           TileTable *tt, bool table, float &zmin, float &zmax)
{
    for (int k = threadIdx.x; k < kTileTable; k += 256) tt->key[k] = 0ull;
    if (threadIdx.x < 4) tt->wcnt[threadIdx.x] = 0;
    const int wave = (int)threadIdx.x >> 6;
    const int cnt = *bin_counter(v, tile);
    const bool fallback = cnt > kBinCap;
    const int n = fallback ? (int)v.ctrl->n_rec : cnt;
    if (threadIdx.x == 0) tt->complete = table && !fallback;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    int4 own[2];           // {bx | by << 16, bz, ptr} of this thread's records of a table's bin
    for (int base = 0; base < n; base += kBinCap) {
        const int m = n - base < kBinCap ? n - base : kBinCap;
        __syncthreads();   // the cleared table, or the previous chunk consumed
#pragma unroll
        for (int h = 0; h < kBinCap / 256; ++h) {
            const int j = (int)threadIdx.x + 256 * h;
            if (j >= m) break;
            const Rec r = fallback ? v.recs[base + j] : *bin_record(v, tile, j);
            if (table && !fallback) {
                // keys in one bin are distinct; the table is at most half full
                const unsigned long long key = pack_key(r.bx, r.by, r.bz);
                uint32_t sl = table_slot(r.bx, r.by, r.bz);
                for (int k = 0; k < kTileTable; ++k) {
                    if (atomicCAS(&tt->key[sl], 0ull, key) == 0ull) {
                        tt->rec[sl] = (uint16_t)j;
                        break;
                    }
                    sl = (sl + 1u) & (uint32_t)(kTileTable - 1);
                }
                own[h] = make_int4((int)((uint32_t)(uint16_t)r.bx | ((uint32_t)(uint16_t)r.by << 16)), r.bz, r.ptr, 0);
            }
            tt->r.box[j] = make_uint4((uint32_t)(uint16_t)r.x0 | ((uint32_t)(uint16_t)r.y0 << 16),
                                    (uint32_t)(uint16_t)r.x1 | ((uint32_t)(uint16_t)r.y1 << 16),
                                    __float_as_uint(r.zlo), __float_as_uint(r.zhi));
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int wx0 = tx0 + (quads ? (w & 1) * 8 : 0), wy0 = ty0 + (quads ? (w >> 1) * 8 : 4 * w);
                const int wx1 = wx0 + (quads ? 7 : 15), wy1 = wy0 + (quads ? 7 : 3);
                if (r.x0 <= wx1 && r.x1 >= wx0 && r.y0 <= wy1 && r.y1 >= wy0)
                    tt->r.wlist[w][atomicAdd(&tt->wcnt[w], 1)] = (uint16_t)j;
            }
        }
        __syncthreads();
        // the order of a wave's list varies with the atomics; min and max do not
        const int nw = __builtin_amdgcn_readfirstlane(tt->wcnt[wave]);
        // kBatch boxes at a time, their LDS reads (list, then box) in flight
        // together; past the end the last one again, which changes nothing
        constexpr int kBatch = 4;
        for (int i = 0; i < nw; i += kBatch) {
            uint4 bb[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) bb[k] = tt->r.box[tt->r.wlist[wave][i + k < nw ? i + k : nw - 1]];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const uint4 b = bb[k];
                const int x0 = (int16_t)(b.x & 0xffffu), y0 = (int16_t)(b.x >> 16);
                const int x1 = (int16_t)(b.y & 0xffffu), y1 = (int16_t)(b.y >> 16);
                if (px >= x0 && px <= x1 && py >= y0 && py <= y1) {
                    const float zl = __uint_as_float(b.z), zh = __uint_as_float(b.w);
                    lo = zl < lo ? zl : lo;
                    hi = zh > hi ? zh : hi;
                }
            }
        }
        // this wave's list is consumed; the next chunk's staging starts after the barrier above
        if ((threadIdx.x & 63) == 0) tt->wcnt[wave] = 0;
    }
    __syncthreads();   // the table is complete before any lookup, the boxes are read
    zmin = lo;
    zmax = hi;
    if (!table || fallback) return;
    // The neighbours of every block of the bin, eight lanes to a record: a ray
    // that crosses a block face then reads them with its own block instead of
    // looking up to seven blocks up one after another (the march's longest
    // chain: 25 to 32% of the kernel).
#pragma unroll
    for (int h = 0; h < kBinCap / 256; ++h) {
        const int j = (int)threadIdx.x + 256 * h;
        if (j >= n) break;
        tt->nb[j][0] = own[h].z;
        tt->nb[j][1] = own[h].x;
        tt->nb[j][2] = own[h].y;
    }
    __syncthreads();
    // A thread takes kLook of them at a time: the table first, then the map
    // reads of all that are not in it, together.
    constexpr int kLook = 2;
    const int nn = (int)threadIdx.x & 7;
    for (int i0 = (int)threadIdx.x; i0 < 8 * n; i0 += kLook * 256) {
        int kxy[kLook], bz[kLook], p[kLook];
        bool ask[kLook];
        MapProbe m[kLook];
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const int i = i0 + 256 * u, j = (i < 8 * n ? i : i0) >> 3;
            kxy[u] = tt->nb[j][1];
            bz[u] = tt->nb[j][2] + (nn >> 2);
        }
        __builtin_amdgcn_wave_barrier();   // the records' eight lanes have read their keys
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const int bx = (int16_t)(kxy[u] & 0xffff) + (nn & 1), by = (int16_t)((uint32_t)kxy[u] >> 16) + ((nn >> 1) & 1);
            p[u] = -1;
            ask[u] = false;
            if (nn != 0 && i0 + 256 * u < 8 * n && in_short_range(bx) && in_short_range(by) && in_short_range(bz[u])) {
                const int k = table_find(tt, bx, by, bz[u]);
                ask[u] = k < 0;
                if (k >= 0) p[u] = tt->nb[k][0];
            }
            if (ask[u]) m[u] = map_probe(v, bx, by, bz[u]);
        }
#pragma unroll
        for (int u = 0; u < kLook; ++u) {
            const int bx = (int16_t)(kxy[u] & 0xffff) + (nn & 1), by = (int16_t)((uint32_t)kxy[u] >> 16) + ((nn >> 1) & 1);
            if (ask[u]) p[u] = map_resolve(v, m[u], bx, by, bz[u]);
            if (nn != 0 && i0 + 256 * u < 8 * n) tt->nb[(i0 + 256 * u) >> 3][nn] = p[u];
        }
    }
    __syncthreads();   // before any lookup
}

// End of a raycast-kind workgroup (every thread calls it, after its last
// read of the tile's bin): clear the tile's bin counter; the last workgroup
// of the launch clears the record counter.  Taken at the end of the kernel,
// the tickets of the workgroups arrive spread out in time.  No fence: every
// workgroup has read the counter before its ticket, and the next launch sees
// the stores.
__device__ __forceinline__ void finish_tile(const Vol &v, int tile, bool count_raycast)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        if (tile >= 0) *bin_counter(v, tile) = 0;
        const uint32_t t = atomicAdd(&v.ctrl->ray_ticket, 1u);
        if (t == gridDim.x - 1u) {
            if (count_raycast) v.ctrl->tot_rec += v.ctrl->n_rec;
            v.ctrl->n_rec = 0u;
            v.ctrl->ray_ticket = 0u;
        }
    }
}

// ============================================================================
// raycast (Sec. 4.4)
// ============================================================================
namespace {


// one-entry block cache (the paper's IndexCache, Sec. 3.3): the last block
// key looked up, its device pointer (-1 = absent or not on the device) and
// its record in the tile's table (-1 = not there); `local`: lookups of this
// ray may trust a miss in the tile's table
struct BlockCache {
    int bx, by, bz, ptr, rec;
    bool local;
};

// device pointer of a block (-1 = absent or not on the device): the tile's
// LDS table first; unless `local`, then the occupancy bricks and the hash table.
// `local` holds for a ray whose points all lie at or beyond the near plane in
// a tile whose table holds its whole bin: every block within kExpandV voxels
// of such a point is in the bin, so a miss proves absence.
__device__ __forceinline__ int lookup_block(const Vol &v, const TileTable *tt, int bx, int by, int bz, bool local)
{
    if (!in_short_range(bx) || !in_short_range(by) || !in_short_range(bz)) return -1;
    const int k = table_find(tt, bx, by, bz);
    if (k >= 0) return tt->nb[k][0];
    return local ? -1 : map_find(v, bx, by, bz);
}

__device__ __forceinline__ int cached_block(const Vol &v, const TileTable *tt, int bx, int by, int bz,
                                            BlockCache &cc)
{
    if (bx == cc.bx && by == cc.by && bz == cc.bz) return cc.ptr;
    cc.bx = bx;
    cc.by = by;
    cc.bz = bz;
    cc.rec = -1;
    cc.ptr = -1;
    if (in_short_range(bx) && in_short_range(by) && in_short_range(bz)) {
        cc.rec = table_find(tt, bx, by, bz);
        if (cc.rec >= 0)
            cc.ptr = tt->nb[cc.rec][0];
        else if (!cc.local)
            cc.ptr = map_find(v, bx, by, bz);
    }
    return cc.ptr;
}

// A trilinear cell ready to load.  Corners c and c + 4 are one voxel apart
// along z, next to each other in memory unless the cell crosses its block's
// upper z face: o[c] are the byte offsets of the four lower corners into the
// voxel array (32-bit when the array spans at most 4 GiB), each read as one
// 4-byte pair; oz[c] those of the upper corners, read only when `sz`.
// `present`: which corners have a block (an absent corner addresses block 0;
// its value is not used).
template <bool kOff32>
struct RayCell {
    using Off = typename std::conditional<kOff32, uint32_t, size_t>::type;
    Off o[4], oz[4];
    uint32_t present;
    bool sz;
    float tx, ty, tz;
};

// byte offset of voxel j of block p into the voxel array
template <bool kOff32>
__device__ __forceinline__ typename RayCell<kOff32>::Off voxel_offset(int p, int j)
{
    const uint32_t pc = p >= 0 ? (uint32_t)p : 0u;
    if (kOff32) return __umul24(pc, (uint32_t)kBlockBytes) + 2u * (uint32_t)j;
    return (typename RayCell<kOff32>::Off)((size_t)pc * kBlockBytes + 2u * (uint32_t)j);
}

// corner blocks: the cell's own block through the ray's cache; where the cell
// crosses a block face (local index 7), the neighbouring blocks from the
// record of the own block, or, for a block outside the tile's table, looked up
template <bool kOff32>
__device__ __forceinline__ void cell_setup(const Vol &v, const TileTable *tt, float X, float Y, float Z,
                                           BlockCache &cc, RayCell<kOff32> &C)
{
    const float bx = floorf(X), by = floorf(Y), bz = floorf(Z);
    C.tx = X - bx;
    C.ty = Y - by;
    C.tz = Z - bz;
    const int ix = (int)bx, iy = (int)by, iz = (int)bz;
    const int Bx = ix >> 3, By = iy >> 3, Bz = iz >> 3;
    const bool sx = (ix & 7) == 7, sy = (iy & 7) == 7, sz = (iz & 7) == 7;
    const int p0 = cached_block(v, tt, Bx, By, Bz, cc);
    int n1 = p0, n2 = p0, n3 = p0, n4 = p0, n5 = p0, n6 = p0, n7 = p0;
    if (sx | sy | sz) {
        if (cc.rec >= 0) {
            const int4 a = *reinterpret_cast<const int4 *>(&tt->nb[cc.rec][0]);
            const int4 b = *reinterpret_cast<const int4 *>(&tt->nb[cc.rec][4]);
            n1 = a.y;
            n2 = a.z;
            n3 = a.w;
            n4 = b.x;
            n5 = b.y;
            n6 = b.z;
            n7 = b.w;
        } else {
            const int need = (sx ? 1 : 0) | (sy ? 2 : 0) | (sz ? 4 : 0);
#pragma unroll 1
            for (int n = 1; n < 8; ++n) {
                if ((n & need) != n) continue;
                const int p = lookup_block(v, tt, Bx + (n & 1), By + ((n >> 1) & 1), Bz + (n >> 2), cc.local);
                n1 = n == 1 ? p : n1;
                n2 = n == 2 ? p : n2;
                n3 = n == 3 ? p : n3;
                n4 = n == 4 ? p : n4;
                n5 = n == 5 ? p : n5;
                n6 = n == 6 ? p : n6;
                n7 = n == 7 ? p : n7;
            }
        }
    }
    const int p[4] = {p0, sx ? n1 : p0, sy ? n2 : p0, sx ? (sy ? n3 : n1) : (sy ? n2 : p0)};
    // in-block indices of the lower corners; a step across a face wraps to index 0
    int j[4];
    j[0] = (iz & 7) + 8 * (iy & 7) + 64 * (ix & 7);
    const int dx = sx ? -448 : 64, dy = sy ? -56 : 8;
    j[1] = j[0] + dx;
    j[2] = j[0] + dy;
    j[3] = j[1] + dy;
    uint32_t present = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        present |= (p[c] >= 0 ? 0x11u : 0u) << c;
        C.o[c] = voxel_offset<kOff32>(p[c], j[c]);
    }
    C.sz = sz;
    if (sz) {
        const int u[4] = {n4, sx ? n5 : n4, sy ? n6 : n4, sx ? (sy ? n7 : n5) : (sy ? n6 : n4)};
        present &= 0xfu;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            present |= (u[c] >= 0 ? 0x10u : 0u) << c;
            C.oz[c] = voxel_offset<kOff32>(u[c], j[c] - 7);
        }
    }
    C.present = present;
}

// The reads are bound by the vector memory unit's rate over the lanes' lines:
// four 4-byte pairs (any 2-byte alignment; voxel 7's pair reads two bytes past
// its column, still within its block) instead of eight 2-byte reads.
template <bool kOff32>
__device__ __forceinline__ void cell_load(const Vol &v, const RayCell<kOff32> &C, int16_t (&s)[8])
{
    uint32_t d[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) d[c] = gload_pair(v.voxels + C.o[c]);
    uint32_t u[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) u[c] = d[c] >> 16;
    if (C.sz) {
#pragma unroll
        for (int c = 0; c < 4; ++c) u[c] = gload(reinterpret_cast<const uint16_t *>(v.voxels + C.oz[c]));
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        s[c] = (int16_t)(d[c] & 0xffffu);
        s[c + 4] = (int16_t)u[c];
    }
}

// trilinear interpolation of F at voxel-unit P (Sec. 4.4)
template <bool kOff32>
__device__ __forceinline__ float trilinear(const Vol &v, const TileTable *tt, float X, float Y, float Z,
                                           BlockCache &cc)
{
    RayCell<kOff32> C;
    int16_t s[8];
    cell_setup(v, tt, X, Y, Z, cc, C);
    cell_load(v, C, s);
    return cell_lerp(C.present, s, C.tx, C.ty, C.tz);
}

// F(A) - F(B) with the sixteen voxel loads of both cells issued together
template <bool kOff32>
__device__ __forceinline__ float trilinear_diff(const Vol &v, const TileTable *tt, float AX, float AY, float AZ,
                                                float BX, float BY, float BZ, BlockCache &cc)
{
    RayCell<kOff32> A, B;
    int16_t sa[8], sb[8];
    cell_setup(v, tt, AX, AY, AZ, cc, A);
    cell_setup(v, tt, BX, BY, BZ, cc, B);
    cell_load(v, A, sa);
    cell_load(v, B, sb);
    return cell_lerp(A.present, sa, A.tx, A.ty, A.tz) - cell_lerp(B.present, sb, B.tx, B.ty, B.tz);
}

// The normal's central differences (Sec. 4.4): g_a = (F(P + e_a) -
// F(P - e_a)) / 2 for the three axes.  The six trilinear cells are those of
// floor(P) -+ e_a; together they read 32 distinct voxels of the 4 x 4 x 4
// around floor(P), which spans at most two blocks per axis, so the block
// pointers are looked up once.  The voxels lie in 12 z columns: four of
// z - 1 .. z + 2 (dx, dy 0..1), read as 8 bytes each, and eight of z .. z + 1
// (dx or dy -1 or 2), read as 4 bytes; where the columns cross the block's z
// face, the rest comes from the block across it.  All loads are issued
// together; 32 single reads cost the vector memory unit twice the lookups.
// Each cell keeps the fractions of its own point P -+ e_a, as separate
// trilinear reads would.  Returns false (nothing computed) when rounding of
// P -+ 1 moves a cell off floor(P) -+ e_a.
template <bool kOff32>
__device__ __forceinline__ bool normal_gradient(const Vol &v, const TileTable *tt, float X, float Y, float Z,
                                                BlockCache &cc, float &gx, float &gy, float &gz)
{
    const float Xp = X + 1.0f, Xm = X - 1.0f, Yp = Y + 1.0f, Ym = Y - 1.0f, Zp = Z + 1.0f, Zm = Z - 1.0f;
    const float fX = floorf(X), fY = floorf(Y), fZ = floorf(Z);
    const float fXp = floorf(Xp), fXm = floorf(Xm), fYp = floorf(Yp), fYm = floorf(Ym), fZp = floorf(Zp),
                fZm = floorf(Zm);
    if (fXp != fX + 1.0f || fXm != fX - 1.0f || fYp != fY + 1.0f || fYm != fY - 1.0f || fZp != fZ + 1.0f ||
        fZm != fZ - 1.0f)
        return false;
    const int ix = (int)fX, iy = (int)fY, iz = (int)fZ;
    const int Bx = ix >> 3, By = iy >> 3, Bz = iz >> 3;
    // the second block the range i - 1 .. i + 2 reaches on each axis (0: none)
    const int ax = (ix & 7) == 0 ? -1 : ((ix & 7) >= 6 ? 1 : 0);
    const int ay = (iy & 7) == 0 ? -1 : ((iy & 7) >= 6 ? 1 : 0);
    const int az = (iz & 7) == 0 ? -1 : ((iz & 7) >= 6 ? 1 : 0);
    int pb[8];
    pb[0] = cached_block(v, tt, Bx, By, Bz, cc);
    // the lowest block of the range: its record's row holds all of them (seven
    // lookups one after the other were 5 to 8% of the kernel)
    const int lx = ax < 0 ? 1 : 0, ly = ay < 0 ? 1 : 0, lz0 = az < 0 ? 1 : 0;
    int rec = cc.rec;
    if (lx | ly | lz0)
        rec = (in_short_range(Bx - lx) && in_short_range(By - ly) && in_short_range(Bz - lz0))
                  ? table_find(tt, Bx - lx, By - ly, Bz - lz0)
                  : -1;
    if (rec >= 0) {
        // a step along an axis leads from the own block (lx, ly, lz0) to the other of the two
#pragma unroll
        for (int c = 1; c < 8; ++c) {
            const int o = (((c & 1) ^ lx) | ((((c >> 1) & 1) ^ ly) << 1) | (((c >> 2) ^ lz0) << 2));
            pb[c] = tt->nb[rec][o];
        }
    } else {
        int q1 = -1, q2 = -1, q3 = -1, q4 = -1, q5 = -1, q6 = -1, q7 = -1;
#pragma unroll 1
        for (int c = 1; c < 8; ++c) {
            const int sx = c & 1, sy = (c >> 1) & 1, sz = c >> 2;
            if ((sx && !ax) || (sy && !ay) || (sz && !az)) continue;
            const int q = lookup_block(v, tt, Bx + (sx ? ax : 0), By + (sy ? ay : 0), Bz + (sz ? az : 0), cc.local);
            q1 = c == 1 ? q : q1;
            q2 = c == 2 ? q : q2;
            q3 = c == 3 ? q : q3;
            q4 = c == 4 ? q : q4;
            q5 = c == 5 ? q : q5;
            q6 = c == 6 ? q : q6;
            q7 = c == 7 ? q : q7;
        }
        pb[1] = q1;
        pb[2] = q2;
        pb[3] = q3;
        pb[4] = q4;
        pb[5] = q5;
        pb[6] = q6;
        pb[7] = q7;
    }
    // columns 0..3: (dx, dy) = (c & 1, c >> 1), z - 1 .. z + 2; 4..7: dx -1 / 2
    // (c & 1), dy 0 / 1 (c >> 1 & 1), and 8..11: dx 0 / 1, dy -1 / 2, z .. z + 1
    constexpr int kCols = 12;
    const int lz = iz & 7;
    const int q0 = lz < 1 ? 0 : (lz > 5 ? 4 : lz - 1);     // first voxel of the own block's 8 bytes
    unsigned long long quad[4];
    uint32_t pair[8], over[4], up[8];
    uint32_t lo = 0u, hi = 0u;                             // columns whose own / other z block is present
    typename RayCell<kOff32>::Off oo[kCols];               // the other z block's reads
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
        const int k = c & 3;
        const int dx = c < 4 || c >= 8 ? k & 1 : ((k & 1) ? 2 : -1);
        const int dy = c < 8 ? k >> 1 : ((k >> 1) ? 2 : -1);
        const int x = ix + dx, y = iy + dy;
        // selects, not an indexed private array (which would live in scratch)
        const bool bx = (x >> 3) != Bx, by = (y >> 3) != By;
        const int pl = by ? (bx ? pb[3] : pb[2]) : (bx ? pb[1] : pb[0]);
        const int ph = by ? (bx ? pb[7] : pb[6]) : (bx ? pb[5] : pb[4]);
        lo |= (pl >= 0 ? 1u : 0u) << c;
        hi |= (ph >= 0 ? 1u : 0u) << c;
        const int j = 8 * (y & 7) + 64 * (x & 7);
        if (c < 4)
            quad[c] = gload_quad(v.voxels + voxel_offset<kOff32>(pl, j + q0));
        else
            pair[c - 4] = gload_pair(v.voxels + voxel_offset<kOff32>(pl, j + lz));
        oo[c] = voxel_offset<kOff32>(ph, j + (c < 4 && lz == 0 ? 6 : 0));
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) over[c] = 0u;
#pragma unroll
    for (int c = 0; c < 8; ++c) up[c] = pair[c] >> 16;
    if (az != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) over[c] = gload_pair(v.voxels + oo[c]);
        if (lz == 7) {
#pragma unroll
            for (int c = 0; c < 8; ++c) up[c] = gload(reinterpret_cast<const uint16_t *>(v.voxels + oo[c + 4]));
        }
    }
    // F of the columns' voxels (an absent voxel reads 1.0): fq[c][k] at z - 1 + k, fp[c][k] at z + k
    const auto value = [](uint32_t s, bool there) {
        return there ? (float)(int16_t)(s & 0xffffu) * (1.0f / 32767.0f) : 1.0f;
    };
    float fq[4][4], fp[8][2];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const bool pl = (lo >> c) & 1u, ph = (hi >> c) & 1u;
        // 16-bit positions 0..3 hold z - 1 .. z + 2: the own block's voxels
        // shifted into place, the other block's in the freed ones
        const unsigned long long own = quad[c], oth = over[c];
        const unsigned long long w = lz == 0   ? (own << 16) | (oth >> 16)
                                     : lz == 7 ? (own >> 32) | (oth << 32)
                                     : lz == 6 ? (own >> 16) | (oth << 48)
                                               : own;
        fq[c][0] = value((uint32_t)w, lz == 0 ? ph : pl);
        fq[c][1] = value((uint32_t)(w >> 16), pl);
        fq[c][2] = value((uint32_t)(w >> 32), lz == 7 ? ph : pl);
        fq[c][3] = value((uint32_t)(w >> 48), lz >= 6 ? ph : pl);
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const bool pl = (lo >> (c + 4)) & 1u, ph = (hi >> (c + 4)) & 1u;
        fp[c][0] = value(pair[c], pl);
        fp[c][1] = value(up[c], lz == 7 ? ph : pl);
    }
    const float tx = X - fX, ty = Y - fY, tz = Z - fZ;
    // cells by their four columns (x, y), (x + 1, y), (x, y + 1), (x + 1, y + 1)
    const float xp[8] = {fq[1][1], fp[1][0], fq[3][1], fp[3][0], fq[1][2], fp[1][1], fq[3][2], fp[3][1]};
    const float xm[8] = {fp[0][0], fq[0][1], fp[2][0], fq[2][1], fp[0][1], fq[0][2], fp[2][1], fq[2][2]};
    gx = (lerp8(xp, Xp - fXp, ty, tz) - lerp8(xm, Xm - fXm, ty, tz)) * 0.5f;
    const float yp[8] = {fq[2][1], fq[3][1], fp[6][0], fp[7][0], fq[2][2], fq[3][2], fp[6][1], fp[7][1]};
    const float ym[8] = {fp[4][0], fp[5][0], fq[0][1], fq[1][1], fp[4][1], fp[5][1], fq[0][2], fq[1][2]};
    gy = (lerp8(yp, tx, Yp - fYp, tz) - lerp8(ym, tx, Ym - fYm, tz)) * 0.5f;
    const float zp[8] = {fq[0][2], fq[1][2], fq[2][2], fq[3][2], fq[0][3], fq[1][3], fq[2][3], fq[3][3]};
    const float zm[8] = {fq[0][0], fq[1][0], fq[2][0], fq[3][0], fq[0][1], fq[1][1], fq[2][1], fq[3][1]};
    gz = (lerp8(zp, tx, ty, Zp - fZp) - lerp8(zm, tx, ty, Zm - fZm)) * 0.5f;
    return true;
}

// "allocated" test of the march: the block of floor(P) has a device block
__device__ __forceinline__ bool allocated_at(const Vol &v, const TileTable *tt, float P0, float P1, float P2,
                                             BlockCache &cc)
{
    return cached_block(v, tt, block_of(P0), block_of(P1), block_of(P2), cc) >= 0;
}

enum { SEARCH_BLOCK_COARSE, SEARCH_BLOCK_FINE, SEARCH_SURFACE, BEHIND_SURFACE, WRONG_SIDE };

}  // namespace

// search range on its own, written as an image (tf_range_image)
__global__ __launch_bounds__(256) void k_range_write(Vol v, Cam c, float *zmin_out, float *zmax_out)
{
    __shared__ TileTable tbl;
    const int ntx = (c.W + kTile - 1) / kTile;
    const int tile = blockIdx.x;
    const int tx0 = (tile % ntx) * kTile, ty0 = (tile / ntx) * kTile;
    const int px = tx0 + (int)(threadIdx.x % kTile);
    const int py = ty0 + (int)(threadIdx.x / kTile);
    float zmin, zmax;
    tile_range(v, tile, tx0, ty0, false, px, py, &tbl, false, zmin, zmax);
    finish_tile(v, tile, false);
    if (px >= c.W || py >= c.H) return;
    zmin_out[(size_t)py * c.W + px] = zmin;
    zmax_out[(size_t)py * c.W + px] = zmax;
}

// ============================================================================
// raycast, one workgroup per 16x16 tile (Sec. 4.4): the tile's search range
// from its bin (LDS), the state machine per pixel, then the two refinement
// steps and the normal for the hits of the wave together
// ============================================================================
// 6 waves per SIMD (80 VGPRs): the larger images have more tiles than one
// round of workgroups holds (1280x720: 130.6 us against 135.8 at 5 waves and
// 90 VGPRs; 640x480, whose 1200 tiles are all resident either way: 77.9
// against 76.4)
template <bool kOff32>
__global__ __launch_bounds__(256, 6) void k_raycast(Vol v, Cam c, int all_blocks, float4 *pts, float4 *nrm)
{
    __shared__ TileTable tbl;
    const int ntx = (c.W + kTile - 1) / kTile, nty = (c.H + kTile - 1) / kTile;
    const int ntiles = ntx * nty;
    // workgroups go round-robin to the 8 XCDs; tiles in launch order, so that
    // the slow tiles of a region (long rays) spread over all XCDs (a band of
    // the image per XCD, for L2 locality, measured 2% slower)
    const int tile = (int)blockIdx.x;
    const bool real = tile < ntiles;
    const int q = (int)threadIdx.x >> 6, i = (int)threadIdx.x & 63;
    const int lx = (q & 1) * 8 + (i & 7), ly = (q >> 1) * 8 + (i >> 3);
    const int tx0 = real ? (tile % ntx) * kTile : 0, ty0 = real ? (tile / ntx) * kTile : 0;
    const int px = tx0 + lx, py = ty0 + ly;
    float zmin = __builtin_inff(), zmax = -__builtin_inff();
    if (real) tile_range(v, tile, tx0, ty0, true, px, py, &tbl, true, zmin, zmax);
    const bool inside = real && px < c.W && py < c.H;
    float4 out_p = make_float4(0.f, 0.f, 0.f, 0.f), out_n = make_float4(0.f, 0.f, 0.f, 0.f);
    if (inside && zmin <= zmax) {
        const float vs = v.voxel;
        const float inv_vs = 1.0f / vs;
        const float mu_v = v.mu * inv_vs;
        const float ox = c.ti[0] * inv_vs, oy = c.ti[1] * inv_vs, oz = c.ti[2] * inv_vs;
        const float a = ((float)px - c.cx) / c.fx;
        const float b = ((float)py - c.cy) / c.fy;
        const float nr = sqrtf((a * a + b * b) + 1.0f);
        const float rcx = a / nr, rcy = b / nr, rcz = 1.0f / nr;
        const float dx = (c.Ri[0] * rcx + c.Ri[1] * rcy) + c.Ri[2] * rcz;
        const float dy = (c.Ri[3] * rcx + c.Ri[4] * rcy) + c.Ri[5] * rcz;
        const float dz = (c.Ri[6] * rcx + c.Ri[7] * rcy) + c.Ri[8] * rcz;
        float t = (zmin * nr) * inv_vs;
        const float t_end = (zmax * nr) * inv_vs;
        int state = SEARCH_BLOCK_COARSE;
        float F = 1.0f;
        // with bins of every allocated block, and every point of this ray
        // (march from t - 8, two refinement steps of at most mu back) at or
        // beyond the near plane, a table miss proves absence.  Bins of the
        // visible list alone do not: trilinear reads may reach allocated
        // blocks outside it.
        const float zscale = vs * rcz;
        const bool local = all_blocks && tbl.complete && (t - 8.0f - 2.0f * mu_v) * zscale >= kZNear;
        BlockCache cc = {0x7fffffff, 0, 0, -1, -1, local};
        int steps = 0;
        while (t < t_end && steps < kMaxRaySteps) {
            if (state == SEARCH_BLOCK_COARSE || state == SEARCH_BLOCK_FINE) {
                // Empty-space skip: the march stays in this state with a fixed
                // step while it finds no block.  Test the occupancy bricks of the next
                // kSkip positions together; a clear bit proves the block absent,
                // so those iterations are exactly the ones the loop would run.
                const float stp = state == SEARCH_BLOCK_COARSE ? 8.0f : mu_v;
                constexpr int kSkip = 4;
                float tk[kSkip];
                uint32_t hk[kSkip], wk[kSkip];
                float tt = t;
#pragma unroll
                for (int k = 0; k < kSkip; ++k) {
                    tk[k] = tt;
                    const int b0 = block_of(ox + tt * dx), b1 = block_of(oy + tt * dy), b2 = block_of(oz + tt * dz);
                    hk[k] = brick_bit(b0, b1, b2);
                    wk[k] = gload(v.brick + brick_word(b0, b1, b2));
                    tt += stp;
                }
                bool stop = false;
#pragma unroll
                for (int k = 0; k < kSkip; ++k) {
                    if (stop) continue;
                    t = tk[k];
                    if (!(t < t_end && steps < kMaxRaySteps) || (wk[k] & hk[k])) {
                        stop = true;
                        continue;
                    }
                    ++steps;                       // an iteration on unallocated space
                }
                if (!stop) t = tt;
                if (!(t < t_end && steps < kMaxRaySteps)) break;
            }
            ++steps;
            const float P0 = ox + t * dx, P1 = oy + t * dy, P2 = oz + t * dz;
            const bool alloc = allocated_at(v, &tbl, P0, P1, P2, cc);
            if (state == SEARCH_BLOCK_COARSE) {
                if (!alloc) {
                    t += 8.0f;
                } else {
                    t -= 8.0f;
                    state = SEARCH_BLOCK_FINE;
                }
            } else if (!alloc) {
                state = SEARCH_BLOCK_FINE;
                t += mu_v;
            } else {
                F = trilinear<kOff32>(v, &tbl, P0, P1, P2, cc);
                if (state == SEARCH_SURFACE) {
                    if (F < 0.0f) {
                        state = BEHIND_SURFACE;
                        break;
                    }
                    const float s = F * mu_v;
                    t += (s > 1.0f) ? s : 1.0f;
                } else if (F < 0.0f) {
                    if (state == SEARCH_BLOCK_FINE) {
                        state = WRONG_SIDE;
                    } else {
                        const float s = -F * mu_v;
                        t += (s > 1.0f) ? s : 1.0f;
                    }
                } else {
                    // FINE or WRONG_SIDE meeting F >= 0 turns to SURFACE without
                    // a step; the SURFACE iteration that follows (if the step
                    // bound allows it) reads the same cell at the same t, so
                    // its step is taken here with this F
                    state = SEARCH_SURFACE;
                    if (steps < kMaxRaySteps) {
                        ++steps;
                        const float s = F * mu_v;
                        t += (s > 1.0f) ? s : 1.0f;
                    }
                }
            }
        }
        if (state == BEHIND_SURFACE) {
            t += F * mu_v;
            float P0 = ox + t * dx, P1 = oy + t * dy, P2 = oz + t * dz;
            F = trilinear<kOff32>(v, &tbl, P0, P1, P2, cc);
            t += F * mu_v;
            P0 = ox + t * dx;
            P1 = oy + t * dy;
            P2 = oz + t * dz;
            out_p = make_float4(P0 * vs, P1 * vs, P2 * vs, 1.0f);
            float gx = 0.0f, gy = 0.0f, gz = 0.0f;
            // the rare rays whose shifted points round across a voxel take the
            // cells one axis per iteration
#pragma unroll 1
            for (int ax = normal_gradient<kOff32>(v, &tbl, P0, P1, P2, cc, gx, gy, gz) ? 3 : 0; ax < 3; ++ax) {
                const float d = trilinear_diff<kOff32>(v, &tbl, ax == 0 ? P0 + 1.0f : P0, ax == 1 ? P1 + 1.0f : P1,
                                                       ax == 2 ? P2 + 1.0f : P2, ax == 0 ? P0 - 1.0f : P0,
                                                       ax == 1 ? P1 - 1.0f : P1, ax == 2 ? P2 - 1.0f : P2, cc) *
                                0.5f;
                gx = ax == 0 ? d : gx;
                gy = ax == 1 ? d : gy;
                gz = ax == 2 ? d : gz;
            }
            const float gn = sqrtf((gx * gx + gy * gy) + gz * gz);
            if (gn > 0.0f) out_n = make_float4(gx / gn, gy / gn, gz / gn, 1.0f);
        }
    }
    __shared__ uint32_t wg_hits;
    if (threadIdx.x == 0) wg_hits = 0;
    __syncthreads();
    if (inside) {
        const size_t p = (size_t)py * c.W + px;
        pts[p] = out_p;
        nrm[p] = out_n;
        if (out_p.w == 1.0f) atomicAdd(&wg_hits, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && wg_hits) v.acc_hits[tile] += wg_hits;
    finish_tile(v, real ? tile : -1, true);
}

// ============================================================================
// host swapping (Sec. 5)
// ============================================================================
// secondary integration of two copies of one block, per voxel: the weighted
// average (w_a F_a + w_b F_b) / (w_a + w_b), weight min(w_a + w_b, maxW); a
// copy with weight 0 carries no observation.  Result into copy a.
__device__ __forceinline__ void merge_voxel(int &sa, int &wa, int sb, int wb, int max_w)
{
    if (wb == 0) return;
    if (wa == 0) {
        sa = sb;
        wa = wb;
        return;
    }
    const float fa = (float)sa * (1.0f / 32767.0f);
    const float fb = (float)sb * (1.0f / 32767.0f);
    const float avg = ((float)wa * fa + (float)wb * fb) / (float)(wa + wb);
    int w = wa + wb;
    if (w > max_w) w = max_w;
    sa = (int16_t)(avg * 32767.0f);
    wa = w;
}

// visible entries whose host store holds data: swap-in candidates, written
// to the host's note; k_swap_note adds their number once all are there
__global__ __launch_bounds__(256) void k_swap_candidates(Vol v)
{
    const uint32_t n = v.ctrl->n_vis;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) {
        const int e = v.vlist[i];
        if (v.host_has[e]) {
            const uint32_t k = atomicAdd(&v.ctrl->n_swap_cand, 1u);
            v.note[1 + k] = (unsigned long long)e;
        }
    }
}

__global__ void k_swap_note(Vol v) { v.note[0] = v.ctrl->n_swap_cand; }

// eight voxels of a block: 16-bit distances and 8-bit weights
struct Voxels8 {
    uint4 s;
    uint2 w;
};

__device__ __forceinline__ Voxels8 load_voxels8(const uint8_t *block, uint32_t lane)
{
    return {reinterpret_cast<const uint4 *>(block)[lane], reinterpret_cast<const uint2 *>(block + 1024)[lane]};
}

__device__ __forceinline__ void store_voxels8(uint8_t *block, uint32_t lane, const Voxels8 &a)
{
    reinterpret_cast<uint4 *>(block)[lane] = a.s;
    reinterpret_cast<uint2 *>(block + 1024)[lane] = a.w;
}

// secondary integration of eight voxels: b into a
__device__ __forceinline__ void merge_voxels8(Voxels8 &a, const Voxels8 &b, int max_w)
{
    uint32_t as[4] = {a.s.x, a.s.y, a.s.z, a.s.w}, aw[2] = {a.w.x, a.w.y};
    const uint32_t bs[4] = {b.s.x, b.s.y, b.s.z, b.s.w}, bw[2] = {b.w.x, b.w.y};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int hs = 16 * (q & 1), hw = 8 * (q & 3);
        int sa = (int16_t)(as[q >> 1] >> hs), wa = (int)((aw[q >> 2] >> hw) & 255u);
        merge_voxel(sa, wa, (int16_t)(bs[q >> 1] >> hs), (int)((bw[q >> 2] >> hw) & 255u), max_w);
        as[q >> 1] = (as[q >> 1] & ~(0xffffu << hs)) | ((uint32_t)(uint16_t)sa << hs);
        aw[q >> 2] = (aw[q >> 2] & ~(0xffu << hw)) | (((uint32_t)wa & 255u) << hw);
    }
    a.s = make_uint4(as[0], as[1], as[2], as[3]);
    a.w = make_uint2(aw[0], aw[1]);
}

// fuse blocks at .. at + n - 1 of the host's transfer buffer into their
// device blocks, read over the link where they lie (each byte once, whole
// lines: a copy to the device first would only add its launch and a pass);
// one wave per block
__global__ __launch_bounds__(256) void k_swap_merge(Vol v, uint32_t at, uint32_t n)
{
    const uint32_t lane = lane_id();
    const uint32_t gwave = (blockIdx.x * 256u + threadIdx.x) / kWave;
    const uint32_t nwaves = gridDim.x * (256u / kWave);
    if (blockIdx.x == 0 && threadIdx.x == 0) v.ctrl->n_swapped_in = at + n;
    for (uint32_t k = at + gwave; k < at + n; k += nwaves) {
        const int e = v.hx_idx[k];
        const Voxels8 b = load_voxels8(v.hx_vox + (size_t)k * kBlockBytes, lane);
        uint8_t *dst = v.voxels + (size_t)load_entry(v.entries, (uint32_t)e).w * kBlockBytes;
        Voxels8 a = load_voxels8(dst, lane);
        merge_voxels8(a, b, v.max_w);
        store_voxels8(dst, lane, a);
        if (lane == 0) v.host_has[e] = 0;
    }
}

// Swap-out of blocks whose host copy never came back in (Sec. 5, secondary
// integration): the store copies of those entries, uploaded to xfer_host,
// are fused with the device copies the gather put into the transfer buffer
// (slot xfer_pend[k]); the result replaces the store copy.  One wave per block.
__global__ __launch_bounds__(256) void k_swap_merge_out(Vol v, uint32_t n)
{
    const uint32_t lane = lane_id();
    const uint32_t gwave = (blockIdx.x * 256u + threadIdx.x) / kWave;
    const uint32_t nwaves = gridDim.x * (256u / kWave);
    for (uint32_t k = gwave; k < n; k += nwaves) {
        uint8_t *a = v.xfer_host + (size_t)k * kBlockBytes;
        const uint8_t *b = v.xfer_vox + (size_t)v.xfer_pend[k] * kBlockBytes;
        Voxels8 x = load_voxels8(a, lane);
        merge_voxels8(x, load_voxels8(b, lane), v.max_w);
        store_voxels8(a, lane, x);
    }
}

// marks the visible entries (val = 1) or clears the marks (val = 0)
__device__ __forceinline__ void mark_visible(const Vol &v, uint8_t val)
{
    const uint32_t n = v.ctrl->n_vis;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) v.vis[v.vlist[i]] = val;
}

__global__ __launch_bounds__(256) void k_mark_visible(Vol v) { mark_visible(v, (uint8_t)1); }

// Swap-out candidates: a device block and not visible.  Ordered selection of
// the lowest entry indices: per-chunk counts, a scan, then in-order writes.
__device__ __forceinline__ uint32_t wg_exclusive_scan(uint32_t x, uint32_t *lds, uint32_t &total)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
    uint32_t incl = x;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d);
        if ((int)lane >= d) incl += t;
    }
    if (lane == kWave - 1) lds[w] = incl;
    __syncthreads();
    uint32_t base = 0;
    for (uint32_t k = 0; k < w; ++k) base += lds[k];
    total = lds[0] + lds[1] + lds[2] + lds[3];
    __syncthreads();
    return base + incl - x;
}

// a chunk is 16 slices of 256 consecutive entries, one entry per thread in a
// slice; the thread's candidates, bit k = slice k.  The marks and occupancy
// bits of all slices are read together, then the entries they leave (a bucket
// whose occupancy bit is clear never held one; in place of the others, entry
// 0): three reads deep instead of 48, count and pick of 163840 entries 13.6 and
// 10.2 -> 4.7 and 6.8 us.
__device__ __forceinline__ uint32_t swap_slices(const Vol &v, uint32_t e0)
{
    uint32_t mark[16], occ[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t e = e0 + 256u * (uint32_t)k, in = e < v.n_entries ? e : 0u;
        mark[k] = gload(v.vis + in);
        occ[k] = gload(v.occ + (in < v.n_buckets ? in >> 5 : 0u));
    }
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t e = e0 + 256u * (uint32_t)k;
        const bool may = e < v.n_entries && mark[k] == 0u && (e >= v.n_buckets || ((occ[k] >> (e & 31u)) & 1u));
        c |= (may ? 1u : 0u) << k;
    }
    int ptr[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) ptr[k] = gload(&v.entries[(c >> k) & 1u ? e0 + 256u * (uint32_t)k : 0u].ptr);
#pragma unroll
    for (int k = 0; k < 16; ++k)
        if (ptr[k] < 0) c &= ~(1u << k);
    return c;
}

__global__ __launch_bounds__(256) void k_swap_count(Vol v)
{
    __shared__ uint32_t lds[4];
    const uint32_t c = swap_slices(v, blockIdx.x * (uint32_t)kSwapChunk + threadIdx.x);
    uint32_t total;
    wg_exclusive_scan((uint32_t)__popc(c), lds, total);
    if (threadIdx.x == 0) v.swap_chunks[blockIdx.x] = total;
}

// a word of the host's note, seen by the host before the kernel ends
__device__ __forceinline__ void note_word(unsigned long long *p, uint32_t value, uint32_t call)
{
    __hip_atomic_store(p, (unsigned long long)value | ((unsigned long long)call << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// offsets of the chunks, and the number of candidates for the host
__global__ __launch_bounds__(256) void k_swap_scan(Vol v, uint32_t nchunks, uint32_t call)
{
    __shared__ uint32_t lds[4];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nchunks; base += 256u) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t x = i < nchunks ? v.swap_chunks[i] : 0u;
        uint32_t total;
        const uint32_t ex = wg_exclusive_scan(x, lds, total);
        if (i < nchunks) v.swap_chunks[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) {
        v.ctrl->n_swap_cand = carry;
        v.ctrl->n_swapped_out = 0u;
        note_word(v.note, carry, call);
    }
}

// in entry order: slice by slice, and within a slice thread by thread
__global__ __launch_bounds__(256) void k_swap_pick(Vol v)
{
    __shared__ uint32_t cnt[16][4];   // candidates of a slice's waves
    const uint32_t base = v.swap_chunks[blockIdx.x];
    if (base >= v.transfer_blocks) return;   // uniform: every pick of this chunk is past the capacity
    const uint32_t e0 = blockIdx.x * (uint32_t)kSwapChunk + threadIdx.x;
    const uint32_t c = swap_slices(v, e0), lane = lane_id(), w = threadIdx.x / kWave;
    uint32_t before[16];   // lanes of this wave before this one, per slice
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const unsigned long long m = __ballot((c >> k) & 1u);
        before[k] = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) cnt[k][w] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    uint32_t pos = base;
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t p = pos + before[k];
            if (u == w && ((c >> k) & 1u) && p < v.transfer_blocks) v.xfer_idx[p] = (int32_t)(e0 + 256u * (uint32_t)k);
            pos += cnt[k][u];
        }
}

// The selected entries' device blocks into the host's transfer buffer, over
// the link from here, and into the device's for the secondary integration; the
// visibility marks cleared on the side.  One wave per block, which notes its
// entry when the block is on the host: the host's copy into its store runs
// while later blocks are on the link.  The block's stores go through the
// caches (system scope), so that waiting for them is all the note needs.
// Bound by the link (4.8 MB in 144 us, 33 GB/s); the launch is small, so that
// blocks arrive one after the other: with a wave for each block they all
// arrive at the end, and the host was 186 us behind instead of 109.
__global__ __launch_bounds__(256) void k_swap_gather(Vol v, uint32_t call)
{
    const uint32_t lane = lane_id();
    const uint32_t gwave = (blockIdx.x * 256u + threadIdx.x) / kWave;
    const uint32_t nwaves = gridDim.x * (256u / kWave);
    const uint32_t cand = v.ctrl->n_swap_cand;
    const uint32_t n = cand < v.transfer_blocks ? cand : v.transfer_blocks;
    for (uint32_t k = gwave; k < n; k += nwaves) {
        const uint32_t e = (uint32_t)v.xfer_idx[k];
        const int ptr = load_entry(v.entries, e).w;
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(v.voxels + (size_t)ptr * kBlockBytes);
        unsigned long long *dev = reinterpret_cast<unsigned long long *>(v.xfer_vox + (size_t)k * kBlockBytes);
        unsigned long long *host = reinterpret_cast<unsigned long long *>(v.hx_vox + (size_t)k * kBlockBytes);
        unsigned long long x[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) x[q] = src[lane + 64u * q];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            __hip_atomic_store(host + lane + 64u * q, x[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            dev[lane + 64u * q] = x[q];
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) note_word(v.note + 1 + k, e, call);
    }
    mark_visible(v, (uint8_t)0);
}

// The first n selected entries' blocks back onto the free stack, the entries
// marked swapped out (one workgroup).  A launch of its own, made once the host
// holds the blocks: until then the map is as it was, whatever fails.
__global__ __launch_bounds__(1024) void k_swap_release(Vol v, uint32_t n)
{
    const int32_t head = v.ctrl->free_blocks;
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n; k += 1024u) {
        const int e = v.xfer_idx[k];
        v.free_blocks[head + (int32_t)k] = v.entries[e].ptr;
        v.entries[e].ptr = kPtrSwapped;
        v.host_has[e] = 1;
    }
    if (threadIdx.x == 0) {
        v.ctrl->free_blocks = head + (int32_t)n;
        v.ctrl->n_swapped_out = n;
    }
}

// ============================================================================
// export of voxels in the in-block order lx + 8 ly + 64 lz
// ============================================================================
__global__ __launch_bounds__(256) void k_export_voxels(Vol v, const int32_t *ids, uint32_t n, int16_t *sdf, uint8_t *wt)
{
    const uint32_t lane = lane_id();
    const uint32_t gwave = (blockIdx.x * 256u + threadIdx.x) / kWave;
    const uint32_t nwaves = gridDim.x * (256u / kWave);
    const int lx = (int)(lane >> 3), ly = (int)(lane & 7);
    for (uint32_t k = gwave; k < n; k += nwaves) {
        const int e = ids[k];
        int ptr = -1;
        if (e >= 0 && (uint32_t)e < v.n_entries) ptr = load_entry(v.entries, (uint32_t)e).w;
        for (int lz = 0; lz < 8; ++lz) {
            int16_t s = 32767;
            uint8_t w = 0;
            if (ptr >= 0) {
                const uint8_t *blk = v.voxels + (size_t)ptr * kBlockBytes;
                s = reinterpret_cast<const int16_t *>(blk)[lane * 8 + lz];
                w = blk[1024 + lane * 8 + lz];
            }
            const size_t o = (size_t)k * kBlockVox + lx + 8 * ly + 64 * lz;
            sdf[o] = s;
            wt[o] = w;
        }
    }
}

// ============================================================================
// camera depth of raycast hits (training targets of the prefilter)
// ============================================================================
struct Row3 {
    float m8, m9, m10, m11;
};

__global__ __launch_bounds__(256) void k_camera_depth(const float4 *pts, int n, Row3 r, float *depth)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const float4 q = pts[p];
    depth[p] = q.w == 1.0f ? ((r.m8 * q.x + r.m9 * q.y) + r.m10 * q.z) + r.m11 : 0.0f;
}

// ============================================================================
// launchers
// ============================================================================
static int cu_grid(size_t work, int per_block, int cap)
{
    size_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > (size_t)cap) g = cap;
    return (int)g;
}

hipError_t launch_init(const Vol &v, uint32_t max_tiles, hipStream_t s)
{
    size_t work = v.n_entries > max_tiles ? v.n_entries : max_tiles;
    if (v.n_blocks > work) work = v.n_blocks;
    if ((size_t)v.reqset_mask + 1 > work) work = (size_t)v.reqset_mask + 1;
    hipLaunchKernelGGL(k_init, dim3(cu_grid(work, 256, 8192)), dim3(256), 0, s, v, max_tiles);
    return hipGetLastError();
}

hipError_t launch_clear_bins(const Vol &v, uint32_t max_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_bins, dim3(cu_grid(max_tiles, 256, 1024)), dim3(256), 0, s, v, max_tiles);
    return hipGetLastError();
}

hipError_t launch_alloc_rays(const Vol &v, const Cam &c, const void *depth, int fmt, hipStream_t s)
{
    const int npix = c.W * c.H;
    const dim3 g((npix + 255) / 256 + kKeepGroups), b(256);
    if (fmt == TF_DEPTH_U16_MM)
        hipLaunchKernelGGL(k_alloc_rays<TF_DEPTH_U16_MM>, g, b, 0, s, v, c, depth);
    else
        hipLaunchKernelGGL(k_alloc_rays<TF_DEPTH_F32_M>, g, b, 0, s, v, c, depth);
    return hipGetLastError();
}

hipError_t launch_insert(const Vol &v, const Cam &c, hipStream_t s)
{
    hipLaunchKernelGGL(k_insert, dim3(512), dim3(256), 0, s, v, c);
    return hipGetLastError();
}

hipError_t launch_visible(const Vol &v, hipStream_t s)
{
    const size_t nchunks = ((size_t)v.n_entries + 15) / 16;
    hipLaunchKernelGGL(k_visible, dim3(cu_grid(nchunks, 256, 4096)), dim3(256), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_depth_convert(const Vol &v, const void *depth, int fmt, int n, hipStream_t s)
{
    const dim3 g((n + 255) / 256), b(256);
    if (fmt == TF_DEPTH_U16_MM)
        hipLaunchKernelGGL(k_depth_convert<TF_DEPTH_U16_MM>, g, b, 0, s, v.depth, depth, n);
    else
        hipLaunchKernelGGL(k_depth_convert<TF_DEPTH_F32_M>, g, b, 0, s, v.depth, depth, n);
    return hipGetLastError();
}

hipError_t launch_integrate(const Vol &v, const Cam &c, bool bin, hipStream_t s)
{
    hipLaunchKernelGGL(k_integrate, dim3(kIntegrateGrid), dim3(256), 0, s, v, c, bin ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_range_bin(const Vol &v, const Cam &c, bool all_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_range_bin, dim3(kBinGrid), dim3(256), 0, s, v, c, all_blocks ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_raycast(const Vol &v, const Cam &c, bool all_blocks, float4 *pts, float4 *nrm, hipStream_t s)
{
    const int grid = ((c.W + kTile - 1) / kTile) * ((c.H + kTile - 1) / kTile);   // one workgroup per tile
    if ((size_t)v.n_blocks * kBlockBytes <= 0xffffffffu)
        hipLaunchKernelGGL(k_raycast<true>, dim3(grid), dim3(256), 0, s, v, c, all_blocks ? 1 : 0, pts, nrm);
    else
        hipLaunchKernelGGL(k_raycast<false>, dim3(grid), dim3(256), 0, s, v, c, all_blocks ? 1 : 0, pts, nrm);
    return hipGetLastError();
}

hipError_t launch_range_write(const Vol &v, const Cam &c, float *zmin, float *zmax, hipStream_t s)
{
    const int ntiles = ((c.W + kTile - 1) / kTile) * ((c.H + kTile - 1) / kTile);
    hipLaunchKernelGGL(k_range_write, dim3(ntiles), dim3(256), 0, s, v, c, zmin, zmax);
    return hipGetLastError();
}

hipError_t launch_camera_depth(const float4 *pts, int n, const float *M, float *depth, hipStream_t s)
{
    const Row3 r = {M[8], M[9], M[10], M[11]};
    hipLaunchKernelGGL(k_camera_depth, dim3((n + 255) / 256), dim3(256), 0, s, pts, n, r, depth);
    return hipGetLastError();
}

hipError_t launch_export_voxels(const Vol &v, const int32_t *ids, uint32_t n, int16_t *sdf, uint8_t *w, hipStream_t s)
{
    hipLaunchKernelGGL(k_export_voxels, dim3(cu_grid((size_t)n * 64, 256, 4096)), dim3(256), 0, s, v, ids, n, sdf, w);
    return hipGetLastError();
}

}  // namespace tsdf

namespace tsdf {
hipError_t launch_swap_candidates(const Vol &v, hipStream_t s)
{
    hipLaunchKernelGGL(k_swap_candidates, dim3(256), dim3(256), 0, s, v);
    hipLaunchKernelGGL(k_swap_note, dim3(1), dim3(1), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_swap_merge(const Vol &v, uint32_t at, uint32_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_swap_merge, dim3(cu_grid((size_t)n * 64, 256, 2048)), dim3(256), 0, s, v, at, n);
    return hipGetLastError();
}

hipError_t launch_swap_select(const Vol &v, uint32_t call, hipStream_t s)
{
    const uint32_t nchunks = (v.n_entries + kSwapChunk - 1) / kSwapChunk;
    hipLaunchKernelGGL(k_mark_visible, dim3(256), dim3(256), 0, s, v);
    hipLaunchKernelGGL(k_swap_count, dim3(nchunks), dim3(256), 0, s, v);
    hipLaunchKernelGGL(k_swap_scan, dim3(1), dim3(256), 0, s, v, nchunks, call);
    return hipGetLastError();
}

hipError_t launch_swap_gather(const Vol &v, uint32_t call, hipStream_t s)
{
    const uint32_t nchunks = (v.n_entries + kSwapChunk - 1) / kSwapChunk;
    hipLaunchKernelGGL(k_swap_pick, dim3(nchunks), dim3(256), 0, s, v);
    // 256 waves of 1.5 KB each cover the link's latency several times
    hipLaunchKernelGGL(k_swap_gather, dim3(64), dim3(256), 0, s, v, call);
    return hipGetLastError();
}

hipError_t launch_swap_release(const Vol &v, uint32_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_swap_release, dim3(1), dim3(1024), 0, s, v, n);
    return hipGetLastError();
}

hipError_t launch_swap_merge_out(const Vol &v, uint32_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_swap_merge_out, dim3(cu_grid((size_t)n * 64, 256, 2048)), dim3(256), 0, s, v, n);
    return hipGetLastError();
}
}  // namespace tsdf

// tsdf_multi.hip -- gfx950 kernels of the batched rigid submaps (Sec. 7.2).
//
//   k_m_alloc / k_m_insert / k_m_visible / k_m_integrate
//       one depth frame into the submaps selected for it, blockIdx.y = slot of
//       the selection; each runs the single-volume body on its submap with the
//       camera composed with that submap's pose
//   k_m_bin<false>, k_m_scan, k_m_bin<true>
//       every allocated block of every submap against every view: count the
//       (block, tile) pairs, exclusive offsets, then fill the tile bins.  A
//       block is binned by its cube grown by kExpand voxels, so that a tile's
//       bin holds every block any trilinear read of its rays can touch
//   k_m_raycast<TW, TH>
//       one workgroup per TWxTH tile of any view: the per-pixel search range,
//       the tile's submap set and an LDS block table from the bin, then the
//       ray state machine on the combined field
//
// The combined field at a world point (voxel units) is the weighted average of
// the submaps' trilinear SDF, each weighted by its trilinear weight, over the
// submaps whose weight there is positive; one contributor gives its value
// unchanged and none gives 1.  Submaps are summed in ascending index order.
#include "tsdf_device.h"

namespace tsdf {

// ============================================================================
// integration of one frame into the selected submaps
// ============================================================================
__global__ __launch_bounds__(256) void k_m_alloc(const Vol *vols, const MFrame *f)
{
    const int y = (int)blockIdx.y;
    if (y >= f->n_sel) return;
    const Vol v = vols[f->sel[y]];
    const Cam c = f->icam[y];
    // every submap reads the one shared depth map; slot 0 writes it
    if (f->fmt == TF_DEPTH_U16_MM)
        alloc_rays_body<TF_DEPTH_U16_MM>(v, c, f->depth, y == 0);
    else
        alloc_rays_body<TF_DEPTH_F32_M>(v, c, f->depth, y == 0);
}

__global__ __launch_bounds__(256) void k_m_insert(const Vol *vols, const MFrame *f)
{
    const int y = (int)blockIdx.y;
    if (y >= f->n_sel) return;
    const Vol v = vols[f->sel[y]];
    const Cam c = f->icam[y];
    insert_body(v, c);
}

__global__ __launch_bounds__(256) void k_m_visible(const Vol *vols, const MFrame *f)
{
    const int y = (int)blockIdx.y;
    if (y >= f->n_sel) return;
    const Vol v = vols[f->sel[y]];
    visible_body(v);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_m_integrate(const Vol *vols, const MFrame *f, int dry)
{
    __shared__ float rcp_w[260];
    __shared__ uint32_t wg_cols;
    const int y = (int)blockIdx.y;
    if (y >= f->n_sel) return;
    const Vol v = vols[f->sel[y]];
    const Cam c = f->icam[y];
    integrate_body<NT>(v, c, rcp_w, &wg_cols, dry != 0);
}

// ============================================================================
// tile bins of every view
// ============================================================================
// LDS of a binning workgroup: the distinct tiles of one chunk of blocks
// (open addressing on the tile index) with their entry counts, then their
// reserved positions
constexpr int kBinSlots = 1024;
constexpr int kBinProbes = 32;        // probes before a tile takes the global path
constexpr int kBinDirect = 16;        // blocks over more tiles take the global path for all of them
constexpr uint32_t kNoTile = 0xffffffffu;
constexpr int kBinBig = 128;          // blocks over many tiles whose tiles the workgroup shares
struct MBinLds {
    uint32_t tile[kBinSlots];
    uint32_t cnt[kBinSlots];
    uint32_t pos[kBinSlots];
    uint32_t first[kMaxSubmaps + 1];   // flat index of each submap's first block
    float C[kMaxSubmaps][12];          // the view's camera composed with each submap pose
    Rec big_rec[kBinBig];              // fill pass: the record of each queued block
    int4 big_box[kBinBig];             // tx0, ty0, tiles per row, tiles
    uint32_t nbig;
    uint32_t pairs;                    // count pass: (block, view) pairs of the workgroup
};

// slot of tile g in the chunk table, inserting it when `insert`; -1 when
// the first kBinProbes slots of its probe sequence hold other tiles (or,
// without insert, do not hold g).  Slots are never emptied within a chunk,
// so a tile refused once is refused for the rest of the chunk.
__device__ __forceinline__ int bin_slot(MBinLds &B, uint32_t g, bool insert)
{
    uint32_t sl = (g * 0x9e3779b1u) >> 22;   // 10 bits
    for (int k = 0; k < kBinProbes; ++k) {
        const uint32_t cur = insert ? atomicCAS(&B.tile[sl], kNoTile, g) : B.tile[sl];
        if (cur == g || (insert && cur == kNoTile)) return (int)sl;
        if (cur == kNoTile) return -1;
        sl = (sl + 1u) & (uint32_t)(kBinSlots - 1);
    }
    return -1;
}

// Every allocated block of every submap against view blockIdx.y: its cube
// grown by kExpand voxels gives the tiles whose bins take its record.  Count
// pass (FILL false): entries per tile; fill pass: the records at the tile's
// offset.  The blocks of all submaps form one flat index range (submap by
// submap); a workgroup takes 256 consecutive blocks at a time and aggregates
// their (block, tile) entries per distinct tile in LDS, so a tile costs one
// global atomic per chunk instead of one per entry (an entry whose tile the
// chunk table refuses takes a global atomic of its own).  A block over more
// than kBinDirect tiles -- near the camera it can cover thousands -- is queued
// and its tiles are shared by the workgroup's threads, one global atomic
// each.  The order of records within a bin is not fixed.
template <bool FILL>
__global__ __launch_bounds__(256) void k_m_bin(const MSub *subs, const MFrame *f, MTiles t, float voxel)
{
    __shared__ MBinLds B;
    const int vi = (int)blockIdx.y;
    if (vi >= f->n_views) return;
    const Cam vc = f->view[vi].cam;
    const int ntx = f->view[vi].ntx, base = f->view[vi].tile_base;
    const int tw = f->tw, th = f->th;
    const int n_sub = f->n_sub;
    for (int k = threadIdx.x; k < kBinSlots; k += 256) {
        B.tile[k] = kNoTile;
        B.cnt[k] = 0u;
    }
    for (int k = threadIdx.x; k < n_sub * 12; k += 256) B.C[k / 12][k % 12] = f->C[vi][k / 12][k % 12];
    if (threadIdx.x == 0) {
        B.nbig = 0u;
        B.pairs = 0u;
        uint32_t acc = 0u;
        for (int sm = 0; sm < n_sub; ++sm) {
            B.first[sm] = acc;
            acc += subs[sm].ctrl->n_alloc;
        }
        B.first[n_sub] = acc;
    }
    const Frustum fr = make_frustum(vc, voxel, kExpand);
    __syncthreads();
    const uint32_t total = B.first[n_sub];
    // whole chunks for every thread of the workgroup (barriers inside)
    for (uint32_t c0 = blockIdx.x * 256u; c0 < total; c0 += gridDim.x * 256u) {
        const uint32_t gi = c0 + threadIdx.x;
        bool hit = false;
        Rec ex, r;
        int bx = 0, by = 0, bz = 0, ptr = 0, sm = 0;
        const float *M = B.C[0];
        if (gi < total) {
            // the submap of flat index gi: the last with first[sm] <= gi
#pragma unroll
            for (int step = kMaxSubmaps / 2; step; step >>= 1)
                if (sm + step < n_sub && B.first[sm + step] <= gi) sm += step;
            M = B.C[sm];
            const int4 b = subs[sm].alist[gi - B.first[sm]];
            bx = (int16_t)(b.x & 0xffff);
            by = (int16_t)((uint32_t)b.x >> 16);
            bz = b.y;
            ptr = b.z;
            hit = !outside_frustum(fr, M, vc, voxel, bx, by, bz) &&
                  cube_record(M, vc, voxel, 8 * bx - kExpand, 8 * by - kExpand, 8 * bz - kExpand, 8 + 2 * kExpand, ex);
        }
        if (!FILL) {
            const unsigned long long m = __ballot(hit);
            if (m && lane_id() == (uint32_t)(__ffsll((long long)m) - 1)) atomicAdd(&B.pairs, (uint32_t)__popcll(m));
        }
        const int tx0 = hit ? ex.x0 / tw : 1, tx1 = hit ? ex.x1 / tw : 0;
        const int ty0 = hit ? ex.y0 / th : 1, ty1 = hit ? ex.y1 / th : 0;
        const int nx = tx1 - tx0 + 1, ntl = nx * (ty1 - ty0 + 1);
        const bool direct = ntl > kBinDirect;
        // a block over many tiles: queued for the whole workgroup (the count
        // pass here, the fill pass with its record below), unless the queue
        // is full; its tiles then take one global atomic each from this thread
        bool queued = false;
        if (!FILL && hit && direct) {
            const uint32_t j = atomicAdd(&B.nbig, 1u);
            if (j < (uint32_t)kBinBig) {
                B.big_box[j] = make_int4(tx0, ty0, nx, ntl);
                queued = true;
            }
        }
        // entries per distinct tile of the chunk
        if (!queued)
            for (int ty = ty0; ty <= ty1; ++ty)
                for (int tx = tx0; tx <= tx1; ++tx) {
                    const uint32_t g = (uint32_t)(base + ty * ntx + tx);
                    const int sl = direct ? -1 : bin_slot(B, g, true);
                    if (sl >= 0)
                        atomicAdd(&B.cnt[sl], 1u);
                    else if (!FILL)
                        atomicAdd(&t.cnt[g], 1);
                }
        __syncthreads();
        const uint32_t nq = FILL ? 0u : (B.nbig < (uint32_t)kBinBig ? B.nbig : (uint32_t)kBinBig);
        // one global atomic per distinct tile: its count, or its range in the bin
        for (int k = threadIdx.x; k < kBinSlots; k += 256) {
            const uint32_t g = B.tile[k];
            if (g == kNoTile) continue;
            if (FILL)
                B.pos[k] = t.off[g] + (uint32_t)atomicAdd(&t.cur[g], (int)B.cnt[k]);
            else
                atomicAdd(&t.cnt[g], (int)B.cnt[k]);
        }
        __syncthreads();
        // count pass: the queued blocks' tiles, shared by every thread
        for (uint32_t j = 0; j < nq; ++j) {
            const int4 bb = B.big_box[j];
            for (int k = (int)threadIdx.x; k < bb.w; k += 256)
                atomicAdd(&t.cnt[(uint32_t)(base + (bb.y + k / bb.z) * ntx + bb.x + k % bb.z)], 1);
        }
        if (FILL && hit) {
            // the search-range box of the block itself (empty when it is
            // behind the near plane or off the image: then it only feeds
            // the table)
            if (!cube_record(M, vc, voxel, 8 * bx, 8 * by, 8 * bz, 8, r)) {
                r.x0 = 1;
                r.x1 = 0;
                r.y0 = 1;
                r.y1 = 0;
                r.zlo = __builtin_inff();
                r.zhi = -__builtin_inff();
            }
            r.bx = (int16_t)bx;
            r.by = (int16_t)by;
            r.bz = (int16_t)bz;
            r.pad = (int16_t)sm;
            r.ptr = ptr;
            r.pad2 = (int32_t)__float_as_uint(ex.zlo);   // the grown cube's least camera depth (table depth cut)
            bool fq = false;
            if (direct) {
                const uint32_t j = atomicAdd(&B.nbig, 1u);
                if (j < (uint32_t)kBinBig) {
                    B.big_rec[j] = r;
                    B.big_box[j] = make_int4(tx0, ty0, nx, ntl);
                    fq = true;
                }
            }
            if (!fq)
                for (int ty = ty0; ty <= ty1; ++ty)
                    for (int tx = tx0; tx <= tx1; ++tx) {
                        const uint32_t g = (uint32_t)(base + ty * ntx + tx);
                        const int sl = direct ? -1 : bin_slot(B, g, false);
                        const uint32_t idx =
                            sl >= 0 ? atomicAdd(&B.pos[sl], 1u) : t.off[g] + (uint32_t)atomicAdd(&t.cur[g], 1);
                        if (idx < t.cap) t.bins[idx] = r;
                    }
        }
        if (FILL) {
            __syncthreads();   // every block queued
            // fill pass: the queued blocks' records, each tile by one thread
            const uint32_t nf = B.nbig < (uint32_t)kBinBig ? B.nbig : (uint32_t)kBinBig;
            for (uint32_t j = 0; j < nf; ++j) {
                const int4 bb = B.big_box[j];
                for (int k = (int)threadIdx.x; k < bb.w; k += 256) {
                    const uint32_t g = (uint32_t)(base + (bb.y + k / bb.z) * ntx + bb.x + k % bb.z);
                    const uint32_t idx = t.off[g] + (uint32_t)atomicAdd(&t.cur[g], 1);
                    if (idx < t.cap) t.bins[idx] = B.big_rec[j];
                }
            }
            __syncthreads();   // every slot position taken and the queue read before both are cleared
        }
        for (int k = threadIdx.x; k < kBinSlots; k += 256) {
            B.tile[k] = kNoTile;
            B.cnt[k] = 0u;
        }
        if (threadIdx.x == 0) B.nbig = 0u;
        __syncthreads();
    }
    // one global atomic per workgroup for the statistics (a same-address
    // atomic from every wave and chunk serialised the count pass)
    if (!FILL && threadIdx.x == 0 && B.pairs) atomicAdd(&t.mc->tot_blkview, (unsigned long long)B.pairs);
}

// exclusive offsets of the tile counts (one workgroup); clears the counts and
// cursors for the next launch
__global__ __launch_bounds__(1024) void k_m_scan(MTiles t)
{
    __shared__ uint32_t part[1024];
    const uint32_t n = t.n_tiles;
    const uint32_t per = (n + 1023u) / 1024u;
    const uint32_t b0 = threadIdx.x * per;
    const uint32_t b1 = b0 + per < n ? b0 + per : n;
    uint32_t sum = 0;
    for (uint32_t i = b0; i < b1; ++i) sum += (uint32_t)t.cnt[i];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t d = 1; d < 1024u; d <<= 1) {
        const uint32_t add = threadIdx.x >= d ? part[threadIdx.x - d] : 0u;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    uint32_t run = part[threadIdx.x] - sum;
    for (uint32_t i = b0; i < b1; ++i) {
        const uint32_t c = (uint32_t)t.cnt[i];
        t.off[i] = run;
        run += c;
        t.cnt[i] = 0;
        t.cur[i] = 0;
    }
    if (threadIdx.x == 1023) {
        const uint32_t total = part[1023];
        t.off[n] = total;
        t.mc->tot_bin += total;
        t.mc->n_raycast += 1ull;
        if (total > t.cap) t.mc->flags |= TF_FLAG_BIN_OVERFLOW;
    }
}

__global__ __launch_bounds__(256) void k_m_clear(MTiles t)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < t.n_tiles; i += gridDim.x * 256u) {
        t.cnt[i] = 0;
        t.cur[i] = 0;
        t.off[i] = 0u;
        t.acc_hits[i] = 0ull;
    }
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < kWorldCells; i += gridDim.x * 256u) t.wmask[i] = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) t.off[t.n_tiles] = 0u;
}

// slot of world cell (cx, cy, cz) (8-voxel cells of world voxel units) in the
// submap-mask array: a 512 x 512 x 128 window, cells a window apart share a
// slot (their masks merge, which only adds submaps to visit)
__device__ __forceinline__ uint32_t wcell_index(int cx, int cy, int cz)
{
    return (((uint32_t)cx & 511u) << 16) | (((uint32_t)cy & 511u) << 7) | ((uint32_t)cz & 127u);
}

// World submap masks: every block a selected submap gained this frame (its
// allocated list past n_marked) sets the submap's bit in the 8-voxel world
// cells of its cube's world-space box, grown by two voxels.  A trilinear
// read at a point reaches voxels within one voxel per submap axis, i.e.
// within sqrt(3) voxels of the point in world space, so a submap with any
// voxel of a block under the read of point P has its bit in P's cell (the
// growth also covers the rounding of the pose transforms).  A cell's mask
// thus lists every submap that can be allocated at, or weigh in the field
// at, any point of the cell.  Blocks are never removed, so bits are never
// cleared.
__global__ __launch_bounds__(256) void k_m_mark(const Vol *vols, const MSub *subs, const MFrame *f,
                                                unsigned long long *wmask)
{
    const int y = (int)blockIdx.y;
    if (y >= f->n_sel) return;
    const int si = f->sel[y];
    const Vol v = vols[si];
    const MSub &S = subs[si];
    const uint32_t n0 = v.ctrl->n_marked;
    uint32_t n1 = v.ctrl->n_alloc;
    if (n1 > v.n_blocks) n1 = v.n_blocks;
    for (uint32_t i = n0 + blockIdx.x * 256u + threadIdx.x; i < n1; i += gridDim.x * 256u) {
        const int4 a = v.alist[i];
        const int bx = (int16_t)(a.x & 0xffff), by = (int16_t)((uint32_t)a.x >> 16), bz = a.y;
        float lo[3] = {__builtin_inff(), __builtin_inff(), __builtin_inff()};
        float hi[3] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
        for (int k = 0; k < 8; ++k) {
            // corner of the block in submap voxel units, to world: P = R^T (Q - s)
            const float q0 = (float)(8 * (bx + (k & 1))) - S.s[0];
            const float q1 = (float)(8 * (by + ((k >> 1) & 1))) - S.s[1];
            const float q2 = (float)(8 * (bz + (k >> 2))) - S.s[2];
            for (int r = 0; r < 3; ++r) {
                const float w = (S.R[r] * q0 + S.R[3 + r] * q1) + S.R[6 + r] * q2;
                lo[r] = w < lo[r] ? w : lo[r];
                hi[r] = w > hi[r] ? w : hi[r];
            }
        }
        int c0[3], c1[3];
        for (int r = 0; r < 3; ++r) {
            c0[r] = ((int)floorf(lo[r] - 2.0f)) >> 3;
            c1[r] = ((int)floorf(hi[r] + 2.0f)) >> 3;
        }
        const unsigned long long bit = 1ull << (uint32_t)si;
        for (int cx = c0[0]; cx <= c1[0]; ++cx)
            for (int cy = c0[1]; cy <= c1[1]; ++cy)
                for (int cz = c0[2]; cz <= c1[2]; ++cz) atomicOr(&wmask[wcell_index(cx, cy, cz)], bit);
    }
}

// ============================================================================
// combined-field raycast
// ============================================================================
namespace {

// Depth buckets of the table cut: 1/32 octave each from the near plane up
// (the float bits of a depth above the near plane, shifted), 256 buckets
// (about 0.05 to 12.8 m; deeper depths share the last)
constexpr uint32_t kZBuckets = 256;
constexpr uint32_t kZNearBits = 0x3d4ccccdu;   // kZNear's float bits

__device__ __forceinline__ uint32_t zbucket(uint32_t zbits)
{
    const int b = (int)(zbits >> 18) - (int)(kZNearBits >> 18);
    return b < 0 ? 0u : (b >= (int)kZBuckets ? kZBuckets - 1u : (uint32_t)b);
}

// least depth of bucket b (b >= 1)
__device__ __forceinline__ float zbucket_floor(uint32_t b)
{
    return __uint_as_float(((kZNearBits >> 18) + b) << 18);
}

// LDS of one tile: the (submap, block) -> pointer table, the tile's submaps
// in ascending order with what the field reads
template <int NT>
struct MTileLds {
    static constexpr int kBits = NT >= 128 ? 12 : 11;
    static constexpr int TT = 1 << kBits;       // table slots (8 bytes each)
    static constexpr int kStage = TT / 4;       // records staged at a time for the range
    union {
        unsigned long long slot[TT];            // 0 = empty, else key << 32 | device pointer
        struct {
            uint4 box[kStage];                  // x0, y0, x1, y1 (int16), zlo, zhi (float)
            uint16_t wlist[NT / 64][kStage];    // per wave: the staged records whose box meets its pixels
            uint32_t zlo[NT], zhi[NT];          // per pixel of the tile, row by row: from boxes of a few pixels
        } r;                                    // before the table is filled
    };
    float Rs[kMaxSubmaps][12];                  // rotation rows, then translation (voxel units)
    const DEntry *ent[kMaxSubmaps];
    const uint32_t *occ[kMaxSubmaps];
    const uint8_t *vox[kMaxSubmaps];
    uint32_t nb[kMaxSubmaps], ne[kMaxSubmaps];
    int smid[kMaxSubmaps];
    int org[kMaxSubmaps][3];                    // block at the low corner of the table's window
    unsigned long long mask;
    uint32_t n_tab, hits;
    uint32_t cut;                               // depth buckets 0 .. cut - 1 are in the table
    uint32_t dlim;                              // a lookup miss proves absence for reads of points shallower
                                                // than this depth (float bits)
    int wcnt[NT / 64];
};

// Table key of a block of the tile's k-th submap: its position within a window
// of 256 blocks per axis, 8 bits each, the submap and a valid bit.  Blocks in
// the table lie at 1 .. 254 of the window, so that the seven neighbours of any
// position 0 .. 254 have the keys key + 1, + 256, + 65536 and their sums, and
// outside that no neighbour is in the table either.  The slot hash is a
// multiplication, so the neighbours' hashes are sums as well: a cell that
// crosses block faces finds its seven blocks with a few additions and seven
// reads in flight, where one lookup after another cost ~70 instructions each.
// A block outside the window gets the valid bit alone: its fields would run into
// one another, and a neighbour's sum could then come to 0, an empty slot's key.
constexpr uint32_t kHashMul = 0x9e3779b1u;

__device__ __forceinline__ uint32_t m_neighbour(int n)   // key offset of neighbour n at (n & 1, n >> 1 & 1, n >> 2)
{
    return (uint32_t)((n & 1) | ((n & 2) << 7) | ((n & 4) << 14));
}

template <int NT>
__device__ __forceinline__ bool m_key(const MTileLds<NT> &L, int k, int bx, int by, int bz, uint32_t &key)
{
    const uint32_t rx = (uint32_t)(bx - L.org[k][0]), ry = (uint32_t)(by - L.org[k][1]),
                   rz = (uint32_t)(bz - L.org[k][2]);
    const uint32_t m = rx > ry ? rx : ry;
    const bool in = (m > rz ? m : rz) <= 254u;
    key = 0x80000000u | (in ? ((uint32_t)k << 24) | (rz << 16) | (ry << 8) | rx : 0u);
    return in;
}

template <int NT>
__device__ __forceinline__ uint32_t m_slot(uint32_t hash)
{
    return hash >> (32 - MTileLds<NT>::kBits);
}

// records of tile g's bin, from o0 on
__device__ __forceinline__ int m_bin_range(const MTiles &t, uint32_t g, uint32_t &o0)
{
    o0 = t.off[g];
    uint32_t o1 = t.off[g + 1];
    if (o1 > t.cap) o1 = t.cap;
    return o1 > o0 ? (int)(o1 - o0) : 0;
}

// Search range of pixel (px, py) -- the calling thread's, in its wave's 8 x 8
// square of the tile [tx0, tx0 + TW) x [ty0, ty0 + TH) -- and the tile's
// submap set from its bin.  Every thread of the workgroup calls it.  The range
// is a min / max over the records covering the pixel.  A record whose box holds
// at most kScatter pixels updates those of the tile in LDS (positive floats order
// like their bits); the others' boxes are staged in LDS (in the bytes of the
// block table, filled afterwards), each listed for the waves whose pixels it
// meets, and every thread goes through its wave's list.  Scattered, a large box
// leaves one lane with two atomics for each of its pixels; listed, every lane
// looks at a box that few of them need, and a view that has a whole map in a
// few tiles has 100 k of those in a bin: six submaps of 2.5 mm voxels 12 m away,
// 64x48 pixels, 22.4 ms with all of them listed, 4.8 with all scattered, 2.8
// with boxes of 9 or of 16 pixels as the line.
constexpr int kScatter = 16;

template <int NT, int TW, int TH>
__device__ __forceinline__ void m_pixel_range(const MTiles &t, uint32_t g, int tx0, int ty0, int px, int py,
                                              MTileLds<NT> &L, float &zmin, float &zmax)
{
    constexpr int kStage = MTileLds<NT>::kStage, kWaves = NT / 64;
    const int wave = (int)threadIdx.x >> 6;
    if (threadIdx.x < kWaves) L.wcnt[threadIdx.x] = 0;
    const int at = (py - ty0) * TW + (px - tx0);
    L.r.zlo[at] = 0x7f800000u;   // +inf
    L.r.zhi[at] = 0u;            // below every depth
    if (threadIdx.x == 0) {
        L.mask = 0ull;
        L.n_tab = 0u;
        L.hits = 0u;
    }
    uint32_t o0;
    const int n = m_bin_range(t, g, o0);
    zmin = __builtin_inff();
    zmax = -__builtin_inff();
    unsigned long long mask = 0ull;   // submaps of this thread's records
    for (int b0 = 0; b0 < n; b0 += kStage) {
        const int m = n - b0 < kStage ? n - b0 : kStage;
        __syncthreads();   // the lists are empty, the previous records consumed
        for (int j = (int)threadIdx.x; j < m; j += NT) {
            const uint4 b = *reinterpret_cast<const uint4 *>(t.bins + o0 + (uint32_t)(b0 + j));
            mask |= 1ull << (uint32_t)t.bins[o0 + (uint32_t)(b0 + j)].pad;
            const int x0 = (int16_t)(b.x & 0xffffu), y0 = (int16_t)(b.x >> 16);
            const int x1 = (int16_t)(b.y & 0xffffu), y1 = (int16_t)(b.y >> 16);
            if ((x1 - x0 + 1) * (y1 - y0 + 1) <= kScatter) {   // (a record without a range has an empty box)
                const int u0 = x0 > tx0 ? x0 : tx0, u1 = x1 < tx0 + TW - 1 ? x1 : tx0 + TW - 1;
                const int v0 = y0 > ty0 ? y0 : ty0, v1 = y1 < ty0 + TH - 1 ? y1 : ty0 + TH - 1;
                for (int v = v0; v <= v1; ++v)
                    for (int u = u0; u <= u1; ++u) {
                        atomicMin(&L.r.zlo[(v - ty0) * TW + u - tx0], b.z);
                        atomicMax(&L.r.zhi[(v - ty0) * TW + u - tx0], b.w);
                    }
                continue;
            }
            L.r.box[j] = b;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const int wx0 = tx0 + (w % (TW / 8)) * 8, wy0 = ty0 + (w / (TW / 8)) * 8;
                if (x0 <= wx0 + 7 && x1 >= wx0 && y0 <= wy0 + 7 && y1 >= wy0)
                    L.r.wlist[w][atomicAdd(&L.wcnt[w], 1)] = (uint16_t)j;
            }
        }
        __syncthreads();
        // the order of a wave's list varies with the atomics; min and max do not
        const int nw = __builtin_amdgcn_readfirstlane(L.wcnt[wave]);
        // kBatch boxes at a time, their LDS reads (list, then box) in flight
        // together; past the end the last one again, which changes nothing
        // (12 submaps, 4 views: with the mask below 3028 -> 2954 us)
        constexpr int kBatch = 4;
        for (int i = 0; i < nw; i += kBatch) {
            uint4 bb[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) bb[k] = L.r.box[L.r.wlist[wave][i + k < nw ? i + k : nw - 1]];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const uint4 b = bb[k];
                const int x0 = (int16_t)(b.x & 0xffffu), y0 = (int16_t)(b.x >> 16);
                const int x1 = (int16_t)(b.y & 0xffffu), y1 = (int16_t)(b.y >> 16);
                if (px >= x0 && px <= x1 && py >= y0 && py <= y1) {
                    const float zl = __uint_as_float(b.z), zh = __uint_as_float(b.w);
                    zmin = zl < zmin ? zl : zmin;
                    zmax = zh > zmax ? zh : zmax;
                }
            }
        }
        if ((threadIdx.x & 63) == 0) L.wcnt[wave] = 0;
    }
    // after the last chunk's barriers (without records, as this thread left them)
    const float slo = __uint_as_float(L.r.zlo[at]), shi = __uint_as_float(L.r.zhi[at]);
    zmin = slo < zmin ? slo : zmin;
    if (shi > 0.0f) zmax = shi > zmax ? shi : zmax;
    // one atomic a wave: those of a wave's lanes on one word wait for each other
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)mask, d), hi = __shfl_xor((uint32_t)(mask >> 32), d);
        mask |= (unsigned long long)lo | ((unsigned long long)hi << 32);
    }
    if ((threadIdx.x & 63) == 0 && mask) atomicOr(&L.mask, mask);
    __syncthreads();   // the boxes are read: their bytes become the table
}

// The tile's block table and its submaps' data, after m_pixel_range (every
// thread of the workgroup calls it).
template <int NT, int TW, int TH>
__device__ __forceinline__ void m_table(const MSub *subs, const MTiles &t, uint32_t g, int tx0, int ty0, const Cam &c,
                                        float voxel, MTileLds<NT> &L)
{
    constexpr int TT = MTileLds<NT>::TT;
    uint32_t o0;
    const int n = m_bin_range(t, g, o0);
    for (int k = threadIdx.x; k < TT; k += NT) L.slot[k] = 0ull;
    uint32_t cut = kZBuckets;
    if (n > TT / 2) {
        // More records than the table holds: those nearest the camera go in.
        // A histogram of the grown cubes' least depths (in the table's first
        // slots, cleared again below) gives the largest bucket prefix that
        // fits; a read at a point shallower than the first left-out bucket
        // cannot touch a left-out block (it lies in that block's grown cube).
        __syncthreads();
        uint32_t *hist = reinterpret_cast<uint32_t *>(L.slot);
        for (int j = (int)threadIdx.x; j < n; j += NT)
            atomicAdd(&hist[zbucket((uint32_t)t.bins[o0 + (uint32_t)j].pad2)], 1u);
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t acc = 0u, c = 0u;
            while (c < kZBuckets && acc + hist[c] <= (uint32_t)(TT / 2)) acc += hist[c++];
            L.cut = c;
        }
        __syncthreads();
        cut = L.cut;
        for (int k = threadIdx.x; k < kZBuckets; k += NT) hist[k] = 0u;
    }
    if (threadIdx.x == 0) L.dlim = __float_as_uint(cut >= kZBuckets ? __builtin_inff() : zbucket_floor(cut));
    // the tile's submaps, ascending, each with its table window: centred 120
    // blocks out on the tile's central ray, so that it holds everything from the
    // camera to twice that whatever the submap's rotation
    if (threadIdx.x < (unsigned)kMaxSubmaps) {
        const unsigned long long m = L.mask;
        const int sm = (int)threadIdx.x;
        if ((m >> sm) & 1ull) {
            const int k = __popcll(m & ((1ull << sm) - 1ull));
            const MSub &S = subs[sm];
            for (int q = 0; q < 9; ++q) L.Rs[k][q] = S.R[q];
            for (int q = 0; q < 3; ++q) L.Rs[k][9 + q] = S.s[q];
            L.ent[k] = S.entries;
            L.occ[k] = S.occ;
            L.vox[k] = S.voxels;
            L.nb[k] = S.n_buckets;
            L.ne[k] = S.n_excess;
            L.smid[k] = sm;
            const float a = ((float)(tx0 + TW / 2) - c.cx) / c.fx, b = ((float)(ty0 + TH / 2) - c.cy) / c.fy;
            const float far = 960.0f / sqrtf((a * a + b * b) + 1.0f), inv_vs = 1.0f / voxel;
            float P[3];
            for (int q = 0; q < 3; ++q)
                P[q] = c.ti[q] * inv_vs + far * ((c.Ri[3 * q] * a + c.Ri[3 * q + 1] * b) + c.Ri[3 * q + 2]);
            for (int q = 0; q < 3; ++q)
                L.org[k][q] =
                    block_of(((S.R[3 * q] * P[0] + S.R[3 * q + 1] * P[1]) + S.R[3 * q + 2] * P[2]) + S.s[q]) - 127;
        }
    }
    __syncthreads();
    for (int j = (int)threadIdx.x; j < n; j += NT) {
        const Rec r = t.bins[o0 + (uint32_t)j];
        if (zbucket((uint32_t)r.pad2) >= cut) continue;    // left out: deeper than the table's depth limit
        const int k = __popcll(L.mask & ((1ull << (uint32_t)r.pad) - 1ull));
        uint32_t key;
        const bool fits = m_key(L, k, r.bx, r.by, r.bz, key) && (key & 0xffu) && (key & 0xff00u) && (key & 0xff0000u);
        if (fits && atomicAdd(&L.n_tab, 1u) < (uint32_t)(TT / 2)) {
            // keys in one bin are distinct; the table is at most half full
            const unsigned long long val = ((unsigned long long)key << 32) | (uint32_t)r.ptr;
            uint32_t sl = m_slot<NT>(key * kHashMul);
            for (int q = 0; q < TT; ++q) {
                if (atomicCAS(&L.slot[sl], 0ull, val) == 0ull) break;
                sl = (sl + 1u) & (uint32_t)(TT - 1);
            }
        } else {
            // left out: reads at points shallower than its grown cube cannot touch it
            atomicMin(&L.dlim, (uint32_t)r.pad2);
        }
    }
    __syncthreads();
}

// Device pointer of block (bx, by, bz) of the k-th submap of the tile (-1 =
// absent) from the submap's bucket bitmap and hash table, in two halves, so that
// lookups can be in flight together: the bucket's occupancy bit and its entry,
// loaded at once; then the answer, along the chain beyond the bucket only when
// the entry is another block's.
struct MProbe {
    uint32_t h, ow;
    int4 w;
};

template <int NT>
__device__ __forceinline__ MProbe m_map_probe(const MTileLds<NT> &L, int k, int bx, int by, int bz)
{
    MProbe q;
    q.h = hash_index(bx, by, bz, L.nb[k] - 1u);
    q.ow = gload(L.occ[k] + (q.h >> 5));
    q.w = load_entry(L.ent[k], q.h);
    return q;
}

template <int NT>
__device__ __forceinline__ int m_map_resolve(const MTileLds<NT> &L, int k, const MProbe &q, int bx, int by, int bz)
{
    const int4 w = q.w;
    if (!((q.ow >> (q.h & 31u)) & 1u)) return -1;
    const uint32_t kxy = (uint32_t)(uint16_t)bx | ((uint32_t)(uint16_t)by << 16);
    if ((uint32_t)w.x == kxy && (int16_t)(w.y & 0xffff) == (int16_t)bz && w.w >= 0) return w.w;
    if (w.z < 1 || (uint32_t)(w.z - 1) >= L.ne[k]) return -1;
    int ptr = -1;
    const int e = find_entry_from(L.ent[k], L.nb[k], L.ne[k], L.nb[k] + (uint32_t)(w.z - 1), bx, by, bz, 0, &ptr);
    return e >= 0 ? ptr : -1;
}

// the LDS table's answer for a key with its hash: the pointer, or -1
template <int NT>
__device__ __forceinline__ int m_table_find(const MTileLds<NT> &L, uint32_t key, uint32_t hash)
{
    constexpr int TT = MTileLds<NT>::TT;
    uint32_t sl = m_slot<NT>(hash);
    for (int it = 0; it < TT; ++it) {
        const unsigned long long kk = L.slot[sl];
        if ((uint32_t)(kk >> 32) == key) return (int)(uint32_t)kk;
        if (kk == 0ull) break;
        sl = (sl + 1u) & (uint32_t)(TT - 1);
    }
    return -1;
}

// Device pointer of block (bx, by, bz) of the k-th submap: the LDS table
// first; unless `local`, then the submap's own table.  `local` holds when the
// read belongs to a ray point at or beyond the near plane and shallower than
// every block left out of the LDS table: every block within 3 voxels of such
// a point is in the bin (blocks are binned by their cube grown by 3 voxels),
// so a miss proves absence.
template <int NT>
__device__ __forceinline__ int m_lookup(const MTileLds<NT> &L, int k, int bx, int by, int bz, bool local)
{
    uint32_t key;
    int p = -1;
    if (m_key(L, k, bx, by, bz, key)) p = m_table_find(L, key, key * kHashMul);
    if (p >= 0 || local || !in_short_range(bx) || !in_short_range(by) || !in_short_range(bz)) return p;
    return m_map_resolve(L, k, m_map_probe(L, k, bx, by, bz), bx, by, bz);
}

template <int NT>
__device__ __forceinline__ void to_sub(const MTileLds<NT> &L, int k, float P0, float P1, float P2, float &Q0,
                                       float &Q1, float &Q2)
{
    const float *R = L.Rs[k];
    Q0 = ((R[0] * P0 + R[1] * P1) + R[2] * P2) + R[9];
    Q1 = ((R[3] * P0 + R[4] * P1) + R[5] * P2) + R[10];
    Q2 = ((R[6] * P0 + R[7] * P1) + R[8] * P2) + R[11];
}

// the tile's submaps that can be allocated at, or weigh in the field at,
// world voxel-unit point P: the mask of P's world cell within the tile's set
template <int NT>
__device__ __forceinline__ unsigned long long m_cell_mask(const MTiles &t, const MTileLds<NT> &L, float P0, float P1,
                                                          float P2)
{
    return gload(t.wmask + wcell_index(block_of(P0), block_of(P1), block_of(P2))) & L.mask;
}

// Turns through the submaps of the lanes' masks cm, in ascending order in every
// lane.  Usually the wave takes the tile's submaps one by one (k the same in
// every lane; a lane takes part in those of its mask): neighbouring rays read
// the same ones.  LANES: each lane takes those of its own mask, as where the
// tile's table is incomplete.  Such a tile spans much of the map: its lanes need
// different submaps, and wait for reads of those submaps' tables at the same
// time (12 submaps 12 m away, 64x48: 1500 us one by one, 1100 so).  Both in one
// kernel and the range's two ways cost four 320x240 views from within the map,
// with no such tile, 2985 -> 3030 us.
template <int NT, bool LANES, typename F>
__device__ __forceinline__ void m_each_submap(const MTileLds<NT> &L, unsigned long long tile, unsigned long long cm, F f)
{
    if (LANES) {
        for (; cm; cm &= cm - 1ull)
            if (!f(__popcll(tile & ((cm & -cm) - 1ull)))) break;
    } else {
        const int nsub = __popcll(tile);
        bool on = true;
        for (int k = 0; k < nsub; ++k) {
            const int sm = __builtin_amdgcn_readfirstlane(L.smid[k]);
            if (on && ((cm >> (uint32_t)sm) & 1ull)) on = f(k);
        }
    }
}

// "allocated" of the combined map: some submap has a device block at
// floor(P_i X); only the submaps of P's cell mask cm can.  `tile`: the tile's
// submaps.
template <int NT, bool LANES>
__device__ __forceinline__ bool m_allocated(const MTileLds<NT> &L, unsigned long long tile, unsigned long long cm,
                                            float P0, float P1, float P2, bool local)
{
    bool found = false;
    m_each_submap<NT, LANES>(L, tile, cm, [&](int k) {
        float Q0, Q1, Q2;
        to_sub(L, k, P0, P1, P2, Q0, Q1, Q2);
        found = m_lookup(L, k, block_of(Q0), block_of(Q1), block_of(Q2), local) >= 0;
        return !found;
    });
    return found;
}

// One submap's term of the combined field at P: its trilinear weight (absent
// voxels weigh 0, the same lerp order as the SDF) and, when positive, its F.
// Corners c and c + 4 are one voxel apart along z, next to each other in
// memory unless the cell crosses its block's upper z face: SDF and weights are
// read as pairs.
template <int NT, bool LANES>
__device__ __forceinline__ void m_term(const MTileLds<NT> &L, int k, float P0, float P1, float P2, bool local, int &cnt,
                                       float &first, float &num, float &den)
{
    float Q0, Q1, Q2;
    to_sub(L, k, P0, P1, P2, Q0, Q1, Q2);
    const float fbx = floorf(Q0), fby = floorf(Q1), fbz = floorf(Q2);
    const float tx = Q0 - fbx, ty = Q1 - fby, tz = Q2 - fbz;
    const int ix = (int)fbx, iy = (int)fby, iz = (int)fbz;
    const int Bx = ix >> 3, By = iy >> 3, Bz = iz >> 3;
    const bool sx = (ix & 7) == 7, sy = (iy & 7) == 7, sz = (iz & 7) == 7;
    const int need = (sx ? 1 : 0) | (sy ? 2 : 0) | (sz ? 4 : 0);
    uint32_t key;
    const bool in = m_key(L, k, Bx, By, Bz, key);
    const uint32_t hash = key * kHashMul;
    // first probes of the block and, for a cell that crosses a face, its seven
    // neighbours; `open`: those still to look up (slot of another block, or a
    // miss that proves nothing)
    int p[8];
    uint32_t open = 0u;
    {
        const unsigned long long kk = in ? L.slot[m_slot<NT>(hash)] : 0ull;
        const uint32_t hi = (uint32_t)(kk >> 32);
        p[0] = hi == key ? (int)(uint32_t)kk : -1;
        open |= (hi != key && (hi != 0u || !local)) ? 1u : 0u;
    }
#pragma unroll
    for (int n = 1; n < 8; ++n) p[n] = -1;
    if (need) {
        unsigned long long kk[8];
#pragma unroll
        for (int n = 1; n < 8; ++n) kk[n] = in ? L.slot[m_slot<NT>(hash + m_neighbour(n) * kHashMul)] : 0ull;
#pragma unroll
        for (int n = 1; n < 8; ++n) {
            const uint32_t hi = (uint32_t)(kk[n] >> 32), kn = key + m_neighbour(n);
            p[n] = hi == kn ? (int)(uint32_t)kk[n] : -1;
            if ((n & need) == n) open |= (hi != kn && (hi != 0u || !local)) ? 1u << n : 0u;
        }
    }
    while (!LANES && open) {
        const int n = __ffs((int)open) - 1;
        open &= open - 1u;
        const int q = m_lookup(L, k, Bx + (n & 1), By + ((n >> 1) & 1), Bz + (n >> 2), local);
#pragma unroll
        for (int m = 0; m < 8; ++m) p[m] = m == n ? q : p[m];
    }
    while (LANES && open) {   // two at a time, their map reads in flight together
        int n[2], q[2];
        MProbe mp[2];
        bool ask[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n[c] = open ? __ffs((int)open) - 1 : -1;
            open &= open - 1u;
            const int bx = Bx + (n[c] & 1), by = By + ((n[c] >> 1) & 1), bz = Bz + (n[c] >> 2);
            q[c] = -1;
            ask[c] = false;
            uint32_t kn;
            if (n[c] >= 0) {
                if (m_key(L, k, bx, by, bz, kn)) q[c] = m_table_find(L, kn, kn * kHashMul);
                ask[c] = q[c] < 0 && !local && in_short_range(bx) && in_short_range(by) && in_short_range(bz);
            }
            if (ask[c]) mp[c] = m_map_probe(L, k, bx, by, bz);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (ask[c]) q[c] = m_map_resolve(L, k, mp[c], Bx + (n[c] & 1), By + ((n[c] >> 1) & 1), Bz + (n[c] >> 2));
#pragma unroll
            for (int m = 0; m < 8; ++m) p[m] = m == n[c] ? q[c] : p[m];
        }
    }
    // corner blocks, lower then upper z
    const int lo[4] = {p[0], sx ? p[1] : p[0], sy ? p[2] : p[0], sx ? (sy ? p[3] : p[1]) : (sy ? p[2] : p[0])};
    const int up[4] = {sz ? p[4] : lo[0], sz ? (sx ? p[5] : p[4]) : lo[1], sz ? (sy ? p[6] : p[4]) : lo[2],
                       sz ? (sx ? (sy ? p[7] : p[5]) : (sy ? p[6] : p[4])) : lo[3]};
    int j[4];
    j[0] = (iz & 7) + 8 * (iy & 7) + 64 * (ix & 7);
    const int dx = sx ? -448 : 64, dy = sy ? -56 : 8;
    j[1] = j[0] + dx;
    j[2] = j[0] + dy;
    j[3] = j[1] + dy;
    const uint8_t *vox = L.vox[k];
    uint32_t sp[4], wp[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint8_t *blk = vox + (size_t)(uint32_t)(lo[c] >= 0 ? lo[c] : 0) * kBlockBytes;
        sp[c] = gload_pair(blk + 2 * j[c]);
        // voxel 7's weight with the one below it (the pair above would end past the block)
        wp[c] = gload_byte_pair(blk + 1024 + (sz ? j[c] - 1 : j[c]));
    }
    int16_t s[8];
    uint32_t w8[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        s[c] = (int16_t)(sp[c] & 0xffffu);
        s[c + 4] = (int16_t)(sp[c] >> 16);
        w8[c] = sz ? wp[c] >> 8 : wp[c] & 0xffu;
        w8[c + 4] = wp[c] >> 8;
    }
    if (sz) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint8_t *blk = vox + (size_t)(uint32_t)(up[c] >= 0 ? up[c] : 0) * kBlockBytes;
            s[c + 4] = gload(reinterpret_cast<const int16_t *>(blk) + (j[c] - 7));
            w8[c + 4] = gload(blk + 1024 + (j[c] - 7));
        }
    }
    float wf[8];
    uint32_t present = 0u;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const bool there = (c < 4 ? lo[c & 3] : up[c & 3]) >= 0;
        wf[c] = there ? (float)w8[c] : 0.0f;
        present |= (there ? 1u : 0u) << c;
    }
    const float w = lerp8(wf, tx, ty, tz);
    if (!(w > 0.0f)) return;
    const float F = cell_lerp(present, s, tx, ty, tz);
    if (cnt == 0) first = F;
    num = num + w * F;
    den = den + w;
    ++cnt;
}

// combined field at world voxel-unit P over the submaps of P's cell mask cm
// (every submap with positive weight at P is one of them), in ascending
// submap order
template <int NT, bool LANES>
__device__ __forceinline__ float m_field(const MTileLds<NT> &L, unsigned long long tile, unsigned long long cm, float P0,
                                         float P1, float P2, bool local)
{
    int cnt = 0;
    float first = 1.0f, num = 0.0f, den = 0.0f;
    m_each_submap<NT, LANES>(L, tile, cm, [&](int k) {
        m_term<NT, LANES>(L, k, P0, P1, P2, local, cnt, first, num, den);
        return true;
    });
    if (cnt == 0) return 1.0f;
    if (cnt == 1) return first;
    return num / den;
}

// M_REFINE: past the surface, the first refinement step taken; M_TAP: at the
// hit, reading the normal's six taps
enum { M_COARSE, M_FINE, M_SURFACE, M_WRONG_SIDE, M_REFINE, M_TAP };

// the view of flat tile index g (views are few; their tile ranges ascend)
__device__ __forceinline__ int view_of(const MFrame *f, int g)
{
    int vi = 0;
    while (vi + 1 < f->n_views && g >= f->view[vi + 1].tile_base) ++vi;
    return vi;
}

}  // namespace

// one workgroup per TW x TH tile of any view; waves cover 8x8 pixel squares
template <int TW, int TH>
__global__ __launch_bounds__(TW *TH) void k_m_raycast(const MSub *subs, const MFrame *f, MTiles t, float voxel,
                                                      float mu)
{
    constexpr int NT = TW * TH;
    __shared__ MTileLds<NT> L;
    const int g = (int)blockIdx.x;
    const int vi = view_of(f, g);
    const MView &V = f->view[vi];
    const int tile = g - V.tile_base;
    const int W = V.cam.W, H = V.cam.H;
    const int q = (int)threadIdx.x >> 6, i = (int)threadIdx.x & 63;
    const int tx0 = (tile % V.ntx) * TW, ty0 = (tile / V.ntx) * TH;
    const int lx = (q % (TW / 8)) * 8 + (i & 7), ly = (q / (TW / 8)) * 8 + (i >> 3);
    const int px = tx0 + lx, py = ty0 + ly;
    float zmin, zmax;
    m_pixel_range<NT, TW, TH>(t, (uint32_t)g, tx0, ty0, px, py, L, zmin, zmax);
    m_table<NT, TW, TH>(subs, t, (uint32_t)g, tx0, ty0, V.cam, voxel, L);
    const unsigned long long tile_mask = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)L.mask) |
                                         ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(L.mask >> 32)) << 32);
    // reads at points shallower than dcut (the table's depth limit less a
    // voxel for the normal's taps and a millimetre for rounding) can trust a
    // table miss
    const float dcut = __uint_as_float(L.dlim) - voxel - 1e-3f;
    const bool inside = px < W && py < H;
    float4 out_p = make_float4(0.f, 0.f, 0.f, 0.f), out_n = make_float4(0.f, 0.f, 0.f, 0.f);
    if (inside && zmin <= zmax) {
        const Cam &c = V.cam;
        const float inv_vs = 1.0f / voxel;
        const float mu_v = mu * inv_vs;
        const float ox = c.ti[0] * inv_vs, oy = c.ti[1] * inv_vs, oz = c.ti[2] * inv_vs;
        const float a = ((float)px - c.cx) / c.fx;
        const float b = ((float)py - c.cy) / c.fy;
        const float nr = sqrtf((a * a + b * b) + 1.0f);
        const float rcx = a / nr, rcy = b / nr, rcz = 1.0f / nr;
        const float zscale = voxel * rcz;   // camera z of ray parameter t (voxel units)
        const float dx = (c.Ri[0] * rcx + c.Ri[1] * rcy) + c.Ri[2] * rcz;
        const float dy = (c.Ri[3] * rcx + c.Ri[4] * rcy) + c.Ri[5] * rcz;
        const float dz = (c.Ri[6] * rcx + c.Ri[7] * rcy) + c.Ri[8] * rcz;
        float tt = (zmin * nr) * inv_vs;
        const float t_end = (zmax * nr) * inv_vs;
        int state = M_COARSE;
        int steps = 0, tap = 0;
        float plus = 0.0f, gx = 0.0f, gy = 0.0f, gz = 0.0f;
        // one loop for the march, the refinement and the normal's taps: the
        // field's code stands once (three copies and their lookups were 100 KB,
        // more than the instruction cache), and lanes at a hit read their taps
        // beside lanes that still march
        auto march = [&](auto lanes) {
            constexpr bool kLanes = decltype(lanes)::value;
            for (;;) {
                const bool marching = state < M_REFINE;
                if (marching && !(tt < t_end && steps < kMaxRaySteps)) break;
                if (state == M_COARSE || state == M_FINE) {
                    // Empty-space skip: while no block is found the march keeps
                    // its fixed step; the world cells of the next kSkip positions
                    // are tested together, a clear cell proves the position
                    // unallocated, so the iterations skipped are those the loop
                    // would run.
                    const float stp = state == M_COARSE ? 8.0f : mu_v;
                    constexpr int kSkip = 4;
                    float tk[kSkip];
                    unsigned long long wk[kSkip];
                    float t2 = tt;
#pragma unroll
                    for (int k = 0; k < kSkip; ++k) {
                        tk[k] = t2;
                        wk[k] = m_cell_mask<NT>(t, L, ox + t2 * dx, oy + t2 * dy, oz + t2 * dz);
                        t2 += stp;
                    }
                    bool stop = false;
#pragma unroll
                    for (int k = 0; k < kSkip; ++k) {
                        if (stop) continue;
                        tt = tk[k];
                        if (!(tt < t_end && steps < kMaxRaySteps) || wk[k]) {
                            stop = true;
                            continue;
                        }
                        ++steps;   // an iteration on unallocated space
                    }
                    if (!stop) tt = t2;
                    if (!(tt < t_end && steps < kMaxRaySteps)) break;
                }
                if (marching) ++steps;
                float P0 = ox + tt * dx, P1 = oy + tt * dy, P2 = oz + tt * dz;
                // the taps P +- e_a lie within a voxel of the hit, which dcut covers
                const bool local = tt * zscale >= kZNear && tt * zscale < dcut;
                if (state == M_TAP) {
                    const float e = (tap & 1) ? -1.0f : 1.0f;
                    P0 = (tap >> 1) == 0 ? P0 + e : P0;
                    P1 = (tap >> 1) == 1 ? P1 + e : P1;
                    P2 = (tap >> 1) == 2 ? P2 + e : P2;
                }
                // only the submaps of P's world cell can be allocated there
                const unsigned long long cm = m_cell_mask<NT>(t, L, P0, P1, P2);
                if (marching) {
                    const bool alloc = cm && m_allocated<NT, kLanes>(L, tile_mask, cm, P0, P1, P2, local);
                    if (!alloc) {
                        tt += state == M_COARSE ? 8.0f : mu_v;
                        state = state == M_COARSE ? M_COARSE : M_FINE;
                        continue;
                    }
                    if (state == M_COARSE) {
                        tt -= 8.0f;
                        state = M_FINE;
                        continue;
                    }
                }
                const float F = m_field<NT, kLanes>(L, tile_mask, cm, P0, P1, P2, local);
                if (state == M_TAP) {
                    if (tap & 1) {
                        const float d = (plus - F) * 0.5f;
                        gx = tap == 1 ? d : gx;
                        gy = tap == 3 ? d : gy;
                        gz = tap == 5 ? d : gz;
                        if (tap == 5) break;
                    } else {
                        plus = F;
                    }
                    ++tap;
                } else if (state == M_REFINE) {
                    tt += F * mu_v;
                    state = M_TAP;
                } else if (state == M_SURFACE) {
                    if (F < 0.0f) {
                        state = M_REFINE;
                        tt += F * mu_v;
                    } else {
                        const float s = F * mu_v;
                        tt += (s > 1.0f) ? s : 1.0f;
                    }
                } else if (F < 0.0f) {
                    if (state == M_FINE) {
                        state = M_WRONG_SIDE;
                    } else {
                        const float s = -F * mu_v;
                        tt += (s > 1.0f) ? s : 1.0f;
                    }
                } else {
                    // FINE or WRONG_SIDE meeting F >= 0 turns to SURFACE without
                    // a step; the SURFACE iteration that follows (if the step
                    // bound allows it) reads the same field at the same t, so
                    // its step is taken here with this F
                    state = M_SURFACE;
                    if (steps < kMaxRaySteps) {
                        ++steps;
                        const float s = F * mu_v;
                        tt += (s > 1.0f) ? s : 1.0f;
                    }
                }
            }
        };
        if (__builtin_amdgcn_readfirstlane((int)L.dlim) == 0x7f800000)   // nothing left out of the table
            march(std::false_type{});
        else
            march(std::true_type{});
        if (state == M_TAP) {
            const float P0 = ox + tt * dx, P1 = oy + tt * dy, P2 = oz + tt * dz;
            out_p = make_float4(P0 * voxel, P1 * voxel, P2 * voxel, 1.0f);
            const float gn = sqrtf((gx * gx + gy * gy) + gz * gz);
            if (gn > 0.0f) out_n = make_float4(gx / gn, gy / gn, gz / gn, 1.0f);
        }
    }
    if (inside) {
        const size_t p = (size_t)py * W + px;
        V.pts[p] = out_p;
        V.nrm[p] = out_n;
        if (out_p.w == 1.0f) atomicAdd(&L.hits, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && L.hits) t.acc_hits[g] += L.hits;
}

// search range of one view written as an image (parity of the range)
template <int TW, int TH>
__global__ __launch_bounds__(TW *TH) void k_m_range_write(const MSub *subs, const MFrame *f, MTiles t, int vi,
                                                          float *zmin_out, float *zmax_out)
{
    constexpr int NT = TW * TH;
    __shared__ MTileLds<NT> L;
    const MView &V = f->view[vi];
    const int g = V.tile_base + (int)blockIdx.x;
    const int tile = (int)blockIdx.x;
    const int q = (int)threadIdx.x >> 6, i = (int)threadIdx.x & 63;
    const int tx0 = (tile % V.ntx) * TW, ty0 = (tile / V.ntx) * TH;
    const int lx = (q % (TW / 8)) * 8 + (i & 7), ly = (q / (TW / 8)) * 8 + (i >> 3);
    const int px = tx0 + lx, py = ty0 + ly;
    float zmin, zmax;
    m_pixel_range<NT, TW, TH>(t, (uint32_t)g, tx0, ty0, px, py, L, zmin, zmax);
    if (px >= V.cam.W || py >= V.cam.H) return;
    zmin_out[(size_t)py * V.cam.W + px] = zmin;
    zmax_out[(size_t)py * V.cam.W + px] = zmax;
}

// ============================================================================
// launchers
// ============================================================================
hipError_t launch_m_alloc(const Vol *vols, const MSub *subs, const MFrame *f, unsigned long long *wmask, int w, int h,
                          hipStream_t s)
{
    const int npix = w * h;
    hipLaunchKernelGGL(k_m_alloc, dim3((npix + 255) / 256 + kKeepGroups, kMaxSel), dim3(256), 0, s, vols, f);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_m_insert, dim3(128, kMaxSel), dim3(256), 0, s, vols, f);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_m_mark, dim3(64, kMaxSel), dim3(256), 0, s, vols, subs, f, wmask);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_m_visible, dim3(256, kMaxSel), dim3(256), 0, s, vols, f);
    return hipGetLastError();
}

hipError_t launch_m_integrate(const Vol *vols, const MFrame *f, int nt, int grid, bool dry, hipStream_t s)
{
    if (grid < 1) grid = 1;
    if (grid > kIntegrateGrid) grid = kIntegrateGrid;
    const dim3 g(grid, kMaxSel);
    switch (nt) {
    case 64: hipLaunchKernelGGL(k_m_integrate<64>, g, dim3(64), 0, s, vols, f, dry ? 1 : 0); break;
    case 128: hipLaunchKernelGGL(k_m_integrate<128>, g, dim3(128), 0, s, vols, f, dry ? 1 : 0); break;
    case 512: hipLaunchKernelGGL(k_m_integrate<512>, g, dim3(512), 0, s, vols, f, dry ? 1 : 0); break;
    default: hipLaunchKernelGGL(k_m_integrate<256>, g, dim3(256), 0, s, vols, f, dry ? 1 : 0); break;
    }
    return hipGetLastError();
}

hipError_t launch_m_bin(const MSub *subs, const MFrame *f, const MTiles &t, int n_views, int grid, float voxel,
                        hipStream_t s)
{
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(k_m_bin<false>, dim3(grid, n_views), dim3(256), 0, s, subs, f, t, voxel);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_m_scan, dim3(1), dim3(1024), 0, s, t);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_m_bin<true>, dim3(grid, n_views), dim3(256), 0, s, subs, f, t, voxel);
    return hipGetLastError();
}

hipError_t launch_m_raycast(const MSub *subs, const MFrame *f, const MTiles &t, float voxel, float mu, int tw, int th,
                            hipStream_t s)
{
    const dim3 g(t.n_tiles);
    if (tw == 32 && th == 8)
        hipLaunchKernelGGL((k_m_raycast<32, 8>), g, dim3(256), 0, s, subs, f, t, voxel, mu);
    else if (tw == 8 && th == 8)
        hipLaunchKernelGGL((k_m_raycast<8, 8>), g, dim3(64), 0, s, subs, f, t, voxel, mu);
    else if (tw == 16 && th == 8)
        hipLaunchKernelGGL((k_m_raycast<16, 8>), g, dim3(128), 0, s, subs, f, t, voxel, mu);
    else if (tw == 16 && th == 16)
        hipLaunchKernelGGL((k_m_raycast<16, 16>), g, dim3(256), 0, s, subs, f, t, voxel, mu);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_m_range_write(const MSub *subs, const MFrame *f, const MTiles &t, int vi, int n_tiles_view,
                                float *zmin, float *zmax, int tw, int th, hipStream_t s)
{
    const dim3 g(n_tiles_view);
    if (tw == 32 && th == 8)
        hipLaunchKernelGGL((k_m_range_write<32, 8>), g, dim3(256), 0, s, subs, f, t, vi, zmin, zmax);
    else if (tw == 8 && th == 8)
        hipLaunchKernelGGL((k_m_range_write<8, 8>), g, dim3(64), 0, s, subs, f, t, vi, zmin, zmax);
    else if (tw == 16 && th == 8)
        hipLaunchKernelGGL((k_m_range_write<16, 8>), g, dim3(128), 0, s, subs, f, t, vi, zmin, zmax);
    else if (tw == 16 && th == 16)
        hipLaunchKernelGGL((k_m_range_write<16, 16>), g, dim3(256), 0, s, subs, f, t, vi, zmin, zmax);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_m_clear(const MTiles &t, hipStream_t s)
{
    hipLaunchKernelGGL(k_m_clear, dim3(2048), dim3(256), 0, s, t);
    return hipGetLastError();
}

}  // namespace tsdf

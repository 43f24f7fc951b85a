// tsdf_mesh.hip -- marching-cubes meshing of the volume (Sec. 4, meshing
// engine) on gfx950.
//
// k_mesh<false> walks the hash entries in chunks of 64, one wave per chunk at
// a time: the allocated entries are found with one ballot, the wave stages
// each such block and its +x/+y/+z halo in LDS, lane (x, y) classifies the 8
// cells of its z column, and the chunk's triangle count is written.
// k_mesh_scan (and k_mesh_groups over many chunks) turns the counts into
// offsets in a fixed order.  k_mesh<true> repeats the walk: a block's
// triangles occupy a contiguous range (chunk offset + earlier blocks), each
// lane's at a wave prefix over the lanes.  The output order is fixed and two
// calls give the same arrays.
//
// The case table is derived at compile time from the cube's faces (constexpr),
// not tabulated: the rule of each face pairs its active edges into segments,
// the segments close into loops, each loop is oriented from the inside corners
// towards the outside ones and fanned from its smallest edge.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsdf_ctx.h"
#include "tsdf_device.h"
#include "tsdf_mesh.h"

namespace {

using namespace tsdf;

struct McTable {
    int8_t e0[12], e1[12], axis[12];   // edge endpoints (corner indices) and axis
    int8_t ntri[256];
    int8_t tri[256][15];               // edge triples, ntri of them
};

constexpr McTable make_mc_table()
{
    McTable T{};
    int ne = 0;
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 8; ++c)
            if (!((c >> a) & 1)) {
                T.e0[ne] = (int8_t)c;
                T.e1[ne] = (int8_t)(c | (1 << a));
                T.axis[ne] = (int8_t)a;
                ++ne;
            }
    // the 6 faces: 4 corners and 4 edges each
    int fc[6][4] = {}, fe[6][4] = {};
    int f = 0;
    for (int a = 0; a < 3; ++a)
        for (int s = 0; s < 2; ++s, ++f) {
            int k = 0;
            for (int c = 0; c < 8; ++c)
                if (((c >> a) & 1) == s) fc[f][k++] = c;
            k = 0;
            for (int e = 0; e < 12; ++e)
                if (T.axis[e] != a && ((T.e0[e] >> a) & 1) == s && ((T.e1[e] >> a) & 1) == s) fe[f][k++] = e;
        }
    for (int m = 0; m < 256; ++m) {
        bool in[8] = {}, act[12] = {};
        for (int c = 0; c < 8; ++c) in[c] = (m >> c) & 1;
        for (int e = 0; e < 12; ++e) act[e] = in[T.e0[e]] != in[T.e1[e]];
        // segment graph: every active edge has exactly two neighbours
        int nb[12][2] = {}, deg[12] = {};
        for (int g = 0; g < 6; ++g) {
            int fa[4] = {}, n = 0;
            for (int k = 0; k < 4; ++k)
                if (act[fe[g][k]]) fa[n++] = fe[g][k];
            if (n == 2) {
                nb[fa[0]][deg[fa[0]]++] = fa[1];
                nb[fa[1]][deg[fa[1]]++] = fa[0];
            } else if (n == 4) {
                // ambiguous face: cut off each inside corner by its own segment
                for (int k = 0; k < 4; ++k) {
                    const int c = fc[g][k];
                    if (!in[c]) continue;
                    int inc[2] = {}, ni = 0;
                    for (int j = 0; j < 4; ++j)
                        if (T.e0[fa[j]] == c || T.e1[fa[j]] == c) inc[ni++] = fa[j];
                    nb[inc[0]][deg[inc[0]]++] = inc[1];
                    nb[inc[1]][deg[inc[1]]++] = inc[0];
                }
            }
        }
        bool seen[12] = {};
        int nt = 0;
        for (int s0 = 0; s0 < 12; ++s0) {
            if (!act[s0] || seen[s0]) continue;
            int loop[12] = {}, len = 0;
            int prev = -1, cur = s0;
            while (true) {
                loop[len++] = cur;
                seen[cur] = true;
                const int nx = nb[cur][0] != prev ? nb[cur][0] : nb[cur][1];
                prev = cur;
                cur = nx;
                if (cur == s0) break;
            }
            // orientation, in doubled integer coordinates: Newell normal of the
            // edge midpoints against the sum of inside -> outside edge directions
            int nvec[3] = {}, dvec[3] = {};
            for (int i = 0; i < len; ++i) {
                const int ea = loop[i], eb = loop[(i + 1) % len];
                int P[3] = {}, Q[3] = {};
                for (int d = 0; d < 3; ++d) {
                    P[d] = ((T.e0[ea] >> d) & 1) + ((T.e1[ea] >> d) & 1);
                    Q[d] = ((T.e0[eb] >> d) & 1) + ((T.e1[eb] >> d) & 1);
                }
                nvec[0] += P[1] * Q[2] - P[2] * Q[1];
                nvec[1] += P[2] * Q[0] - P[0] * Q[2];
                nvec[2] += P[0] * Q[1] - P[1] * Q[0];
                const int sg = in[T.e0[ea]] ? 1 : -1;      // from the inside corner to the outside one
                dvec[T.axis[ea]] += sg;
            }
            if (nvec[0] * dvec[0] + nvec[1] * dvec[1] + nvec[2] * dvec[2] < 0) {
                for (int i = 1, j = len - 1; i < j; ++i, --j) {
                    const int t = loop[i];
                    loop[i] = loop[j];
                    loop[j] = t;
                }
            }
            for (int i = 1; i + 1 < len; ++i) {
                T.tri[m][3 * nt + 0] = (int8_t)loop[0];
                T.tri[m][3 * nt + 1] = (int8_t)loop[i];
                T.tri[m][3 * nt + 2] = (int8_t)loop[i + 1];
                ++nt;
            }
        }
        T.ntri[m] = (int8_t)nt;
    }
    return T;
}

__constant__ McTable kMc = make_mc_table();

constexpr int kChunk = 64;            // hash entries per wave (one ballot)
constexpr int kWaves = 4;             // waves per workgroup, each on chunks of its own
constexpr int kGrid = 2048;           // persistent workgroups: 8 waves per SIMD on 256 CUs
constexpr int kCap = 256;             // triangles listed in LDS per write-out round
constexpr int kCols = 81;             // 9 x 9 voxel columns of a block and its +x/+y halo
constexpr int kColStride = 10;        // shorts per column (9 used): 5 dwords, so columns spread over the banks
constexpr uint32_t kScanGroup = 4096; // chunks per workgroup of the offset scan

struct MeshOut {
    float *verts;
    long long *keys;
    unsigned long long max_tri;
    uint32_t *chunk_off;              // per chunk: triangle count, then offset within its scan group
    unsigned long long *group;        // per scan group: total, then exclusive offset (unused with one group)
    unsigned long long *total;
    uint32_t chunks, groups;
};

struct Vert {
    float x, y, z;
};

// one wave's LDS
struct WaveLds {
    int16_t g[kCols * kColStride + 2];   // column y * 9 + x: SDF of z = 0..8
    uint32_t cb[kCols];                  // column y * 9 + x: bit z inside (SDF < 0), bit 16 + z unobserved
};

// order one wave's LDS accesses (its own tile: no other wave reads it)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One voxel column of block `ptr` (8 voxels from in-block index idx, a
// multiple of 8: one 16-byte and one 8-byte load) and the voxel above it
// (in-block index tidx of block `top`); an absent block is unobserved.
struct Column {
    uint4 s;
    uint2 w;
    int ts, tw;
};

__device__ __forceinline__ Column load_column(const uint8_t *voxels, int ptr, int idx, int top)
{
    Column c;
    c.s = make_uint4(0u, 0u, 0u, 0u);
    c.w = make_uint2(0u, 0u);
    c.ts = 0;
    c.tw = 0;
    if (ptr >= 0) {
        const uint8_t *blk = voxels + (size_t)ptr * kBlockBytes;
        c.s = *reinterpret_cast<const uint4 *>(blk + 2 * idx);
        c.w = *reinterpret_cast<const uint2 *>(blk + 1024 + idx);
    }
    if (top >= 0) {
        const uint8_t *blk = voxels + (size_t)top * kBlockBytes;
        c.ts = *reinterpret_cast<const int16_t *>(blk + 2 * idx);
        c.tw = blk[1024 + idx];
    }
    return c;
}

template <bool EMIT>
__device__ __forceinline__ void store_column(const Column &c, int col, WaveLds &L)
{
    const uint32_t s[4] = {c.s.x, c.s.y, c.s.z, c.s.w};
    const uint32_t w[2] = {c.w.x, c.w.y};
    uint32_t bits = (c.ts < 0 ? 1u << 8 : 0u) | (c.tw == 0 ? 1u << 24 : 0u);
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        bits |= ((s[z >> 1] >> (16 * (z & 1) + 15)) & 1u) << z;
        bits |= (((w[z >> 2] >> (8 * (z & 3))) & 0xffu) == 0u ? 1u : 0u) << (16 + z);
    }
    L.cb[col] = bits;
    if (EMIT) {
        uint32_t *g = reinterpret_cast<uint32_t *>(L.g + col * kColStride);
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k] = s[k];
        L.g[col * kColStride + 8] = (int16_t)c.ts;
    }
}

// Bound: memory (the blocks and their halo read, 60 bytes written per
// triangle).  A wave takes the live entries of a chunk one after another; the
// block and its halo are 81 voxel columns of 9, loaded by one 16-byte and one
// 8-byte access per column all in flight together, and kept in LDS as the SDF
// and one word of sign and observed bits per column, from which a lane forms
// the 8 cases of its cell column by bit operations.  EMIT lists the block's
// triangles in LDS (lane prefix order) and then gives every vertex a lane, so
// that the lanes stay full however the triangles sit in the block and
// consecutive lanes write consecutive 12-byte vertices and 8-byte keys.
// Before: triangles built by the lane that owns their cell column (mostly
// idle lanes, the case table and corners gathered from memory), one wave per
// workgroup with 18 KB of LDS: 941 us to emit and 76 us to count at 58 k
// blocks, 5.4 M triangles and 4.7 M entries; a whole call 1182 us before and
// 286 us with this split and the scan below.
template <bool EMIT>
__global__ __launch_bounds__(64 * kWaves) void k_mesh(Vol v, MeshOut o, float voxel)
{
    __shared__ WaveLds lds[kWaves];
    __shared__ uint32_t list[EMIT ? kWaves : 1][EMIT ? kCap : 1];   // cell | t << 9 | case << 12
    __shared__ int8_t ntri[256];
    __shared__ int8_t tri[EMIT ? 256 * 15 : 1];
    ntri[threadIdx.x] = kMc.ntri[threadIdx.x];
    if (EMIT)
        for (int i = (int)threadIdx.x; i < 256 * 15; i += 64 * kWaves) tri[i] = (&kMc.tri[0][0])[i];
    __syncthreads();
    const int lane = (int)lane_id();
    const int wv = (int)threadIdx.x >> 6;
    WaveLds &L = lds[wv];
    const int cx = lane & 7, cy = lane >> 3;          // the lane's cell column
    for (uint32_t chunk = blockIdx.x * kWaves + (uint32_t)wv; chunk < o.chunks; chunk += gridDim.x * kWaves) {
        unsigned long long base = 0ull;
        if (EMIT) {
            const uint32_t gr = chunk / kScanGroup;
            const unsigned long long g0 = o.groups > 1 ? o.group[gr] : 0ull;
            const unsigned long long g1 = gr + 1 < o.groups ? o.group[gr + 1] : *o.total;
            base = g0 + o.chunk_off[chunk];
            const bool last = chunk + 1 == o.chunks || (chunk + 1) % kScanGroup == 0u;
            if ((last ? g1 : g0 + o.chunk_off[chunk + 1]) == base) continue;   // no triangle
        }
        uint32_t count = 0;
        const uint32_t e = chunk * kChunk + (uint32_t)lane;
        int4 w = make_int4(0, 0, 0, -2);
        if (e < v.n_entries) w = load_entry(v.entries, e);
        unsigned long long live = __ballot(w.w >= 0);
        while (live) {
            const int src = __ffsll((long long)live) - 1;
            live &= live - 1;
            const int kxy = __shfl(w.x, src, 64), kz = __shfl(w.y, src, 64), ptr = __shfl(w.w, src, 64);
            const int bx = (int16_t)(kxy & 0xffff), by = (int16_t)((uint32_t)kxy >> 16), bz = (int16_t)(kz & 0xffff);
            // neighbour n = 1..7 at (n & 1, n >> 1 & 1, n >> 2 & 1); lane n looks it up, lane 0 keeps the block
            int np = lane == 0 ? ptr : -1;
            if (lane > 0 && lane < 8) {
                int p = -1;
                if (find_entry(v, bx + (lane & 1), by + ((lane >> 1) & 1), bz + (lane >> 2), 0, &p) >= 0) np = p;
            }
            // own column: x = lane >> 3, y = lane & 7 (in-block order z + 8 y + 64 x)
            const Column own = load_column(v.voxels, ptr, 8 * lane, __shfl(np, 4, 64));
            // halo columns, lanes 0..16: (8, y) of neighbours 1 and 5, (x, 8) of 2 and 6, (8, 8) of 3 and 7
            const int hn = lane < 8 ? 1 : (lane < 16 ? 2 : 3);
            const int hp = __shfl(np, hn, 64), ht = __shfl(np, hn + 4, 64);
            const int hi = lane < 8 ? 8 * lane : (lane < 16 ? 64 * (lane - 8) : 0);
            const int hcol = lane < 8 ? 9 * lane + 8 : (lane < 16 ? 72 + lane - 8 : 80);
            Column halo = {};
            if (lane < 17) halo = load_column(v.voxels, hp, hi, ht);
            wave_sync();                             // the previous block's reads are done
            store_column<EMIT>(own, (lane & 7) * 9 + (lane >> 3), L);
            if (lane < 17) store_column<EMIT>(halo, hcol, L);
            wave_sync();
            // the cell column's corners: columns A (x, y), B (x + 1, y), C (x, y + 1), D (x + 1, y + 1)
            const uint32_t A = L.cb[cy * 9 + cx], B = L.cb[cy * 9 + cx + 1], C = L.cb[cy * 9 + cx + 9],
                           D = L.cb[cy * 9 + cx + 10];
            const uint32_t any = A | B | C | D, all = A & B & C & D;
            const uint32_t un = any >> 16;
            // cells with every corner observed and corners on both sides
            uint32_t act = (any | (any >> 1)) & ~(all & (all >> 1)) & ~(un | (un >> 1)) & 0xffu;
            const auto cell_case = [&](int z) {
                const uint32_t a = (A >> z) & 3u, b = (B >> z) & 3u, c = (C >> z) & 3u, d = (D >> z) & 3u;
                return (a & 1u) | ((b & 1u) << 1) | ((c & 1u) << 2) | ((d & 1u) << 3) | ((a & 2u) << 3) |
                       ((b & 2u) << 4) | ((c & 2u) << 5) | ((d & 2u) << 6);
            };
            int n = 0;
            for (uint32_t k = act; k; k &= k - 1) n += ntri[cell_case(__ffs((int)k) - 1)];
            if (!EMIT) {
                count += (uint32_t)n;                // summed over lanes below
                continue;
            }
            // exclusive prefix of n over the lanes: the lane's first triangle in the block
            int pre = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(pre, d, 64);
                if (lane >= d) pre += t;
            }
            const int tot = __shfl(pre, 63, 64);
            const int first = pre - n;
            // the block's triangles are contiguous in the output: list kCap of
            // them at a time, then a lane per vertex
            uint32_t *ls = list[wv];
            for (int r0 = 0; r0 < tot; r0 += kCap) {
                if (first < r0 + kCap && first + n > r0) {
                    int li = first - r0;
                    for (uint32_t k = act; k; k &= k - 1) {
                        const int z = __ffs((int)k) - 1;
                        const uint32_t m = cell_case(z);
                        const int nt = ntri[m];
                        const uint32_t d = (uint32_t)(cx | (cy << 3) | (z << 6)) | (m << 12);
                        for (int t = 0; t < nt; ++t, ++li)
                            if (li >= 0 && li < kCap) ls[li] = d | ((uint32_t)t << 9);
                    }
                }
                wave_sync();
                const int cnt = tot - r0 < kCap ? tot - r0 : kCap;
                const unsigned long long t0 = base + (unsigned long long)r0;
                const unsigned long long lim = o.max_tri > t0 ? o.max_tri - t0 : 0ull;
                const int keep = lim < (unsigned long long)cnt ? (int)lim : cnt;
                for (int i = lane; i < 3 * keep; i += 64) {
                    const int ti = (int)(((uint32_t)i * 43691u) >> 17);   // i / 3, exact below 2^16
                    const uint32_t d = ls[ti];
                    // edge 4 a + k runs along axis a from the k-th corner whose bit a is 0
                    const int ed = tri[(int)(d >> 12) * 15 + 3 * (int)((d >> 9) & 7u) + (i - 3 * ti)];
                    const int ax = ed >> 2, k = ed & 3;
                    const int c0 = ax == 0 ? 2 * k : (ax == 1 ? (k & 1) | ((k & 2) << 1) : k);
                    const int lx = (int)(d & 7u) + (c0 & 1), ly = (int)((d >> 3) & 7u) + ((c0 >> 1) & 1),
                              lz = (int)((d >> 6) & 7u) + (c0 >> 2);
                    const int at = (ly * 9 + lx) * kColStride + lz;
                    const int s0 = L.g[at], s1 = L.g[at + (ax == 0 ? kColStride : (ax == 1 ? 9 * kColStride : 1))];
                    const float f0 = (float)s0 * (1.0f / 32767.0f);
                    const float f1 = (float)s1 * (1.0f / 32767.0f);
                    const float tt = f0 / (f0 - f1);
                    const int gx = 8 * bx + lx, gy = 8 * by + ly, gz = 8 * bz + lz;
                    float px = (float)gx, py = (float)gy, pz = (float)gz;
                    if (ax == 0) px = px + tt;
                    else if (ax == 1) py = py + tt;
                    else pz = pz + tt;
                    const unsigned long long at3 = t0 * 3 + (unsigned long long)i;
                    if (o.verts) {
                        const Vert q = {px * voxel, py * voxel, pz * voxel};
                        reinterpret_cast<Vert *>(o.verts)[at3] = q;
                    }
                    if (o.keys)
                        o.keys[at3] = (long long)(((unsigned long long)(gx + (1 << 19)) << 42) |
                                                  ((unsigned long long)(gy + (1 << 19)) << 22) |
                                                  ((unsigned long long)(gz + (1 << 19)) << 2) | (unsigned long long)ax);
                }
                wave_sync();                         // the list is rewritten by the next round
            }
            base += (unsigned long long)tot;
        }
        if (!EMIT) {
            for (int off = 32; off > 0; off >>= 1) count += __shfl_xor(count, off, 64);
            if (lane == 0) o.chunk_off[chunk] = count;
        }
    }
}

// Exclusive offsets of the chunk counts within a group of kScanGroup chunks
// (one workgroup each, 16 consecutive chunks per thread) and the group's
// total; with a single group the total is the mesh's.  Bound: one read and
// one write of 4 bytes per chunk; one workgroup over every chunk took 125 us
// at 74 k chunks.
__global__ __launch_bounds__(256) void k_mesh_scan(MeshOut o)
{
    __shared__ uint32_t wsum[4];
    const uint32_t b = blockIdx.x * kScanGroup + threadIdx.x * 16u;
    uint32_t c[16], s = 0;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) c[i] = b + i < o.chunks ? o.chunk_off[b + i] : 0u;
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) s += c[i];
    uint32_t incl = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(incl, d, 64);
        if ((int)lane_id() >= d) incl += t;
    }
    if (lane_id() == 63) wsum[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t run = incl - s;
    for (uint32_t k = 0; k < threadIdx.x >> 6; ++k) run += wsum[k];
#pragma unroll
    for (uint32_t i = 0; i < 16; ++i) {
        if (b + i < o.chunks) o.chunk_off[b + i] = run;
        run += c[i];
    }
    if (threadIdx.x == 255) *(o.groups > 1 ? o.group + blockIdx.x : o.total) = run;
}

// exclusive offsets of the group totals and the mesh's total (one workgroup; at most 512 groups)
__global__ __launch_bounds__(512) void k_mesh_groups(MeshOut o)
{
    __shared__ unsigned long long part[512];
    const uint32_t t = threadIdx.x;
    const unsigned long long s = t < o.groups ? o.group[t] : 0ull;
    part[t] = s;
    __syncthreads();
    for (uint32_t d = 1; d < 512; d <<= 1) {
        const unsigned long long x = t >= d ? part[t - d] : 0ull;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    if (t < o.groups) o.group[t] = part[t] - s;
    if (t == 511) *o.total = part[511];
}

uint32_t mesh_chunks(uint32_t n_entries) { return (n_entries + kChunk - 1) / kChunk; }

}  // namespace

extern "C" {

size_t tf_mesh_workspace_bytes(const tf_params *p)
{
    if (!p || tf_workspace_bytes(p) == 0) return 0;
    const uint32_t n_entries = p->n_buckets + p->n_excess;
    return (size_t)mesh_chunks(n_entries) * sizeof(unsigned long long);
}

int tf_mesh(tf_ctx *ctx, float *d_vertices, int64_t *d_edge_keys, uint64_t max_triangles, uint64_t *d_count,
            void *d_workspace, size_t workspace_bytes, tf_stream stream)
{
    if (!ctx || !d_count || !d_workspace) return TF_E_INVAL;
    if (((uintptr_t)d_count & 7u) || ((uintptr_t)d_workspace & 7u) || ((uintptr_t)d_vertices & 3u) ||
        ((uintptr_t)d_edge_keys & 7u))
        return TF_E_INVAL;
    const uint32_t chunks = mesh_chunks(ctx->v.n_entries);
    if (workspace_bytes < (size_t)chunks * sizeof(unsigned long long)) return TF_E_SPACE;
    MeshOut o;
    o.verts = d_vertices;
    o.keys = (long long *)d_edge_keys;
    o.max_tri = max_triangles;
    // 8 bytes per chunk hold a 4-byte offset each and, from two scan groups on, the groups' totals behind them
    o.chunk_off = (uint32_t *)d_workspace;
    o.group = (unsigned long long *)((uint32_t *)d_workspace + (chunks + 1) / 2 * 2);
    o.total = (unsigned long long *)d_count;
    o.chunks = chunks;
    o.groups = (chunks + kScanGroup - 1) / kScanGroup;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t wgs = (chunks + kWaves - 1) / kWaves;
    const dim3 grid(wgs < (uint32_t)kGrid ? wgs : (uint32_t)kGrid), block(64 * kWaves);
    hipLaunchKernelGGL(k_mesh<false>, grid, block, 0, s, ctx->v, o, ctx->p.voxel_size);
    hipLaunchKernelGGL(k_mesh_scan, dim3(o.groups), dim3(256), 0, s, o);
    if (o.groups > 1) hipLaunchKernelGGL(k_mesh_groups, dim3(1), dim3(512), 0, s, o);
    if (d_vertices || d_edge_keys)
        hipLaunchKernelGGL(k_mesh<true>, grid, block, 0, s, ctx->v, o, ctx->p.voxel_size);
    return hipGetLastError() == hipSuccess ? TF_OK : TF_E_HIP;
}

}  // extern "C"

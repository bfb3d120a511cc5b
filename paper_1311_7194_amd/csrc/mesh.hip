// Marching-cubes extraction over the allocated blocks (Section 5: the
// polygonisation alternative to raycasting, in three stages: occupied cells
// and their output counts, a prefix sum into output offsets, polygonisation
// of the occupied cells only).
//
//   count   one wavefront per pool slot: the block's 9^3 corner tile (its own
//           512 voxels plus the x = 0 / y = 0 / z = 0 layers of its seven
//           +x/+y/+z neighbours) in registers, a z column per lane, as two
//           sign bits per corner; the triangles of the cells that the surface
//           crosses are summed
//   scan    per tile of 1024 slots, an exclusive scan of the block counts;
//           then one workgroup scans the tile sums and writes the total
//   emit    blocks with triangles reload their tile, also into LDS; a scan
//           over the 512 cells (in x + 8y + 64z order) places each cell's
//           triangles after the block's offset; then lanes take vertices
//
// What bounds it: count, the latency of the loads (keys, neighbours' slots,
// voxels); emit, the 72 bytes it writes a triangle.  On 56,000 blocks of FP32
// (2 mm, 3.8 million triangles): count 61 -> 44 us once a cell's case came from
// sign bits, eight cells at a time, instead of comparing eight floats from LDS
// each (57 % vector issue); emit 141 -> 98 us with the same, one scan for three
// layers, and lanes that write consecutive vertices instead of a triangle each
// (strides of 24, 12 and 36 bytes).  Not kept: loads of the next block's
// neighbour slots and key ahead of its turn (46 + 110 us), contiguous shares
// of the pool per XCD (47 + 112 us), more wavefronts by spilling registers.
//
// Cells: a cell spans the voxel centres g + {0,1}^3 and is valid when all
// eight hold a distance (|T_hat| <= 1) in allocated blocks inside the grid.
// Corner k (offset (k & 1, k >> 1 & 1, k >> 2 & 1)) is inside when F < 0.
// A crossed cell edge from voxel g along axis a carries one vertex, id
// 3 (gx + G0 (gy + G1 gz)) + a, at t = F(g) / (F(g) - F(g + e_a)).
//
// The case table is generated at compile time from this rule: on each cube
// face, walked counter-clockwise as seen from outside the cube, every
// crossing where the walk enters the inside corners is joined to the next
// crossing where it leaves them (so diagonal inside corners of an ambiguous
// face are cut off one by one, and the inside lies to the right of each
// segment seen from outside); the segments close into loops, and each loop,
// started at its smallest edge number, is fanned from that edge.  Cube edge
// 4a + m runs along axis a from the corner whose other two coordinates, in
// increasing axis order, are (m & 1, m >> 1).
#include <math.h>

#include "tsdf_internal.h"
#include "tsdf_mesh.h"

namespace tsdf {
namespace {

constexpr int kMcMaxTris = 5;

struct McTable {
    uint8_t ntri[256];
    uint8_t edge[256][3 * kMcMaxTris];
    bool overflow;   // a case needed more than kMcMaxTris triangles (rejected at compile time)
};

// Cube edge joining corners p and q (which differ in one coordinate bit).
constexpr int mc_edge(int p, int q)
{
    const int d = p ^ q;
    const int a = d == 1 ? 0 : (d == 2 ? 1 : 2);
    const int lo = p & q;
    const int u = a == 0 ? 1 : 0, w = a == 2 ? 1 : 2;
    return 4 * a + ((lo >> u) & 1) + 2 * ((lo >> w) & 1);
}

constexpr McTable make_mc_table()
{
    McTable tab{};
    for (int c = 0; c < 256; ++c) {
        int next[12] = {-1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
        for (int a = 0; a < 3; ++a) {
            for (int side = 0; side < 2; ++side) {
                const int u = a == 0 ? 1 : 0, w = a == 2 ? 1 : 2;
                const int b = side << a;
                int ring[4] = {b, b | (1 << u), b | (1 << u) | (1 << w), b | (1 << w)};
                // the ring above turns counter-clockwise about +e_a for a = 0, 2 and
                // clockwise for a = 1 (e_u x e_w = -e_y); seen from outside the face
                // (normal (2 side - 1) e_a) reverse it where the two disagree
                const bool ccw_about_plus = a != 1;
                if (ccw_about_plus != (side == 1)) {
                    const int t = ring[1];
                    ring[1] = ring[3];
                    ring[3] = t;
                }
                for (int k = 0; k < 4; ++k) {
                    const bool in_k = (c >> ring[k]) & 1, in_k1 = (c >> ring[(k + 1) & 3]) & 1;
                    if (in_k || !in_k1) continue;   // not an entering crossing
                    int j = (k + 1) & 3;
                    while (!(((c >> ring[j]) & 1) && !((c >> ring[(j + 1) & 3]) & 1))) j = (j + 1) & 3;
                    next[mc_edge(ring[k], ring[(k + 1) & 3])] = mc_edge(ring[j], ring[(j + 1) & 3]);
                }
            }
        }
        bool seen[12] = {};
        int nt = 0;
        for (int e0 = 0; e0 < 12; ++e0) {
            if (next[e0] < 0 || seen[e0]) continue;
            int loop[12] = {};
            int len = 0;
            for (int e = e0; !seen[e]; e = next[e]) {
                seen[e] = true;
                loop[len++] = e;
            }
            for (int i = 1; i + 1 < len; ++i) {
                if (nt == kMcMaxTris) {
                    tab.overflow = true;
                    break;
                }
                tab.edge[c][3 * nt + 0] = (uint8_t)loop[0];
                tab.edge[c][3 * nt + 1] = (uint8_t)loop[i];
                tab.edge[c][3 * nt + 2] = (uint8_t)loop[i + 1];
                ++nt;
            }
        }
        tab.ntri[c] = (uint8_t)nt;
    }
    return tab;
}

constexpr McTable kMcTableHost = make_mc_table();
static_assert(!kMcTableHost.overflow, "marching-cubes case with more than kMcMaxTris triangles");
static_assert(kMcTableHost.ntri[0] == 0 && kMcTableHost.ntri[255] == 0 && kMcTableHost.ntri[1] == 1,
              "marching-cubes table");

// A case in one word: its triangles' edges, 4 bits each from bit 0, and their
// number from bit 60.
struct McCases {
    unsigned long long word[256];
};
static_assert(3 * kMcMaxTris * 4 <= 60, "a case's edges and triangle count fit a word");

constexpr McCases make_mc_cases()
{
    McCases m{};
    for (int c = 0; c < 256; ++c) {
        unsigned long long w = (unsigned long long)kMcTableHost.ntri[c] << 60;
        for (int k = 0; k < 3 * kMcTableHost.ntri[c]; ++k) w |= (unsigned long long)kMcTableHost.edge[c][k] << (4 * k);
        m.word[c] = w;
    }
    return m;
}

__constant__ McCases kMcCases = make_mc_cases();

constexpr int kMcLanes = 64;         // one wavefront per block: lane (x, y) takes the cells of its z column
constexpr int kTile = 9;             // corner tile edge
// Single-wavefront workgroups striding over the pool: blocks differ in work, and
// a workgroup that gets few of them leaves the rest to the dispatcher (56,000
// blocks: 16384 workgroups 47 + 109 us, 32768 44 + 98 us, 65536 the same), but
// an empty one costs too, so a small pool gets a quarter of its capacity (pools
// are rarely full), or one round of resident wavefronts (8192).
constexpr uint32_t kMcGrid = 32768;
constexpr uint32_t kScanTile = 1024; // slots per first-level scan tile
constexpr int kOwnerChunk = 512;     // output triangles of a block placed per round

template <typename S>
__device__ __forceinline__ float mc_load(const S *p);
template <>
__device__ __forceinline__ float mc_load<float>(const float *p) { return *p; }
template <>
__device__ __forceinline__ float mc_load<__half>(const __half *p) { return __half2float(*p); }

struct McLds {
    float f[kTile * kTile * kTile];   // corner tile, x fastest
    uint32_t owner[kOwnerChunk];      // cell | its three edges << 9 (4 bits each) of a round's triangles
};

__device__ __forceinline__ int tidx(int x, int y, int z) { return x + kTile * y + kTile * kTile * z; }

// Corner tile of a block over the lanes of a wavefront, lane (x, y) = t & 7,
// t >> 3: its own z column, and of the neighbours' layers
//   halo[0]  (8, t >> 3, t & 7)    halo[1]  (t >> 3, 8, t & 7)    halo[2]  (x, y, 8)
//   halo[3]  t < 8: (8, 8, t)   t < 16: (8, t - 8, 8)   t < 24: (t - 16, 8, 8)   24: (8, 8, 8)
// (chi where a neighbour block is unallocated or outside the grid).
struct TileRegs {
    float own[8], halo[4];
};

template <typename S>
__device__ __forceinline__ void load_tile(const VolumeView &v, uint32_t slot, uint32_t key, TileRegs &r)
{
    const int t = threadIdx.x;
    const S *T = (const S *)v.poolT;
    int bx, by, bz;
    unpack_key(key, bx, by, bz);
    int32_t s = -1;   // lanes 1..7: pool slots of the +x/+y/+z neighbours (-1: none)
    if (t >= 1 && t < 8) {
        const int nx = bx + (t & 1), ny = by + ((t >> 1) & 1), nz = bz + (t >> 2);
        if (nx < v.nblk[0] && ny < v.nblk[1] && nz < v.nblk[2]) {
            if (v.block_index) {
                s = v.block_index[block_linear(v, nx, ny, nz)];
            } else {
                s = hash_find(v, pack_key(nx, ny, nz));
            }
        }
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) r.own[z] = mc_load<S>(T + (size_t)slot * kBlockVoxels + t + 64 * z);
    const int32_t s1 = __builtin_amdgcn_readlane(s, 1), s2 = __builtin_amdgcn_readlane(s, 2),
                  s4 = __builtin_amdgcn_readlane(s, 4);
    const int n3 = t < 8 ? 3 : t < 16 ? 5 : t < 24 ? 6 : 7;
    const int32_t s3 = __shfl(s, n3);
    const uint32_t at = t < 8 ? 64 * t : t < 16 ? 8 * (t - 8) : t < 24 ? t - 16 : 0;
    r.halo[0] = r.halo[1] = r.halo[2] = r.halo[3] = kChi;
    if (s1 >= 0) r.halo[0] = mc_load<S>(T + (size_t)s1 * kBlockVoxels + 8 * (t >> 3) + 64 * (t & 7));
    if (s2 >= 0) r.halo[1] = mc_load<S>(T + (size_t)s2 * kBlockVoxels + (t >> 3) + 64 * (t & 7));
    if (s4 >= 0) r.halo[2] = mc_load<S>(T + (size_t)s4 * kBlockVoxels + t);
    if (t < 25 && s3 >= 0) r.halo[3] = mc_load<S>(T + (size_t)s3 * kBlockVoxels + at);
}

// Signs of the four corner columns of a lane's cells (bit z: F < 0 at layer z =
// 0..8), and which of its eight cells have triangles: all corners distances,
// some but not all inside.  Everything a cell's case needs is two bits a
// corner, so a column of them fits a register, neighbours' columns come by
// shuffle, and the cells are tested eight at a time.
struct Columns {
    uint32_t neg[4];   // columns (x, y), (x + 1, y), (x, y + 1), (x + 1, y + 1)
    uint32_t mixed;    // bit z
};

__device__ __forceinline__ Columns column_signs(const TileRegs &r)
{
    const int t = threadIdx.x, x = t & 7, y = t >> 3;
    uint32_t c00 = 0;   // bits 0..8: a distance; bits 16..24: below zero
#pragma unroll
    for (int z = 0; z < 9; ++z) {
        const float f = z < 8 ? r.own[z < 8 ? z : 0] : r.halo[2];
        c00 |= (fabsf(f) <= 1.0f ? 1u << z : 0u) | (f < 0.0f ? 0x10000u << z : 0u);
    }
    unsigned long long ok[3], ng[3];   // the neighbours' layers 0, 1 and 3 as bits
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const float f = r.halo[q == 2 ? 3 : q];
        ok[q] = __ballot(fabsf(f) <= 1.0f);
        ng[q] = __ballot(f < 0.0f);
    }
    auto column = [](unsigned long long m, int byte, unsigned long long top, int bit) {
        return ((uint32_t)(m >> (8 * byte)) & 0xffu) | ((uint32_t)(top >> bit) & 1u) << 8;
    };
    uint32_t c10 = (uint32_t)__shfl((int)c00, t + 1), c01 = (uint32_t)__shfl((int)c00, t + 8);
    if (x == 7) c10 = column(ok[0], y, ok[2], 8 + y) | column(ng[0], y, ng[2], 8 + y) << 16;
    if (y == 7) c01 = column(ok[1], x, ok[2], 16 + x) | column(ng[1], x, ng[2], 16 + x) << 16;
    uint32_t c11 = (uint32_t)__shfl((int)c10, t + 8);
    const uint32_t c11y = (uint32_t)__shfl((int)c01, t + 1);
    if (y == 7) c11 = x < 7 ? c11y : column(ok[2], 0, ok[2], 24) | column(ng[2], 0, ng[2], 24) << 16;
    Columns c;
    c.neg[0] = c00 >> 16;
    c.neg[1] = c10 >> 16;
    c.neg[2] = c01 >> 16;
    c.neg[3] = c11 >> 16;
    const uint32_t all = c00 & c10 & c01 & c11, any = (c00 | c10 | c01 | c11) >> 16;
    c.mixed = (all & all >> 1) & (any | any >> 1) & ~(all >> 16 & all >> 17) & 0xffu;
    return c;
}

// Word of the case table of the lane's cell z.
__device__ __forceinline__ unsigned long long cell_case(const Columns &c, int z)
{
    uint32_t k = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t two = c.neg[q] >> z;
        k |= (two & 1u) << q | (two & 2u) << (q + 3);
    }
    return kMcCases.word[k];
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += (uint32_t)__shfl_xor((int)x, off);
    return x;
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
    const int lane = __lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, off);
        if (lane >= off) x += y;
    }
    return x;
}

template <typename S>
__global__ __launch_bounds__(kMcLanes) void mc_count_kernel(VolumeView v, uint32_t *__restrict__ counts)
{
    const uint32_t n = min(v.state->pool_count, v.capacity);
    for (uint32_t slot = blockIdx.x; slot < n; slot += gridDim.x) {
        const uint32_t key = v.pool_keys[slot];
        if (key == kEmptyKey) {   // a slot whose insertion failed holds no block
            if (threadIdx.x == 0) counts[slot] = 0;
            continue;
        }
        TileRegs r;
        load_tile<S>(v, slot, key, r);
        const Columns c = column_signs(r);
        uint32_t nt = 0;
        for (uint32_t m = c.mixed; m; m &= m - 1u) nt += (uint32_t)(cell_case(c, __builtin_ctz(m)) >> 60);
        nt = wave_sum(nt);
        if (threadIdx.x == 0) counts[slot] = nt;
    }
}

// Exclusive scan of counts within each tile of kScanTile slots (256 lanes x
// 4 slots); tile sums to tile_sum.
__global__ __launch_bounds__(256) void mc_scan_tiles_kernel(const VolumeView v, const uint32_t *__restrict__ counts,
                                                            uint32_t *__restrict__ offsets,
                                                            uint32_t *__restrict__ tile_sum)
{
    __shared__ uint32_t wtot[4];
    const uint32_t n = min(v.state->pool_count, v.capacity);
    const uint32_t base = blockIdx.x * kScanTile;
    if (base >= n) return;   // uniform over the workgroup
    const uint32_t i0 = base + 4 * threadIdx.x;
    uint32_t c[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = i0 + k < n ? counts[i0 + k] : 0u;
        s += c[k];
    }
    const uint32_t inc = wave_inclusive_scan(s);
    const int wave = threadIdx.x >> 6;
    if (__lane_id() == 63) wtot[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wtot[w];
    uint32_t run = before + inc - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (i0 + k < n) offsets[i0 + k] = run;
        run += c[k];
    }
    if (threadIdx.x == 255) tile_sum[blockIdx.x] = run;
}

// One workgroup: exclusive scan of the tile sums into tile_base; the total
// triangle count to *count.
__global__ __launch_bounds__(1024) void mc_scan_top_kernel(const VolumeView v, const uint32_t *__restrict__ tile_sum,
                                                           unsigned long long *__restrict__ tile_base,
                                                           unsigned long long *__restrict__ count)
{
    __shared__ unsigned long long wtot[16];
    __shared__ unsigned long long carry;
    const uint32_t n = min(v.state->pool_count, v.capacity);
    const uint32_t ntiles = (n + kScanTile - 1) / kScanTile;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = __lane_id();
    for (uint32_t b = 0; b < ntiles; b += 1024) {
        const uint32_t i = b + threadIdx.x;
        unsigned long long x = i < ntiles ? tile_sum[i] : 0ull;
        unsigned long long inc = x;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned long long y = __shfl_up(inc, off);
            if (lane >= off) inc += y;
        }
        if (lane == 63) wtot[wave] = inc;
        __syncthreads();
        unsigned long long before = carry;
        for (int w = 0; w < wave; ++w) before += wtot[w];
        if (i < ntiles) tile_base[i] = before + inc - x;
        __syncthreads();
        if (threadIdx.x == 1023) carry = before + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = carry;
}

// Emit: the block's triangles are placed in rounds of kOwnerChunk; in each
// round every cell writes, for each of its triangles in the round, its number
// and the triangle's edges into `owner` at the triangle's position, then lane
// k computes and writes the round's vertices k, k + 64, ...: consecutive lanes
// write consecutive elements of all three arrays.
template <typename S>
__global__ __launch_bounds__(kMcLanes) void mc_emit_kernel(VolumeView v, const uint32_t *__restrict__ counts,
                                                           const uint32_t *__restrict__ offsets,
                                                           const unsigned long long *__restrict__ tile_base,
                                                           unsigned long long cap, long long *__restrict__ vid,
                                                           float *__restrict__ tpar, float *__restrict__ xyz)
{
    __shared__ McLds L;
    const uint32_t n = min(v.state->pool_count, v.capacity);
    const int t = threadIdx.x;
    const long long G0 = v.dims[0], G1 = v.dims[1];
    for (uint32_t slot = blockIdx.x; slot < n; slot += gridDim.x) {
        const uint32_t total = counts[slot], key = v.pool_keys[slot];   // (four loads at once)
        const unsigned long long base = tile_base[slot / kScanTile] + offsets[slot];
        if (total == 0 || base >= cap) continue;   // uniform: no triangles (or no block) in this slot, or no room
        TileRegs r;
        load_tile<S>(v, slot, key, r);
        {
            const int x = t & 7, y = t >> 3;
#pragma unroll
            for (int z = 0; z < 8; ++z) L.f[tidx(x, y, z)] = r.own[z];
            L.f[tidx(8, y, x)] = r.halo[0];
            L.f[tidx(y, 8, x)] = r.halo[1];
            L.f[tidx(x, y, 8)] = r.halo[2];
            if (t < 25)
                L.f[t < 8 ? tidx(8, 8, t) : t < 16 ? tidx(8, t - 8, 8) : t < 24 ? tidx(t - 16, 8, 8) : tidx(8, 8, 8)] =
                    r.halo[3];
        }
        const Columns c = column_signs(r);
        // exclusive prefix of the triangle counts in cell order (x + 8y + 64z):
        // a field of ten bits a layer (at most 320 triangles), three to a word
        uint32_t nt[3] = {0, 0, 0}, pre[3], layer[9];
        for (uint32_t m = c.mixed; m; m &= m - 1u) {
            const int z = __builtin_ctz(m), w = z >= 6 ? 2 : z >= 3 ? 1 : 0;
            const uint32_t add = (uint32_t)(cell_case(c, z) >> 60) << (10 * (z - 3 * w));
            nt[0] += w == 0 ? add : 0u;
            nt[1] += w == 1 ? add : 0u;
            nt[2] += w == 2 ? add : 0u;
        }
        uint32_t run = 0;   // triangles of the layers below
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            const uint32_t inc = wave_inclusive_scan(nt[w]);
            const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            pre[w] = inc - nt[w];
            layer[3 * w] = run;
            layer[3 * w + 1] = run += sum & 1023u;
            layer[3 * w + 2] = run += sum >> 10 & 1023u;
            run += sum >> 20;
        }
        int bx, by, bz;
        unpack_key(key, bx, by, bz);
        // the block's first edge id; a cell's ids add less than 2^32 (at most
        // 8192 voxels a side)
        const long long first_id = 3 * (8LL * bx + G0 * (8LL * by + G1 * 8LL * bz));
        for (uint32_t r0 = 0; r0 < total; r0 += kOwnerChunk) {
            for (uint32_t m = c.mixed; m; m &= m - 1u) {
                const int z = __builtin_ctz(m), w = z >= 6 ? 2 : z >= 3 ? 1 : 0;
                const unsigned long long word = cell_case(c, z);
                uint32_t k = (w == 0 ? pre[0] : w == 1 ? pre[1] : pre[2]) >> (10 * (z - 3 * w)) & 1023u;
#pragma unroll
                for (int q = 0; q < 8; ++q) k += z == q ? layer[q] : 0u;
                k -= r0;   // (wraps for the triangles of earlier rounds)
                for (uint32_t i = 0; i < (uint32_t)(word >> 60); ++i)
                    if (k + i < (uint32_t)kOwnerChunk)
                        L.owner[k + i] = (uint32_t)(t + 64 * z) | (uint32_t)(word >> (12 * i) & 0xfffu) << 9;
            }
            __syncthreads();
            const unsigned long long o0 = base + r0;   // the round's first triangle
            const uint32_t room = (uint32_t)min(cap - min(o0, cap), (unsigned long long)kOwnerChunk);
            const uint32_t n_vert = 3u * min(min(total - r0, (uint32_t)kOwnerChunk), room);
            long long *vid_r = vid + 3 * o0;
            float *tpar_r = tpar + 3 * o0, *xyz_r = xyz + 9 * o0;
            for (uint32_t k = t; k < n_vert; k += kMcLanes) {
                const uint32_t tri = k / 3u, j = k - 3u * tri;
                const uint32_t e = L.owner[tri];
                const int cx = (int)(e & 7u), cy = (int)(e >> 3 & 7u), cz = (int)(e >> 6 & 7u);
                const int ed = (int)(e >> (9u + 4u * j) & 15u);
                const int a = ed >> 2, m = ed & 3;   // the edge's lower corner
                const int lx = a == 0 ? 0 : m & 1, ly = a == 0 ? m & 1 : a == 2 ? m >> 1 : 0, lz = a == 2 ? 0 : m >> 1;
                const int dx = cx + lx, dy = cy + ly, dz = cz + lz;
                const int at = tidx(dx, dy, dz), step = a == 0 ? 1 : a == 1 ? kTile : kTile * kTile;
                const float flo = L.f[at], fhi = L.f[at + step];
                const float te = flo / (flo - fhi);
                vid_r[k] = first_id + (long long)(3u * ((uint32_t)dx + (uint32_t)G0 * ((uint32_t)dy + (uint32_t)G1 * (uint32_t)dz)) +
                                                  (uint32_t)a);
                tpar_r[k] = te;
                if (xyz) {
                    const double p[3] = {(double)(8 * bx + dx) + 0.5 + (a == 0 ? (double)te : 0.0),
                                         (double)(8 * by + dy) + 0.5 + (a == 1 ? (double)te : 0.0),
                                         (double)(8 * bz + dz) + 0.5 + (a == 2 ? (double)te : 0.0)};
#pragma unroll
                    for (int q = 0; q < 3; ++q) xyz_r[3 * k + q] = (float)(v.origin[q] + p[q] * v.vs);
                }
            }
            __syncthreads();
        }
    }
}

struct MeshWork {
    uint32_t *counts, *offsets, *tile_sum;
    unsigned long long *tile_base;
    uint64_t bytes;
};

uint64_t align256(uint64_t b) { return (b + 255) & ~(uint64_t)255; }

MeshWork mesh_work(const VolumeView &v, void *base)
{
    const uint64_t cap = v.capacity, tiles = (cap + kScanTile - 1) / kScanTile;
    MeshWork w{};
    uint8_t *p = (uint8_t *)base;
    w.counts = (uint32_t *)p;
    p += align256(4 * cap);
    w.offsets = (uint32_t *)p;
    p += align256(4 * cap);
    w.tile_sum = (uint32_t *)p;
    p += align256(4 * tiles);
    w.tile_base = (unsigned long long *)p;
    p += align256(8 * tiles);
    w.bytes = (uint64_t)(p - (uint8_t *)base);
    return w;
}

}  // namespace
}  // namespace tsdf

using namespace tsdf;

extern "C" {

int32_t tsdf_mesh_case(int32_t c, int32_t edges[15])
{
    if (c < 0 || c > 255 || !edges) return -1;
    for (int i = 0; i < 15; ++i) edges[i] = i < 3 * kMcTableHost.ntri[c] ? kMcTableHost.edge[c][i] : -1;
    return kMcTableHost.ntri[c];
}

uint64_t tsdf_mesh_workspace_bytes(const tsdf_volume *vol)
{
    if (!vol) return 0;
    return mesh_work(volume_view(vol), nullptr).bytes;
}

tsdf_status tsdf_extract_mesh(tsdf_volume *vol, int64_t *vertex_id_dev, float *t_dev, float *xyz_dev, uint64_t cap,
                              void *work_dev, uint64_t work_bytes, uint64_t *count_dev, hipStream_t stream)
{
    if (!vol || !count_dev || !work_dev || work_bytes < tsdf_mesh_workspace_bytes(vol) ||
        (cap > 0 && (!vertex_id_dev || !t_dev)))
        return TSDF_EINVAL;
    const tsdf_status st = volume_enqueue(vol, stream, nullptr);
    if (st != TSDF_OK) return st;
    const VolumeView v = volume_view(vol);
    const MeshWork w = mesh_work(v, work_dev);
    const uint32_t tiles = (v.capacity + kScanTile - 1) / kScanTile;
    const uint32_t round = v.capacity < 8192u ? v.capacity : 8192u;
    const uint32_t want = v.capacity / 4 > round ? v.capacity / 4 : round;
    const dim3 grid(want < kMcGrid ? want : kMcGrid);
    const bool f16 = v.storage == TSDF_F16;
    if (f16)
        hipLaunchKernelGGL(mc_count_kernel<__half>, grid, dim3(kMcLanes), 0, stream, v, w.counts);
    else
        hipLaunchKernelGGL(mc_count_kernel<float>, grid, dim3(kMcLanes), 0, stream, v, w.counts);
    hipLaunchKernelGGL(mc_scan_tiles_kernel, dim3(tiles), dim3(256), 0, stream, v, w.counts, w.offsets, w.tile_sum);
    hipLaunchKernelGGL(mc_scan_top_kernel, dim3(1), dim3(1024), 0, stream, v, w.tile_sum, w.tile_base,
                       (unsigned long long *)count_dev);
    if (cap > 0) {
        if (f16)
            hipLaunchKernelGGL(mc_emit_kernel<__half>, grid, dim3(kMcLanes), 0, stream, v, w.counts,
                               w.offsets, w.tile_base, (unsigned long long)cap, (long long *)vertex_id_dev, t_dev,
                               xyz_dev);
        else
            hipLaunchKernelGGL(mc_emit_kernel<float>, grid, dim3(kMcLanes), 0, stream, v, w.counts,
                               w.offsets, w.tile_base, (unsigned long long)cap, (long long *)vertex_id_dev, t_dev,
                               xyz_dev);
    }
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

}  // extern "C"

// Device bodies of the range pass and the raycast march, shared by the
// single-volume kernels (raycast.hip) and the batched kernels (batch.hip).
// See raycast.hip for the method.
#pragma once

#include "tsdf_internal.h"

namespace tsdf {

constexpr int kRT = 8;                      // raycast tile edge in pixels
constexpr uint32_t kInfBits = 0x7f800000u;  // +inf as float bits
constexpr int kCellFootprint = 64;          // largest footprint (cells) a block widens cell by cell
// ------------------------------------------------------------ range maps

constexpr int kCellsPerTile = kRT / kCell;   // cells along a tile edge

// Clears the depth spans of one frame: thread gt of a launch space of
// (tiles x 64) clears cell `gt % 64` of tile `gt / 64` (if the tile has that
// many cells), and the tile itself.
__device__ __forceinline__ void range_clear_body(const VolumeView &v, int tiles_x, int tiles_y, int width,
                                                 int height, long long gt)
{
    const long long tile = gt >> 6;
    const int within = (int)(gt & 63);
    const long long nt = (long long)tiles_x * tiles_y;
    if (tile >= nt) return;
    if (within == 0) {
        v.tile_range[tile] = kInfBits;
        v.tile_range[nt + tile] = 0u;
    }
    if (within >= kCellsPerTile * kCellsPerTile) return;
    const int cw = (width + kCell - 1) / kCell, ch = (height + kCell - 1) / kCell;
    const int ci = (int)(tile % tiles_x) * kCellsPerTile + within % kCellsPerTile;
    const int cj = (int)(tile / tiles_x) * kCellsPerTile + within / kCellsPerTile;
    if (ci < cw && cj < ch) {
        const size_t c = (size_t)cj * cw + ci;
        v.pix_range[c] = kInfBits;
        v.pix_range[(size_t)cw * ch + c] = 0u;
    }
}

// ------------------------------------------------------------ range pass

// Block of the virtual grid -> pool slot, or -1.  The block must lie in the grid.
template <bool kDense>
__device__ __forceinline__ int32_t block_slot(const VolumeView &v, int bx, int by, int bz)
{
    if constexpr (kDense) return v.block_index[(uint32_t)block_linear(v, bx, by, bz)];
    return occupied(v, bx, by, bz) ? hash_find(v, pack_key(bx, by, bz)) : -1;
}

// Cell spans gathered in LDS by one workgroup before they go to memory:
// consecutive pool slots are neighbours in space, so their blocks widen the
// same cells, and one pair of memory atomics per distinct cell replaces one
// per block.  Keys are (scene << 26) | cell.
constexpr int kSpanLds = 512;
constexpr uint32_t kSpanEmpty = 0xffffffffu;
constexpr int kRangeChunk = 64;   // pool slots a workgroup takes at a time
struct RangeLds {
    uint32_t key[kSpanLds], lo[kSpanLds], hi[kSpanLds];   // span table
    uint32_t slot[kRangeChunk], bkey[kRangeChunk];        // the chunk's blocks in view
    uint32_t box[kRangeChunk];                            // their boxes
    uint4 rect[kRangeChunk];                              // what these cover: cells c0 | c1 << 16, d0 | d1 << 16, depths
    uint32_t n;
};

__device__ __forceinline__ void span_lds_init(RangeLds &L)
{
    for (int e = threadIdx.x; e < kSpanLds; e += blockDim.x) {
        L.key[e] = kSpanEmpty;
        L.lo[e] = kInfBits;
        L.hi[e] = 0u;
    }
}

// Widens the entry of `key` (false when its probe run is full).
__device__ __forceinline__ bool span_lds_add(RangeLds &L, uint32_t key, uint32_t zl, uint32_t zh)
{
    uint32_t h = (key * 2654435761u) >> (32 - 9);
#pragma unroll 1
    for (int p = 0; p < 8; ++p) {
        const uint32_t k = atomicCAS(&L.key[h], kSpanEmpty, key);
        if (k == kSpanEmpty || k == key) {
            atomicMin(&L.lo[h], zl);
            atomicMax(&L.hi[h], zh);
            return true;
        }
        h = (h + 1) & (kSpanLds - 1);
    }
    return false;
}

// Projection of a box of voxel-centre coordinates q in [8B + lo, 8B + hi]
// (x = origin + (q + 1/2) voxel): its camera depths and the pixel centres it
// may cover.
struct BoxView {
    float zlo, zhi;
    int i0, i1, j0, j1;
    bool behind;    // reaches the camera plane: depths and pixels are not bounded
    bool visible;   // in front of the camera and over at least one pixel centre (or behind)
};

__device__ __forceinline__ BoxView project_box(const VolumeView &v, const Camera &cam, int bx, int by, int bz,
                                               const int lo[3], const int hi[3])
{
    // camera axes in float: x_c = R^T (x - t)
    const float R[9] = {(float)cam.R[0], (float)cam.R[1], (float)cam.R[2], (float)cam.R[3], (float)cam.R[4],
                        (float)cam.R[5], (float)cam.R[6], (float)cam.R[7], (float)cam.R[8]};
    const float fx = (float)cam.fx, fy = (float)cam.fy, cx = (float)cam.cx, cy = (float)cam.cy;
    const float bwx = (float)((hi[0] - lo[0]) * v.vs), bwy = (float)((hi[1] - lo[1]) * v.vs),
                bwz = (float)((hi[2] - lo[2]) * v.vs);
    // its min corner relative to the camera centre, in double then float
    const float ox = (float)(v.origin[0] + (8.0 * bx + lo[0] + 0.5) * v.vs - cam.t[0]);
    const float oy = (float)(v.origin[1] + (8.0 * by + lo[1] + 0.5) * v.vs - cam.t[1]);
    const float oz = (float)(v.origin[2] + (8.0 * bz + lo[2] + 0.5) * v.vs - cam.t[2]);
    float zlo = 3.4e38f, zhi = -3.4e38f, ulo = 3.4e38f, uhi = -3.4e38f, vlo = 3.4e38f, vhi = -3.4e38f;
    BoxView w;
    w.behind = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float dx = ox + ((k & 1) ? bwx : 0.0f), dy = oy + ((k & 2) ? bwy : 0.0f),
                    dz = oz + ((k & 4) ? bwz : 0.0f);
        const float xc = R[0] * dx + R[3] * dy + R[6] * dz;
        const float yc = R[1] * dx + R[4] * dy + R[7] * dz;
        const float zc = R[2] * dx + R[5] * dy + R[8] * dz;
        zlo = fminf(zlo, zc);
        zhi = fmaxf(zhi, zc);
        w.behind |= !(zc > 1e-4f);
        const float rz = 1.0f / zc;
        ulo = fminf(ulo, fx * xc * rz + cx);
        uhi = fmaxf(uhi, fx * xc * rz + cx);
        vlo = fminf(vlo, fy * yc * rz + cy);
        vhi = fmaxf(vhi, fy * yc * rz + cy);
    }
    // pixel centres (i, j) inside the projected box; eps bounds the float
    // error of the projected corners (positions rounded to float relative to
    // the camera, then three products and a reciprocal)
    const float eps = 1e-5f * (fabsf(ulo - cx) + fabsf(uhi - cx) + fabsf(vlo - cy) + fabsf(vhi - cy) + fx + fy) +
                      1e-3f;
    const float ulo_e = fmaxf(ulo - eps, -1.0f), uhi_e = fminf(uhi + eps, (float)cam.width);
    const float vlo_e = fmaxf(vlo - eps, -1.0f), vhi_e = fminf(vhi + eps, (float)cam.height);
    w.zlo = zlo;
    w.zhi = zhi;
    w.i0 = max((int)ceilf(ulo_e), 0);
    w.i1 = min((int)floorf(uhi_e), cam.width - 1);
    w.j0 = max((int)ceilf(vlo_e), 0);
    w.j1 = min((int)floorf(vhi_e), cam.height - 1);
    w.visible = zhi > 0.0f && (w.behind || (ulo_e <= uhi_e && vlo_e <= vhi_e && w.i0 <= w.i1 && w.j0 <= w.j1));
    return w;
}

// Records of the blocks in view of a chunk (L.slot, L.bkey: `count` of them),
// by 16 lanes each (r = lane & 15): lanes 0..7 look up the block and its upper
// neighbours B + {0,1}^3, lanes 0..8 combine one row (fixed y) of voxel masks
// each, row 8 being the first row of the upper y neighbours.  F is a convex
// combination of its cell's eight voxels, so a bracket can end (F <= 0) only
// in a cell without a chi voxel and with one at or below zero, and begin
// (F > 0) only in one without a chi voxel and with one above zero.  L.box
// receives the bounding box of the cells of the first kind.
//
// The work is a chain of three dependent loads (neighbour slots, masks) and
// little arithmetic, so a thread's four blocks go through it together.
template <bool kDense>
__device__ __forceinline__ void block_records(const VolumeView &v, uint32_t count, RangeLds &L)
{
    constexpr int kPer = kRangeChunk / 16;
    const int r = threadIdx.x & 15, group = threadIdx.x & 48, e0 = threadIdx.x >> 4;
    const int row = r & 7, ny = r == 8 ? 2 : 0;   // the row's y, and the y neighbour it is taken from
    int32_t sl[kPer];
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        if (16u * t >= count) break;   // uniform over the workgroup
        const uint32_t e = min((uint32_t)(e0 + 16 * t), count - 1u);
        int bx, by, bz;
        unpack_key(L.bkey[e], bx, by, bz);
        const int x = bx + (r & 1), y = by + ((r >> 1) & 1), z = bz + ((r >> 2) & 1);
        const bool in = x < v.nblk[0] && y < v.nblk[1] && z < v.nblk[2];
        if constexpr (kDense) {
            const int32_t i = v.block_index[(uint32_t)(in ? block_linear(v, x, y, z) : block_linear(v, bx, by, bz))];
            sl[t] = in ? i : -1;
        } else {
            sl[t] = r < 8 && in ? block_slot<false>(v, x, y, z) : -1;
        }
    }
    unsigned long long oI[kPer], oV[kPer], zI[kPer], zV[kPer];
    uint32_t xI[kPer], xV[kPer], xzI[kPer], xzV[kPer];
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        if (16u * t >= count) break;
        const int32_t s0 = __shfl(sl[t], group | ny), sx = __shfl(sl[t], group | ny | 1),
                      sz = __shfl(sl[t], group | ny | 4), sxz = __shfl(sl[t], group | ny | 5);
        // an absent block's masks are those of this block, replaced by zeros below
        const int32_t self = __shfl(sl[t], group);
        const VoxelMasks *m0 = v.masks + (s0 < 0 ? self : s0), *mx = v.masks + (sx < 0 ? self : sx),
                         *mz = v.masks + (sz < 0 ? self : sz), *mxz = v.masks + (sxz < 0 ? self : sxz);
        const unsigned long long *r0 = (const unsigned long long *)m0, *rz = (const unsigned long long *)mz;
        oI[t] = r0[row];
        oV[t] = r0[8 + row];
        zI[t] = rz[row];
        zV[t] = rz[8 + row];
        xI[t] = mx->inside[8 * row];
        xV[t] = mx->value[8 * row];
        xzI[t] = mxz->inside[8 * row];
        xzV[t] = mxz->value[8 * row];
        if (s0 < 0) oV[t] = 0;     // (without a value the rest does not matter)
        if (sx < 0) xV[t] = 0;
        if (sz < 0) zV[t] = 0;
        if (sxz < 0) xzV[t] = 0;
    }
    const unsigned long long kLow = 0x0101010101010101ull, kBut7 = 0x7f7f7f7f7f7f7f7full;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        if (16u * t >= count) break;
        const uint32_t e = min((uint32_t)(e0 + 16 * t), count - 1u);
        BlockRec *rec = v.recs + L.slot[e];
        if (r < 8) rec->base[r] = (sl[t] < 0 ? v.capacity : (uint32_t)sl[t]) * (uint32_t)kBlockVoxels;   // absent: chi
        // per row, byte x and bit z: some voxel of the cell inside (any), all
        // inside (all), none chi (val)
        // bit z: voxels z and z + 1, the latter from the z neighbour for z = 7
        const unsigned long long up = ((oI[t] >> 1) & kBut7) | ((zI[t] & kLow) << 7);
        unsigned long long all = oI[t] & up, any = oI[t] | up;
        unsigned long long val = oV[t] & (((oV[t] >> 1) & kBut7) | ((zV[t] & kLow) << 7));
        const uint32_t xup = (xI[t] >> 1) | ((xzI[t] & 1u) << 7);
        const uint32_t xall = xI[t] & xup, xany = xI[t] | xup, xval = xV[t] & ((xV[t] >> 1) | ((xzV[t] & 1u) << 7));
        // byte x: columns x and x + 1
        any |= (any >> 8) | ((unsigned long long)xany << 56);
        all &= (all >> 8) | ((unsigned long long)xall << 56);
        val &= (val >> 8) | ((unsigned long long)xval << 56);
        // rows y and y + 1
        any |= (unsigned long long)__shfl_down((long long)any, 1);
        all &= (unsigned long long)__shfl_down((long long)all, 1);
        val &= (unsigned long long)__shfl_down((long long)val, 1);
        const unsigned long long A = r < 8 ? any & val : 0ull;
        const unsigned long long B = val & ~all;
        if (r < 8) {
            uint32_t w[4];   // columns 2k and 2k + 1: the bytes of A and B interleaved
#pragma unroll
            for (int k = 0; k < 4; ++k)
                w[k] = __builtin_amdgcn_perm((uint32_t)(B >> (k & 2 ? 32 : 0)), (uint32_t)(A >> (k & 2 ? 32 : 0)),
                                             k & 1 ? 0x07030602u : 0x05010400u);
            ((uint4 *)rec->cell)[r] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        // bounding box: z bits and x bits of the row, then over the rows
        const uint32_t lo = (uint32_t)A, hi = (uint32_t)(A >> 32);
        uint32_t zb = lo | hi;
        zb |= zb >> 16;
        zb = (zb | (zb >> 8)) & 0xffu;
        // columns of the row that are not empty: bit 7 of each byte, gathered
        const uint32_t nl = (((lo & 0x7f7f7f7fu) + 0x7f7f7f7fu) | lo) & 0x80808080u;
        const uint32_t nh = (((hi & 0x7f7f7f7fu) + 0x7f7f7f7fu) | hi) & 0x80808080u;
        const uint32_t xb = (((nl >> 7) * 0x01020408u) >> 24 & 0xfu) | ((((nh >> 7) * 0x01020408u) >> 24 & 0xfu) << 4);
        uint32_t m = zb | (xb << 8) | (A ? 1u << (16 + r) : 0u);
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) m |= (uint32_t)__shfl_xor((int)m, off);
        if (r == 0 && e0 + 16 * t < (int)count) {
            uint32_t box = 0;
            if (m) {
                const uint32_t z = m & 0xffu, x = (m >> 8) & 0xffu, y = (m >> 16) & 0xffu;
                box = box_make(__builtin_ctz(x), __builtin_ctz(y), __builtin_ctz(z), 31 - __builtin_clz(x),
                               31 - __builtin_clz(y), 31 - __builtin_clz(z));
            }
            rec->box = box;
            L.box[e] = box;
        }
    }
}

// The pool slots [first, first + kRangeChunk) below n of one scene, by a
// workgroup of 256 threads: the blocks in view, their active cells, and the
// spans of those.  Cell spans go to `emit(cell, zl, zh)`; tile spans and the
// near-plane stamp go to memory.  Ends with a barrier.
template <bool kDense, typename Emit>
__device__ __forceinline__ void range_chunk(const VolumeView &v, const Camera &cam, uint32_t stamp, int tiles_x,
                                            int tiles_y, uint32_t first, uint32_t n, RangeLds &L, Emit &&emit)
{
    const int tid = threadIdx.x;
    if (tid == 0) L.n = 0;
    __syncthreads();
    if (tid < kRangeChunk) {
        // samples based in block B have q in [8B, 8B + 8], and a pixel's rays
        // need the records of the blocks up to one voxel off them (normals)
        const uint32_t slot = first + tid;
        const uint32_t key = slot < n ? v.pool_keys[slot] : kEmptyKey;
        bool in = false;
        if (key != kEmptyKey) {   // (a slot whose insertion failed holds no block)
            int bx, by, bz;
            unpack_key(key, bx, by, bz);
            const int lo[3] = {-1, -1, -1}, hi[3] = {9, 9, 9};
            in = project_box(v, cam, bx, by, bz, lo, hi).visible;
        }
        const unsigned long long m = __ballot(in);   // one wavefront
        if (in) {
            const int e = __popcll(m & ((1ull << tid) - 1ull));
            L.slot[e] = slot;
            L.bkey[e] = key;
        }
        if (tid == 0) L.n = (uint32_t)__popcll(m);
    }
    __syncthreads();
    const uint32_t count = L.n;
    if (count) block_records<kDense>(v, count, L);
    __syncthreads();
    if ((uint32_t)tid < count) {
        uint4 rect = make_uint4(1u, 1u, 0u, 0u);   // no cells
        const uint32_t box = L.box[tid];
        if (box & kBoxValid) {
            int bx, by, bz;
            unpack_key(L.bkey[tid], bx, by, bz);
            // samples based in these cells: q in [8B + lo, 8B + hi + 1]
            const int lo[3] = {box_lo(box, 0), box_lo(box, 1), box_lo(box, 2)};
            const int hi[3] = {box_hi(box, 0) + 1, box_hi(box, 1) + 1, box_hi(box, 2) + 1};
            const BoxView w = project_box(v, cam, bx, by, bz, lo, hi);
            if (w.visible && w.behind) {
                v.state->near_stamp = stamp;   // reaches the camera plane: rays start at the camera
            } else if (w.visible) {
                const uint32_t zl = __float_as_uint(fmaxf(w.zlo * (1.0f - 1e-5f) - 1e-6f, 0.0f));
                const uint32_t zh = __float_as_uint(w.zhi * (1.0f + 1e-5f) + 1e-6f);
                const int c0 = w.i0 / kCell, c1 = w.i1 / kCell, d0 = w.j0 / kCell, d1 = w.j1 / kCell;
                if ((c1 - c0 + 1) * (d1 - d0 + 1) <= kCellFootprint) {
                    rect = make_uint4((uint32_t)c0 | ((uint32_t)c1 << 16), (uint32_t)d0 | ((uint32_t)d1 << 16), zl, zh);
                } else {
                    // large footprint (blocks close to the camera): widen whole tiles
                    uint32_t *tmin = v.tile_range;
                    uint32_t *tmax = v.tile_range + (size_t)tiles_x * tiles_y;
                    for (int tj = w.j0 / kRT; tj <= w.j1 / kRT; ++tj)
                        for (int ti = w.i0 / kRT; ti <= w.i1 / kRT; ++ti) {
                            const size_t t = (size_t)tj * tiles_x + ti;
                            if (tmin[t] > zl) atomicMin(&tmin[t], zl);
                            if (tmax[t] < zh) atomicMax(&tmax[t], zh);
                        }
                }
            }
        }
        L.rect[tid] = rect;
    }
    __syncthreads();
    // small footprint: widen the span of every cell it covers (four lanes a block)
    if ((uint32_t)(tid >> 2) < count) {
        const uint4 rect = L.rect[tid >> 2];
        const int c0 = rect.x & 0xffffu, c1 = rect.x >> 16, d0 = rect.y & 0xffffu, d1 = rect.y >> 16;
        const int w = c1 - c0 + 1, ncell = w * (d1 - d0 + 1), cw = (cam.width + kCell - 1) / kCell;
        if (w > 0)
            for (int k = tid & 3; k < ncell; k += 4) {
                const int dy = k / w;
                emit((uint32_t)((d0 + dy) * cw + c0 + (k - dy * w)), rect.z, rect.w);
            }
    }
    __syncthreads();
}

// ------------------------------------------------------------ march

// Rays in voxel-centre coordinates q = (x - origin) / voxel - 1/2: q = q0 + s dq,
// q0 the camera centre (Camera::q0, the same for every ray).
struct Ray {
    const double *q0;
    double dq[3];    // dq/ds: the unit world direction over the voxel size
};

// Reciprocal and reciprocal square root to about an ulp: the hardware
// estimate and two Newton steps.
__device__ __forceinline__ double fast_rcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double fast_rsqrt(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = y * fma(-0.5 * x * y, y, 1.5);
    return y * fma(-0.5 * x * y, y, 1.5);
}

template <typename S>
__device__ __forceinline__ float ld(const S *p);
template <>
__device__ __forceinline__ float ld<float>(const float *p) { return *p; }
template <>
__device__ __forceinline__ float ld<__half>(const __half *p) { return __half2float(*p); }

// The block a lane's last sample was based in: its packed coordinates, and the
// pool offsets of it and its upper neighbours (absent ones: the chi block, so
// that a stencil reaching them reads chi and is invalid without a branch).
struct BlockCache {
    uint32_t key;
    uint32_t base[8];
};

template <bool kDense>
__device__ __forceinline__ void enter_block(const VolumeView &v, BlockCache &cache, const int c[3])
{
    const int bx = c[0] >> 3, by = c[1] >> 3, bz = c[2] >> 3;
    const uint32_t key = pack_key(bx, by, bz);
    if (key == cache.key) return;
    cache.key = key;
    const int32_t slot = block_slot<kDense>(v, bx, by, bz);
    if (slot >= 0) {
        const uint4 *b = (const uint4 *)v.recs[slot].base;
        const uint4 lo = b[0], hi = b[1];
        cache.base[0] = lo.x;
        cache.base[1] = lo.y;
        cache.base[2] = lo.z;
        cache.base[3] = lo.w;
        cache.base[4] = hi.x;
        cache.base[5] = hi.y;
        cache.base[6] = hi.z;
        cache.base[7] = hi.w;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) cache.base[k] = v.capacity * (uint32_t)kBlockVoxels;
    }
}

// Trilinear F at integer base c (global voxel indices) with fractions f, c in
// the cached block.  False when invalid.
template <typename S>
__device__ __forceinline__ bool interp(const VolumeView &v, const BlockCache &cache, const int c[3], const float f[3],
                                       float &F)
{
    const S *__restrict__ pool = (const S *)v.poolT;
    const uint32_t l0 = c[0] & 7, l1 = c[1] & 7, l2 = c[2] & 7;
    // the stencil's upper neighbour leaves the block along an axis only from local index 7
    const bool cx = l0 == 7, cy = l1 == 7, cz = l2 == 7;
    const uint32_t x0 = l0, x1 = cx ? 0u : l0 + 1u;
    const uint32_t y0 = 8u * l1, y1 = cy ? 0u : y0 + 8u;
    const uint32_t z0 = 64u * l2, z1 = cz ? 0u : z0 + 64u;
    // block of each corner (x fastest): select along x, then y, then z
    const uint32_t *b = cache.base;
    const uint32_t b0 = b[0], b1 = cx ? b[1] : b0;
    const uint32_t b2 = cy ? b[2] : b0, b3 = cy ? (cx ? b[3] : b[2]) : b1;
    const uint32_t t45 = cx ? b[5] : b[4], t67 = cx ? b[7] : b[6];
    const uint32_t b4 = cz ? b[4] : b0, b5 = cz ? t45 : b1;
    const uint32_t b6 = cz ? (cy ? b[6] : b[4]) : b2, b7 = cz ? (cy ? t67 : t45) : b3;
    const float v0 = ld(pool + (b0 + x0 + y0 + z0)), v1 = ld(pool + (b1 + x1 + y0 + z0));
    const float v2 = ld(pool + (b2 + x0 + y1 + z0)), v3 = ld(pool + (b3 + x1 + y1 + z0));
    const float v4 = ld(pool + (b4 + x0 + y0 + z1)), v5 = ld(pool + (b5 + x1 + y0 + z1));
    const float v6 = ld(pool + (b6 + x0 + y1 + z1)), v7 = ld(pool + (b7 + x1 + y1 + z1));
    const float m = fmaxf(fmaxf(fmaxf(fabsf(v0), fabsf(v1)), fmaxf(fabsf(v2), fabsf(v3))),
                          fmaxf(fmaxf(fabsf(v4), fabsf(v5)), fmaxf(fabsf(v6), fabsf(v7))));
    const float x00 = v0 + f[0] * (v1 - v0);
    const float x10 = v2 + f[0] * (v3 - v2);
    const float x01 = v4 + f[0] * (v5 - v4);
    const float x11 = v6 + f[0] * (v7 - v6);
    const float y0f = x00 + f[1] * (x10 - x00);
    const float y1f = x01 + f[1] * (x11 - x01);
    F = y0f + f[2] * (y1f - y0f);
    return m <= 1.0f;
}

__device__ __forceinline__ void q_at(const Ray &r, double s, double q[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) q[a] = r.q0[a] + s * r.dq[a];
}

// Stencil base voxel and fractions of q; false outside the grid.
__device__ __forceinline__ bool stencil(const VolumeView &v, const double q[3], int c[3], float f[3])
{
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double fl = floor(q[a]);
        inside &= (fl >= 0.0 && fl + 1.0 <= (double)(v.dims[a] - 1));
        c[a] = inside ? (int)fl : 0;
        f[a] = (float)(q[a] - fl);
    }
    return inside;
}

// F at q, NaN when the sample is invalid.
template <typename S, bool kDense>
__device__ __forceinline__ float sample(const VolumeView &v, BlockCache &cache, const double q[3])
{
    int c[3];
    float f[3];
    float F = __builtin_nanf("");
    if (stencil(v, q, c, f)) {
        enter_block<kDense>(v, cache, c);
        float Fs;
        if (interp<S>(v, cache, c, f, Fs)) F = Fs;
    }
    return F;
}

// First lattice index past the cells of block B, or of the aligned group of
// 2^sh blocks per axis around it, along the ray (the caller's samples before
// it all have their base voxel in there).  The division by h is a
// product with 1/h: the index found lies within one of the exit, and the
// test of its sample then returns the exit or one index before it (a later
// resume point is never returned).
__device__ __forceinline__ int cell_exit_sample(const Ray &r, const int B[3], int sh, double h, double inv_h)
{
    double s_exit = 1e300;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int lo = (B[a] >> sh) << (sh + 3);
        const double face = (double)(r.dq[a] > 0.0 ? lo + (8 << sh) : lo);
        if (r.dq[a] != 0.0) s_exit = fmin(s_exit, (face - r.q0[a]) * fast_rcp(r.dq[a]));
    }
    const int m = (int)fmin(floor(s_exit * inv_h), 2.0e9);
    double qm[3];
    q_at(r, (double)m * h, qm);
    const bool still = ((int)floor(qm[0]) >> (sh + 3)) == (B[0] >> sh) && ((int)floor(qm[1]) >> (sh + 3)) == (B[1] >> sh) &&
                       ((int)floor(qm[2]) >> (sh + 3)) == (B[2] >> sh);
    return still ? m + 1 : m;
}

// Shuffle inside a group of G lanes: value of lane `src` of this lane's group.
template <int G>
__device__ __forceinline__ int group_lane(int lane, int src) { return (lane & ~(G - 1)) | src; }

// Whether no voxel of the block in `slot` and its upper neighbours is at or below zero.
__device__ __forceinline__ bool all_positive(const VolumeView &v, int32_t slot)
{
    const BlockRec *rec = v.recs + slot;
    if (rec->box) return false;   // one of its cells has such a voxel
    for (int k = 0; k < 8; ++k) {
        const uint32_t s = rec->base[k] / (uint32_t)kBlockVoxels;
        if (s >= v.capacity) continue;   // absent
        const unsigned long long *m = (const unsigned long long *)v.masks[s].inside;
        unsigned long long any = 0;
#pragma unroll
        for (int y = 0; y < 8; ++y) any |= m[y];
        if (any) return false;
    }
    return true;
}

// The footprint query's march: sets the bit of every allocated block that a
// sample is based in, from the ray's depth span's start to the crossing at
// sample n_hit, where a group takes G samples a step (those of the crossing's
// step count whole) and jumps over the rest of a block that is absent or, with
// its upper neighbours, holds no value at or below zero.
template <int G, bool kDense>
__device__ void mark_blocks(const VolumeView &v, const Ray &r, int n_lo, int n_end, int n_hit, bool active, double h,
                            double inv_h)
{
    const int lane = threadIdx.x & 63, j = lane & (G - 1);
    int n_base = n_lo;
    bool done = !(active && n_lo <= n_end);
    while (__ballot(!done)) {
        double q[3];
        q_at(r, (double)(n_base + j) * h, q);
        int c[3];
        float f[3];
        uint32_t info = kEmptyKey;   // of the last sample, if it decides a jump (bit 30: absent block)
        if (!done && n_base + j <= n_end && stencil(v, q, c, f)) {
            const int bx = c[0] >> 3, by = c[1] >> 3, bz = c[2] >> 3;
            const int32_t slot = block_slot<kDense>(v, bx, by, bz);
            if (slot >= 0) {
                const uint64_t b = block_linear(v, bx, by, bz);
                if (!((v.mark_bits[b >> 5] >> (b & 31)) & 1u)) atomicOr(&v.mark_bits[b >> 5], 1u << (b & 31));
            }
            if (j == G - 1 && (slot < 0 || all_positive(v, slot)))
                info = pack_key(bx, by, bz) | (slot < 0 ? 1u << 30 : 0u);
        }
        info = (uint32_t)__shfl((int)info, group_lane<G>(lane, G - 1));
        if (!done) {
            const int last = n_base + G - 1;
            n_base = last + 1;
            if (info != kEmptyKey) {
                int B[3];
                unpack_key(info, B[0], B[1], B[2]);
                // (the last sample of a positive block can begin a bracket)
                n_base = max(n_base, cell_exit_sample(r, B, 0, h, inv_h) - (info >> 30 ? 0 : 1));
            }
            done = last >= n_hit || n_base > n_end;
        }
    }
}

// Thread `gt` of a launch space of (tiles x 64 rays x G lanes) for one frame.
// kMark: also set the bit of every block a sample up to the crossing is based
// in (the footprint query; the timed raycast is instantiated without it).
template <typename S, int G, bool kDense, bool kMark = false>
__device__ __forceinline__ void raycast_body(const VolumeView &v, const Camera &cam, uint32_t stamp, int tiles_x,
                                             int tiles_y, float4 *__restrict__ vertex, float4 *__restrict__ normal,
                                             long long gt)
{
    static_assert(G >= 1 && G <= 16 && (G & (G - 1)) == 0, "group size");
    const int lane = threadIdx.x & 63;
    const int j = lane & (G - 1);                       // sample slot inside the ray's group
    // rays in 8x8-pixel tile order: 64 consecutive rays form one tile (the
    // launch covers fewer than 2^31 rays)
    const int ray = (int)(gt / G);
    const int tile = ray >> 6;
    const int within = ray & 63;
    const int ti = tile % tiles_x, tj = tile / tiles_x;
    // 16 consecutive rays cover one 4x4-pixel cell of the tile: they share
    // the cell's depth span and mostly the same blocks
    const int cq = within >> 4, k16 = within & 15;
    const int i = ti * kRT + (cq & 1) * 4 + (k16 & 3), jpix = tj * kRT + (cq >> 1) * 4 + (k16 >> 2);
    const bool active = tj < tiles_y && i < cam.width && jpix < cam.height;
    const double h = 0.5 * v.vs, inv_h = 2.0 * v.inv_vs;

    Ray r;
    r.q0 = cam.q0;
#pragma unroll
    for (int a = 0; a < 3; ++a) r.dq[a] = 0.0;
    int n_lo = 1, n_end = 0;   // sample indices (a ray crosses the grid in fewer than 2^31 samples)
    float zmin_t = 0.0f, zmax_t = -1.0f;
    bool near = false;
    if (active) {
        const size_t t = (size_t)tj * tiles_x + ti;
        // the pixel's cell span joined with its tile's (blocks with large footprints)
        const int cw = (cam.width + kCell - 1) / kCell, ch = (cam.height + kCell - 1) / kCell;
        const size_t cell = (size_t)(jpix / kCell) * cw + i / kCell;
        zmin_t = __uint_as_float(min(v.tile_range[t], v.pix_range[cell]));
        zmax_t =
            __uint_as_float(max(v.tile_range[(size_t)tiles_x * tiles_y + t], v.pix_range[(size_t)cw * ch + cell]));
        near = v.state->near_stamp == stamp;
    }
    // a ray with an empty span (and no block at the camera plane) misses
    // without a sample: the ray itself is only set up for the others
    if (active && (near || zmin_t <= zmax_t)) {
        const double dc0 = (i - cam.cx) * cam.inv_fx, dc1 = (jpix - cam.cy) * cam.inv_fy;
        const double len2 = dc0 * dc0 + dc1 * dc1 + 1.0;
        const double inv_len = fast_rsqrt(len2), len = len2 * inv_len;
        double inv[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r.dq[a] = (cam.R[3 * a] * dc0 + cam.R[3 * a + 1] * dc1 + cam.R[3 * a + 2]) * inv_len * v.inv_vs;
            inv[a] = r.dq[a] != 0.0 ? fast_rcp(r.dq[a]) : 0.0;
        }
        // valid samples need every stencil voxel in the grid: q in [0, G-1]
        double s_in = 0.0, s_out = 1e300;
        bool miss = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double hiq = (double)(v.dims[a] - 1);
            if (r.dq[a] == 0.0) {
                miss |= (r.q0[a] < 0.0 || r.q0[a] > hiq);
            } else {
                const double s0 = (0.0 - r.q0[a]) * inv[a], s1 = (hiq - r.q0[a]) * inv[a];
                s_in = fmax(s_in, fmin(s0, s1));
                s_out = fmin(s_out, fmax(s0, s1));
            }
        }
        if (!near) {   // the depth span (camera z = s / len along this ray)
            s_in = fmax(s_in, (double)zmin_t * len);
            s_out = fmin(s_out, (double)zmax_t * len);
        }
        if (!miss && s_in <= s_out) {
            // (a sample more at either end than the span needs: s_in and s_out
            // are products with reciprocals good to a few ulp)
            n_lo = max((int)fmin(floor(s_in * inv_h) - 1.0, 2.0e9), 1);
            n_end = (int)fmin(ceil(s_out * inv_h) + 1.0, 2.0e9);
        }
    }

    // ---- march: per step a group tests the samples n_base .. n_base + kSpan - 1
    // (lane j those at j, j + G, ...), two bits each: whether a bracket can end
    // in the sample's cell and whether one can begin there.  Only where one can
    // end at a sample and begin at the one before (a candidate), the group
    // evaluates F: at the two and (with the lanes left) at the samples after them,
    // and looks for the first crossing; then at the step's next candidate.  An
    // invalid sample carries F = NaN, so every comparison with it fails.
    //
    // A group with candidates evaluates F in the same turn in which the others take
    // a step, and a step's candidates are kept until all are looked at.  Where
    // groups that had found one waited until every group had, a wavefront's rays
    // marched one after the other: in a room scanned from ten sides (1 mm, 640x480,
    // 8 lanes) one wavefront took 197 steps for the 55 of its longest ray, 293 us
    // of a kernel whose others ended by 70; 314 -> 191 us (4 lanes: 417 -> 198).
    //
    // A step is a chain of two dependent loads (block, cell) whatever the
    // number of samples, and the rays of a wavefront wait for the longest:
    // kPerLane samples a lane make the steps fewer.
    constexpr int kPerLane = G >= 16 ? 2 : G == 8 ? 4 : 8;
    constexpr int kSpan = G * kPerLane;   // at most 32: a bit each
    // a step of 32 samples (16 voxels) is longer than the way through a block:
    // only larger empty groups of blocks are worth a jump then
    constexpr bool kJumpBlock = kSpan < 32;
    const float kNaN = __builtin_nanf("");
    BlockCache cache;
    cache.key = kEmptyKey;
#pragma unroll
    for (int k = 0; k < 8; ++k) cache.base[k] = v.capacity * (uint32_t)kBlockVoxels;
    int n_base = n_lo;
    bool done = !(active && n_lo <= n_end);
    bool hit = false;
    bool begin = true;       // whether a bracket can begin at sample n_base - 1 (true: not known)
    uint32_t cand = 0;       // candidates of the step at n_base that are still to be looked at
    double s_lo = 0.0, s_hi = 0.0;
    float F_lo = 0.0f, F_hi = 0.0f;
    while (__ballot(!done)) {
        const bool march = !done && !cand;
        if (__ballot(march)) {
            int32_t slot[kPerLane];
            uint32_t cell[kPerLane];   // column of the cell's low corner | bit << 8
            uint32_t last_key = 0;
            unsigned long long occ0 = 0, occ1 = 0;
            bool inside = false;
#pragma unroll
            for (int k = 0; k < kPerLane; ++k) {
                const int n = n_base + k * G + j;
                double q[3];
                q_at(r, (double)n * h, q);
                int c[3];
                inside = march && n <= n_end;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    c[a] = (int)floor(q[a]);
                    inside &= (uint32_t)c[a] < (uint32_t)(v.dims[a] - 1);
                }
                cell[k] = (uint32_t)((c[0] & 7) | ((c[1] & 7) << 3) | ((c[2] & 7) << 8));
                slot[k] = -1;
                if (inside) {
                    const int bx = c[0] >> 3, by = c[1] >> 3, bz = c[2] >> 3;
                    slot[k] = block_slot<kDense>(v, bx, by, bz);
                    if (k == kPerLane - 1) {
                        last_key = pack_key(bx, by, bz);
                        if (j == G - 1) {
                            occ0 = v.occ[occ_word(v, 0, bx, by, bz)];
                            occ1 = v.occ[occ_word(v, 1, bx, by, bz)];
                        }
                    }
                }
            }
            uint32_t ends = 0, begins = 0, box = 0;
#pragma unroll
            for (int k = 0; k < kPerLane; ++k)
                if (slot[k] >= 0) {
                    const BlockRec *rec = v.recs + slot[k];
                    const uint32_t w = (uint32_t)rec->cell[cell[k] & 63u] >> (cell[k] >> 8);
                    ends |= (w & 1u) << (k * G + j);
                    begins |= ((w >> 8) & 1u) << (k * G + j);
                    if (kJumpBlock && k == kPerLane - 1 && j == G - 1) box = rec->box;
                }
#pragma unroll
            for (int off = 1; off < G; off <<= 1) {
                ends |= (uint32_t)__shfl_xor((int)ends, off);
                begins |= (uint32_t)__shfl_xor((int)begins, off);
            }
            if (march) cand = ends & ((begins << 1) | (begin ? 1u : 0u));
            // (march, begin and the masks are the same in every lane of a group)
            // the group's last sample decides a jump past the cells of its block
            // when no bracket can end there, or of the largest aligned group of
            // blocks around it that is empty (bits 30-31: log4 of its edge)
            const uint32_t skip = inside && (kJumpBlock ? !box : !occ0)
                                      ? last_key | (occ0 ? 0u : occ1 ? 1u << 30 : 2u << 30) : kEmptyKey;
            const uint32_t jump = (uint32_t)__shfl((int)skip, group_lane<G>(lane, G - 1));
            if (march) {
                begin = (begins >> (kSpan - 1)) & 1u;
                if (!cand) {
                    n_base += kSpan;
                    if (jump != kEmptyKey) {
                        int B[3];
                        unpack_key(jump, B[0], B[1], B[2]);
                        const int exit_n = cell_exit_sample(r, B, 2 * (int)(jump >> 30), h, inv_h);
                        if (exit_n > n_base) {
                            n_base = exit_n;
                            begin = true;
                        }
                    }
                    done = n_base > n_end;
                }
            }
        }
        if (!__ballot(cand && !done)) continue;
        // F at the samples from the one before the first candidate on, a lane each
        // (with one lane per ray: two rounds)
        constexpr int kEval = G == 1 ? 2 : G;
        const int c0 = cand ? __builtin_ctz(cand) : 0, n0 = n_base + c0 - 1;
        float F[G == 1 ? 2 : 1];
#pragma unroll
        for (int t = 0; t < (G == 1 ? 2 : 1); ++t) {
            const int k = G == 1 ? t : j, n = n0 + k;
            F[t] = kNaN;
            if (!done && cand && n >= 1 && n <= n_end) {
                double q[3];
                q_at(r, (double)n * h, q);
                F[t] = sample<S, kDense>(v, cache, q);
            }
        }
        int first = 0;   // the crossing ends at sample n0 + first (0: none)
        float Fl, Fh;
        if constexpr (G == 1) {
            first = F[0] > 0.0f && F[1] <= 0.0f ? 1 : 0;
            Fl = F[0];
            Fh = F[1];
        } else {
            const float Fp = __shfl(F[0], group_lane<G>(lane, (j + G - 1) & (G - 1)));
            const unsigned long long m = __ballot(j > 0 && Fp > 0.0f && F[0] <= 0.0f);
            const uint32_t gm = (uint32_t)(m >> (lane & ~(G - 1))) & ((1u << G) - 1u);
            first = gm ? __builtin_ctz(gm) : 0;
            Fl = __shfl(F[0], group_lane<G>(lane, max(first - 1, 0)));
            Fh = __shfl(F[0], group_lane<G>(lane, first));
        }
        if (!done && cand) {
            if (first) {
                s_lo = (double)(n0 + first - 1) * h;
                s_hi = (double)(n0 + first) * h;
                F_lo = Fl;
                F_hi = Fh;
                hit = done = true;
            } else {
                const int next = c0 + kEval - 1;
                cand = next < 32 ? cand >> next << next : 0u;
                if (!cand) {
                    n_base += kSpan;
                    if (n_base > n_end) done = true;
                }
            }
        }
    }

    if constexpr (kMark) mark_blocks<G, kDense>(v, r, n_lo, n_end, hit ? (int)rint(s_hi * inv_h) : 2147483647, active, h, inv_h);

    // ---- refinement: quaternary search inside [s_lo, s_hi] (F_lo > 0 >= F_hi),
    // six steps that shrink the bracket 4096-fold.  Each looks at the 3 inner
    // quarter points (point m by lane m % G of the group, in ceil(3 / G) rounds),
    // so the points and hence the result do not depend on the group size.  Inside
    // one cell F along the ray is a cubic: once a step's bracket lies in one (most
    // rays: the second step's), the steps that are left are taken on the cubic
    // through its points, in registers, by all of the wavefront's rays at once.
    // The cubic only says where to look: F is then evaluated at both ends of its
    // bracket, along with the normal's samples, and where they do not enclose the
    // crossing (a root within rounding of an end) the ray goes on with sampled
    // steps.  The crossing is that of six sampled steps, whatever the cubic's
    // rounding (taken from the cubic, it was off by 1.2 times as much); the
    // normal's samples are placed by the cubic's own, 1e-7 voxel beside it.
    constexpr int kPts = 3, kSteps = 6, kRounds = (kPts + G - 1) / G;
    double a = s_lo, b = s_hi;
    float Fa = F_lo, Fb = F_hi;
    bool refine = hit;                        // takes sampled steps
    bool cubic = false, sampled = false;      // has a cubic to check; does without one
    int left = kSteps;
    // ---- normal: central differences one voxel apart, lanes share the 6 samples
    float g[3] = {0.f, 0.f, 0.f};
    bool ok = false, fresh = hit;             // fresh: its normal is still to be taken
    while (__ballot(fresh)) {
        // the cubic through f0.. at u = 0..3 (Newton's forward differences); the
        // bracket [a, b] is [u0, u0 + 1]
        float f0 = 0.0f, d1 = 0.0f, d2 = 0.0f, d3 = 0.0f, u0 = 0.0f;
        while (__ballot(refine)) {
            float Fp[kPts];
#pragma unroll
            for (int rd = 0; rd < kRounds; ++rd) {
                const int m = rd * G + j;
                float Fm = kNaN;
                if (refine && m < kPts) {
                    double qm[3];
                    q_at(r, a + (b - a) * (double)(m + 1) * 0.25, qm);
                    Fm = sample<S, kDense>(v, cache, qm);
                }
#pragma unroll
                for (int mm = rd * G; mm < (rd + 1) * G && mm < kPts; ++mm)
                    Fp[mm] = __shfl(Fm, group_lane<G>(lane, mm - rd * G));
            }
            if (!refine) continue;
            // an invalid point inside the bracket: keep the bracket
            if (Fp[0] != Fp[0] || Fp[1] != Fp[1] || Fp[2] != Fp[2]) {
                refine = false;
                continue;
            }
            // first non-positive point: the root lies in (point k - 1, point k]
            const bool n0 = Fp[0] <= 0.0f, n1 = Fp[1] <= 0.0f, n2 = Fp[2] <= 0.0f;
            const int k = n0 ? 0 : n1 ? 1 : n2 ? 2 : 3;
            double qa[3], qb[3];
            q_at(r, a, qa);
            q_at(r, b, qb);
            --left;
            cubic = !sampled && left > 0 && floor(qa[0]) == floor(qb[0]) && floor(qa[1]) == floor(qb[1]) &&
                    floor(qa[2]) == floor(qb[2]);
            refine = !cubic && left > 0;
            // the four of the five points around the root's quarter
            const bool upper = k >= 2;
            const float g1 = upper ? Fp[1] : Fp[0], g2 = upper ? Fp[2] : Fp[1], g3 = upper ? Fb : Fp[2];
            f0 = upper ? Fp[0] : Fa;
            d1 = g1 - f0;
            const float e1 = g2 - g1, e2 = g3 - g2, c1 = e1 - d1;
            d2 = 0.5f * c1;
            d3 = ((e2 - e1) - c1) * (1.0f / 6.0f);
            u0 = k == 0 || k == 2 ? (upper ? 1.0f : 0.0f) : (upper ? 2.0f : 1.0f);
            Fb = n0 ? Fp[0] : n1 ? Fp[1] : n2 ? Fp[2] : Fb;
            Fa = n0 ? Fa : n1 ? Fp[0] : n2 ? Fp[1] : Fp[2];
            const double w = (b - a) * 0.25;
            a += w * (double)k;
            b = a + w;
        }
        double ca = a, cb = b;
        float cFa = Fa, cFb = Fb;
        if (__ballot(cubic)) {
            float t = 0.0f, dt = 1.0f;   // the bracket is u0 + [t, t + dt]
            auto P = [&](float u) { return fmaf(u, fmaf(u - 1.0f, fmaf(u - 2.0f, d3, d2), d1), f0); };
#pragma unroll
            for (int st = 0; st < kSteps - 1; ++st) {
                const float q = 0.25f * dt;
                const float p0 = P(u0 + (t + q)), p1 = P(u0 + (t + 2.0f * q)), p2 = P(u0 + (t + 3.0f * q));
                if (st < left) {
                    dt = q;
                    t = fmaf(p0 <= 0.0f ? 0.0f : p1 <= 0.0f ? 1.0f : p2 <= 0.0f ? 2.0f : 3.0f, q, t);
                }
            }
            if (cubic) {
                const double w = b - a;
                ca = a + w * (double)t;
                cb = ca + w * (double)dt;
                cFa = P(u0 + t);
                cFb = P(u0 + (t + dt));
            }
        }
        double qh[3];
        q_at(r, cFa - cFb > 0.0f ? ca + (cb - ca) * ((double)cFa / ((double)cFa - (double)cFb)) : 0.5 * (ca + cb), qh);
        float Fs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) Fs[e] = kNaN;
        // samples {+x, -x, +y, -y, +z, -z} around the crossing and the two ends of
        // the cubic's bracket, sample e by lane e % G of the group.  A lane taking
        // several samples looks up every block before it reads a voxel, so the
        // loads are all in flight together (with one or two lanes per ray the last
        // two samples follow by themselves: 176 VGPRs otherwise).
        constexpr int kFirst = G <= 2 ? 6 : 8, kPer = (kFirst + G - 1) / G;
        int nc[kPer][3];
        float nf[kPer][3];
        bool nin[kPer];
        BlockCache ncache[kPer];
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const int e = j + t * G;
            nin[t] = fresh && (e < 6 || (cubic && e < kFirst));
            ncache[t] = cache;
            if (nin[t]) {
                double qe[3];
                if (e < 6) {
#pragma unroll
                    for (int x = 0; x < 3; ++x) qe[x] = qh[x];
                    qe[e >> 1] += (e & 1) ? -1.0 : 1.0;
                } else {
                    q_at(r, e == 6 ? ca : cb, qe);
                }
                nin[t] = stencil(v, qe, nc[t], nf[t]);
                if (nin[t]) enter_block<kDense>(v, ncache[t], nc[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            float Fv;
            if (nin[t] && interp<S>(v, ncache[t], nc[t], nf[t], Fv)) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e == j + t * G) Fs[e] = Fv;
            }
        }
        if constexpr (kFirst == 6) {
#pragma unroll
            for (int e = 6 + j; e < 8; e += G)
                if (cubic) {
                    double qe[3];
                    q_at(r, e == 6 ? ca : cb, qe);
                    Fs[e] = sample<S, kDense>(v, cache, qe);
                }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) Fs[e] = __shfl(Fs[e], group_lane<G>(lane, e % G));
        if (fresh) {
            refine = cubic && !(Fs[6] > 0.0f && Fs[7] <= 0.0f);
            if (cubic && !refine) {
                a = ca;
                b = cb;
                Fa = Fs[6];
                Fb = Fs[7];
            }
            fresh = sampled = refine;
            cubic = false;
            ok = true;
#pragma unroll
            for (int e = 0; e < 6; ++e) ok = ok && Fs[e] == Fs[e];   // NaN: invalid
            g[0] = Fs[0] - Fs[1];
            g[1] = Fs[2] - Fs[3];
            g[2] = Fs[4] - Fs[5];
        }
    }
    const double sh = hit ? ((Fa - Fb) > 0.0f ? a + (b - a) * ((double)Fa / ((double)Fa - (double)Fb)) : 0.5 * (a + b))
                          : 0.0;
    if (active && j == 0) {
        float4 vout = make_float4(0.f, 0.f, 0.f, 0.f), nout = vout;
        const float gl = sqrtf(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
        if (ok && gl > 0.0f) {
            const double m = sh * v.vs;   // along dq in voxels
            vout = make_float4((float)(cam.t[0] + m * r.dq[0]), (float)(cam.t[1] + m * r.dq[1]),
                               (float)(cam.t[2] + m * r.dq[2]), 1.0f);
            nout = make_float4(g[0] / gl, g[1] / gl, g[2] / gl, 1.0f);
        }
        const size_t pix = (size_t)jpix * cam.width + i;
        vertex[pix] = vout;
        normal[pix] = nout;
    }
}

}  // namespace tsdf

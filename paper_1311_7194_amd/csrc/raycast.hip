// Raycast of the block-sparse TSDF into vertex and normal maps (Section 5).
//
// Each ray (through a pixel centre) is sampled at s_n = n * voxel/2, n >= 1.
// A sample's value F is the trilinear interpolation over the 8 voxel
// centres around it; it is invalid if any of them is outside the grid, in
// an unallocated block or chi.  The hit is the first n with both F(s_n) > 0
// and F(s_{n+1}) <= 0 valid; the bracket is refined to the root and central
// differences one voxel apart give the normal.
//
// Block records and range shrinking.  The paper rasterises the faces of
// occupied blocks into per-pixel start and end textures so that rays only
// traverse the depth span of occupied blocks.  Here a compute pass over the
// allocated blocks in view does more, from two bits per voxel that fusion
// keeps (not chi; at or below zero): it finds the cells where a bracket can
// end (no chi voxel, one at or below zero) and where one can begin (no chi
// voxel, one above zero), stores them with the pool offsets of the block's
// upper neighbours in a record per block, projects the box of the cells of the
// first kind and widens the [min, max] camera depth of every 4x4-pixel cell
// holding a pixel centre the projection may cover (boxes over more than 64
// cells widen whole 8x8-pixel tiles instead).  Every bracket's end lies in
// such a box, so starting and ending each ray at its cell's span (joined with
// its tile's) loses none.
//
// March.  A group of G lanes marches one ray, up to 32 samples per step, and a
// sample costs one bit pair of its block's record instead of its eight voxels:
// F is evaluated only where a bracket can begin at one sample and end at the
// next (1-2 times a ray).  Samples live in voxel-centre coordinates
// q = (x - origin)/voxel - 1/2, where the 8 voxels around a sample are
// floor(q) + {0,1}^3.  When a step finds nothing and its last sample lies in a
// largest empty aligned group of 4^3 or 16^3 blocks, the group jumps past it
// (past a single block without cells where a bracket can end only if its step
// is shorter than 32 samples).
//
// What bounds it: instruction issue and the chains of dependent loads (the
// march's two per step), not bytes.  Evaluating F at every sample of the band
// kept the vector units 80 % busy on the 640x480 orbit (1 mm); with the
// records, a ray's cubic inside a cell in place of most of the refinement's
// dependent steps, and a ray's setup without divisions and square roots in the
// library's form: 263 -> 168 us there (8 lanes per ray, a step of 32 samples),
// 20 -> 17 us at 160x120, 128 -> 94 us on the 1280x960 hand (0.15 mm, 4 lanes;
// 78 us from a list of its tiles, see kListGrid), 188 -> 67 us with the hash only
// (4 mm, FP16).  The records make the range pass longer (eight neighbour lookups
// for each block in view: 34 -> 49 us at 640x480, 6.8 -> 11 us at 160x120), which
// the march repays also where few rays look at many blocks: views of 16x12 to
// 640x480 pixels of a room scanned from ten sides (253,000 blocks, 1 mm), from
// far away, from its side and from inside, take 155-328 us without them and
// 40-271 us with them.
#include "raycast_device.h"

namespace tsdf {

__global__ void range_clear_kernel(VolumeView v, int tiles_x, int tiles_y, int width, int height)
{
    range_clear_body(v, tiles_x, tiles_y, width, height, (long long)blockIdx.x * blockDim.x + threadIdx.x);
}

template <bool kDense>
__global__ __launch_bounds__(256) void range_kernel(VolumeView v, Camera cam, uint32_t stamp, int tiles_x,
                                                    int tiles_y)
{
    __shared__ RangeLds L;
    const uint32_t n = min(v.state->pool_count, v.capacity);
    if (blockIdx.x == 0 && threadIdx.x == 0) v.state->long_tiles = v.state->short_tiles = 0;   // for tiles_kernel
    if (blockIdx.x * (uint32_t)kRangeChunk >= n) return;   // (the whole workgroup)
    span_lds_init(L);
    const int cw = (cam.width + kCell - 1) / kCell, ch = (cam.height + kCell - 1) / kCell;
    uint32_t *cmin = v.pix_range, *cmax = v.pix_range + (size_t)cw * ch;
    for (uint32_t first = blockIdx.x * (uint32_t)kRangeChunk; first < n; first += gridDim.x * (uint32_t)kRangeChunk)
        range_chunk<kDense>(v, cam, stamp, tiles_x, tiles_y, first, n, L, [&](uint32_t c, uint32_t zl, uint32_t zh) {
            if (!span_lds_add(L, c, zl, zh)) {
                atomicMin(&cmin[c], zl);   // no return value: the lane does not wait
                atomicMax(&cmax[c], zh);
            }
        });
    for (int e = threadIdx.x; e < kSpanLds; e += 256) {
        const uint32_t c = L.key[e];
        if (c != kSpanEmpty) {
            atomicMin(&cmin[c], L.lo[e]);
            atomicMax(&cmax[c], L.hi[e]);
        }
    }
}

// Footprint query: widens the spans that range_kernel left to those of the
// samples whose voxels may all hold a distance, a lane per allocated block: q in
// the box of the block's non-chi voxels, extended by one voxel upwards.
__global__ __launch_bounds__(256) void footprint_range_kernel(VolumeView v, Camera cam, uint32_t stamp, int tiles_x,
                                                              int tiles_y)
{
    const uint32_t n = min(v.state->pool_count, v.capacity);
    const int cw = (cam.width + kCell - 1) / kCell, ch = (cam.height + kCell - 1) / kCell;
    for (uint32_t slot = blockIdx.x * 256u + threadIdx.x; slot < n; slot += gridDim.x * 256u) {
        const uint32_t key = v.pool_keys[slot];
        if (key == kEmptyKey) continue;
        const unsigned long long *m = (const unsigned long long *)v.masks[slot].value;
        unsigned long long all = 0;
        uint32_t xb = 0, yb = 0, zb = 0;
        for (int y = 0; y < 8; ++y) {
            all |= m[y];
            yb |= (m[y] ? 1u : 0u) << y;
        }
        if (!all) continue;
        for (int x = 0; x < 8; ++x) {
            const uint32_t col = (uint32_t)(all >> (8 * x)) & 0xffu;
            xb |= (col ? 1u : 0u) << x;
            zb |= col;
        }
        const int lo[3] = {__builtin_ctz(xb), __builtin_ctz(yb), __builtin_ctz(zb)};
        const int hi[3] = {32 - __builtin_clz(xb), 32 - __builtin_clz(yb), 32 - __builtin_clz(zb)};
        int bx, by, bz;
        unpack_key(key, bx, by, bz);
        const BoxView w = project_box(v, cam, bx, by, bz, lo, hi);
        if (!w.visible) continue;
        if (w.behind) {
            v.state->near_stamp = stamp;
            continue;
        }
        const uint32_t zl = __float_as_uint(fmaxf(w.zlo * (1.0f - 1e-5f) - 1e-6f, 0.0f));
        const uint32_t zh = __float_as_uint(w.zhi * (1.0f + 1e-5f) + 1e-6f);
        int c0 = w.i0 / kCell, c1 = w.i1 / kCell, d0 = w.j0 / kCell, d1 = w.j1 / kCell, width = cw;
        uint32_t *smin = v.pix_range, *smax = smin + (size_t)cw * ch;
        if ((c1 - c0 + 1) * (d1 - d0 + 1) > kCellFootprint) {   // large: whole tiles
            c0 = w.i0 / kRT, c1 = w.i1 / kRT, d0 = w.j0 / kRT, d1 = w.j1 / kRT, width = tiles_x;
            smin = v.tile_range, smax = smin + (size_t)tiles_x * tiles_y;
        }
        for (int d = d0; d <= d1; ++d)
            for (int c = c0; c <= c1; ++c) {
                atomicMin(&smin[(size_t)d * width + c], zl);
                atomicMax(&smax[(size_t)d * width + c], zh);
            }
    }
}

// Sorts the frame's 8x8-pixel tiles, kTilesPerGroup to a workgroup: a tile without a depth
// span is background, and its part of the maps is cleared here; the others go to
// the tile list, those with a long span at its front (their rays march longest
// and must not start last), the rest from its back.
// (hand at 1280x960, 8 lanes: 62 us with the line at 80 voxels, 75 at 20 or 320
// and without one)
constexpr int kTilesPerGroup = 16;
constexpr float kLongSpan = 80.0f;   // voxels

__global__ __launch_bounds__(256) void tiles_kernel(VolumeView v, int width, int height, uint32_t stamp, int tiles_x,
                                                    int n_tiles, float4 *__restrict__ vertex,
                                                    float4 *__restrict__ normal)
{
    __shared__ unsigned long long empty;
    const int tid = threadIdx.x, lane = tid & 63;
    const int first = blockIdx.x * kTilesPerGroup;
    if (tid < kTilesPerGroup) {   // in one wavefront
        const int tile = first + lane;
        const bool valid = tile < n_tiles;
        bool any = false, is_long = false;
        if (valid) {
            const bool near = v.state->near_stamp == stamp;
            const int cw = (width + kCell - 1) / kCell, ch = (height + kCell - 1) / kCell;
            const int ci = (tile % tiles_x) * kCellsPerTile, cj = (tile / tiles_x) * kCellsPerTile;
            const uint32_t tlo = v.tile_range[tile], thi = v.tile_range[(size_t)n_tiles + tile];
            any = is_long = near;
#pragma unroll
            for (int q = 0; q < kCellsPerTile * kCellsPerTile; ++q) {
                // (a border tile's missing cells: its last ones again)
                const size_t c = (size_t)min(cj + q / kCellsPerTile, ch - 1) * cw +
                                 (size_t)min(ci + q % kCellsPerTile, cw - 1);
                const float lo = __uint_as_float(min(tlo, v.pix_range[c]));
                const float hi = __uint_as_float(max(thi, v.pix_range[(size_t)cw * ch + c]));
                any |= lo <= hi;
                is_long |= hi - lo > kLongSpan * (float)v.vs;
            }
        }
        const unsigned long long ml = __ballot(any && is_long), ms = __ballot(any && !is_long),
                                 me = __ballot(valid && !any);
        uint32_t bl = 0, bs = 0;
        if (lane == 0) {
            if (ml) bl = atomicAdd(&v.state->long_tiles, (uint32_t)__popcll(ml));
            if (ms) bs = atomicAdd(&v.state->short_tiles, (uint32_t)__popcll(ms));
            empty = me;
        }
        bl = (uint32_t)__shfl((int)bl, 0);
        bs = (uint32_t)__shfl((int)bs, 0);
        const unsigned long long below = (1ull << lane) - 1ull;
        const uint32_t at = is_long ? bl + (uint32_t)__popcll(ml & below)
                                    : (uint32_t)n_tiles - 1u - (bs + (uint32_t)__popcll(ms & below));
        // (in range unless two raycasts of one volume run at once, which is the caller's error)
        if (any && at < (uint32_t)n_tiles) v.tile_list[at] = (uint32_t)tile;
    }
    __syncthreads();
    // background: a wavefront per tile, a lane per pixel
    unsigned long long rest = empty;
    for (int k = 0; rest; ++k) {
        const int tile = first + __builtin_ctzll(rest);
        rest &= rest - 1ull;
        if ((k & 3) != (tid >> 6)) continue;
        const int i = (tile % tiles_x) * kRT + (lane & 7), jpix = (tile / tiles_x) * kRT + (lane >> 3);
        if (i < width && jpix < height) {
            const size_t pix = (size_t)jpix * width + i;
            vertex[pix] = make_float4(0.f, 0.f, 0.f, 0.f);
            normal[pix] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

// One wavefront per workgroup: march lengths differ widely between
// wavefronts (most rays of a frame march little or not at all), and a CU
// takes a new workgroup only where all of its wavefronts fit, so single-wave
// workgroups keep the SIMDs fuller (1280x960 hand sequence: 141 -> 124 us
// at 4 lanes per ray; 640x480 orbit: 284 -> 246 us, now at 8 lanes per ray).
constexpr int kRayWG = 64;

// March from a tile list.  A wavefront takes 1.2 us to find that its tile is
// background, G of them a tile, and the list starts the tiles with long depth
// spans first; it costs a launch of 9 us and wavefronts that take several tiles
// each.  What it gives depends on the scene, which the host does not know, so a
// frame of at least a volume's list_tiles takes it: kListTiles until
// tsdf_autotune_raycast has timed both forms on a view.  Raycast with the list
// and without, us (G lanes per ray; hand: nine tiles in ten background, orbit:
// under half):
//   1280x960 (19200 tiles)  hand    79 / 94 (G = 4)    62 / 95 (G = 8)
//                           orbit  411 / 394, 332 / 310, 293 / 262 (1, 2, 4 mm, G = 4)
//                                  499 / 481, 435 / 407, 396 / 366 (the same, G = 8)
//   640x480 (4800 tiles)    hand    71 / 69            48 / 52
//                           orbit  153 / 167, 119 / 121, 106 / 92 (1, 2, 4 mm, G = 4)
//                                  162 / 166, 137 / 132, 126 / 112 (the same, G = 8)
// Large frames lose up to 11 % one way and a third the other, so they take the
// list by default; smaller ones gain or lose a tenth, and do not.
//
// kListGrid workgroups stride over the list: with 16384 the full frames took
// 543 us (1 mm, G = 8) for 499, with one each the hand's took 67 for 62.
constexpr uint32_t kListGrid = 65536;   // a multiple of 8 * 16

enum MarchMode { kMarchAll, kMarchMark, kMarchList };

// From the list four wavefronts a SIMD for the loop's few registers more (hand,
// 8 lanes: 70 -> 62 us), but not with the 1 or 2 lanes per ray that would spill
// for it (210 us, 188 without, at 1 lane).
template <typename S, int G, bool kDense, MarchMode kMode>
__global__ __launch_bounds__(kRayWG) __attribute__((amdgpu_waves_per_eu(kMode == kMarchList && G >= 4 ? 4 : 1))) void raycast_kernel(
    VolumeView v, Camera cam, uint32_t stamp, int tiles_x, int tiles_y, float4 *__restrict__ vertex,
    float4 *__restrict__ normal)
{
    // Workgroups are dealt to the 8 XCDs in turn.  With up to 4 lanes per ray
    // the G wavefronts of a tile go to one XCD, where they read the same
    // blocks through its L2, and neighbouring tiles to different ones (the
    // grid is then a multiple of 8 G): 124 -> 120 us on the 1280x960 hand
    // sequence at 4 lanes.  At 8 lanes the plain order measured faster.
    uint32_t wg = blockIdx.x;
    if constexpr (G <= 4) {
        const uint32_t grp = blockIdx.x / (8u * G), r = blockIdx.x % (8u * G);
        wg = grp * (8u * G) + (r & 7u) * G + (r >> 3);
    }
    if constexpr (kMode == kMarchList) {
        const uint32_t n_tiles = (uint32_t)(tiles_x * tiles_y), n_long = min(v.state->long_tiles, n_tiles);
        const uint32_t n = min(n_long + v.state->short_tiles, n_tiles);
        for (uint32_t t = wg / G; t < n; t += gridDim.x / G) {
            const uint32_t tile = v.tile_list[t < n_long ? t : n_tiles - 1u - (t - n_long)];
            raycast_body<S, G, kDense, false>(v, cam, stamp, tiles_x, tiles_y, vertex, normal,
                                              ((long long)tile * G + wg % G) * kRayWG + threadIdx.x);
        }
    } else {
        raycast_body<S, G, kDense, kMode == kMarchMark>(v, cam, stamp, tiles_x, tiles_y, vertex, normal,
                                                        (long long)wg * kRayWG + threadIdx.x);
    }
}

template <typename S, bool kDense, MarchMode kMode>
static void launch_group(int G, dim3 grid, hipStream_t s, const VolumeView &v, const Camera &cam, uint32_t stamp,
                         int tx, int ty, float4 *vertex, float4 *normal)
{
    switch (G) {
    case 1: hipLaunchKernelGGL((raycast_kernel<S, 1, kDense, kMode>), grid, dim3(kRayWG), 0, s, v, cam, stamp, tx, ty, vertex, normal); break;
    case 2: hipLaunchKernelGGL((raycast_kernel<S, 2, kDense, kMode>), grid, dim3(kRayWG), 0, s, v, cam, stamp, tx, ty, vertex, normal); break;
    case 4: hipLaunchKernelGGL((raycast_kernel<S, 4, kDense, kMode>), grid, dim3(kRayWG), 0, s, v, cam, stamp, tx, ty, vertex, normal); break;
    case 16: hipLaunchKernelGGL((raycast_kernel<S, 16, kDense, kMode>), grid, dim3(kRayWG), 0, s, v, cam, stamp, tx, ty, vertex, normal); break;
    default: hipLaunchKernelGGL((raycast_kernel<S, 8, kDense, kMode>), grid, dim3(kRayWG), 0, s, v, cam, stamp, tx, ty, vertex, normal); break;
    }
}

template <typename S, bool kDense>
static void launch_group(MarchMode mode, int G, dim3 grid, hipStream_t s, const VolumeView &v, const Camera &cam,
                         uint32_t stamp, int tx, int ty, float4 *vertex, float4 *normal)
{
    if (mode == kMarchMark) launch_group<S, kDense, kMarchMark>(G, grid, s, v, cam, stamp, tx, ty, vertex, normal);
    else if (mode == kMarchList) launch_group<S, kDense, kMarchList>(G, grid, s, v, cam, stamp, tx, ty, vertex, normal);
    else launch_group<S, kDense, kMarchAll>(G, grid, s, v, cam, stamp, tx, ty, vertex, normal);
}

hipError_t launch_range(const VolumeView &v, const Camera &cam, uint32_t stamp, hipStream_t s)
{
    const int tiles_x = (cam.width + kRT - 1) / kRT, tiles_y = (cam.height + kRT - 1) / kRT;
    const int n_tiles = tiles_x * tiles_y;
    hipLaunchKernelGGL(range_clear_kernel, dim3((n_tiles * 64 + 255) / 256), dim3(256), 0, s, v, tiles_x, tiles_y,
                       cam.width, cam.height);
    // range pass over the allocated blocks (grid-stride; the block count stays on the device)
    if (v.block_index)
        hipLaunchKernelGGL(range_kernel<true>, dim3(2048), dim3(256), 0, s, v, cam, stamp, tiles_x, tiles_y);
    else
        hipLaunchKernelGGL(range_kernel<false>, dim3(2048), dim3(256), 0, s, v, cam, stamp, tiles_x, tiles_y);
    return hipGetLastError();
}

hipError_t launch_footprint_range(const VolumeView &v, const Camera &cam, uint32_t stamp, hipStream_t s)
{
    hipLaunchKernelGGL(footprint_range_kernel, dim3(1024), dim3(256), 0, s, v, cam, stamp, (cam.width + kRT - 1) / kRT,
                       (cam.height + kRT - 1) / kRT);
    return hipGetLastError();
}

hipError_t launch_march(const VolumeView &v, const Camera &camera, uint32_t stamp, int group, int list_tiles,
                        float4 *vertex, float4 *normal, hipStream_t s, bool mark)
{
    Camera cam = camera;
    set_ray_origin(cam, v);
    const int tiles_x = (cam.width + kRT - 1) / kRT, tiles_y = (cam.height + kRT - 1) / kRT;
    const int G = (group == 1 || group == 2 || group == 4 || group == 16) ? group : 8;
    const long long threads = (long long)tiles_x * tiles_y * 64 * G;
    const long long unit = (G <= 4 ? 8LL * G : 1LL) * kRayWG;   // whole groups of 8 tiles' wavefronts
    dim3 grid((unsigned)((threads + unit - 1) / unit * (unit / kRayWG)));
    MarchMode mode = mark ? kMarchMark : kMarchAll;
    const int n_tiles = tiles_x * tiles_y;
    if (!mark && n_tiles >= list_tiles) {
        mode = kMarchList;
        grid = dim3(grid.x < kListGrid ? grid.x : kListGrid);
        hipLaunchKernelGGL(tiles_kernel, dim3((n_tiles + kTilesPerGroup - 1) / kTilesPerGroup), dim3(256), 0, s, v,
                           cam.width, cam.height, stamp, tiles_x, n_tiles, vertex, normal);
    }
    const bool dense = v.block_index != nullptr;
    if (v.storage == TSDF_F16) {
        if (dense) launch_group<__half, true>(mode, G, grid, s, v, cam, stamp, tiles_x, tiles_y, vertex, normal);
        else launch_group<__half, false>(mode, G, grid, s, v, cam, stamp, tiles_x, tiles_y, vertex, normal);
    } else {
        if (dense) launch_group<float, true>(mode, G, grid, s, v, cam, stamp, tiles_x, tiles_y, vertex, normal);
        else launch_group<float, false>(mode, G, grid, s, v, cam, stamp, tiles_x, tiles_y, vertex, normal);
    }
    return hipGetLastError();
}

// Number of set bits of a bitmap, added to the device state's footprint field.
__global__ __launch_bounds__(256) void count_bits_kernel(const uint32_t *__restrict__ bits, uint64_t words,
                                                         unsigned long long *__restrict__ out)
{
    unsigned long long c = 0;
    for (uint64_t w = (uint64_t)blockIdx.x * 256 + threadIdx.x; w < words; w += (uint64_t)gridDim.x * 256)
        c += (unsigned long long)__popc(bits[w]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(out, c);
}

hipError_t launch_count_bits(const uint32_t *bits, uint64_t words, unsigned long long *out, hipStream_t s)
{
    hipLaunchKernelGGL(count_bits_kernel, dim3(1024), dim3(256), 0, s, bits, words, out);
    return hipGetLastError();
}

}  // namespace tsdf

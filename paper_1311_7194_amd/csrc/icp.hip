// Point-to-plane ICP iteration on raycast maps (Section 6); tsdf_icp.h
// documents the steps.
//
//   icp_pairs_kernel  one pass over the live pixels: live point and normal,
//                     projective match into the model maps, rejection, and
//                     per-thread sums of the unscaled normal equations and the
//                     box of the kept points; workgroups write partial sums
//   icp_solve_kernel  one workgroup adds the partials; its first wavefront
//                     forms the scaled system from the unscaled sums, eigen-
//                     decomposes it, keeps the directions above the threshold,
//                     and composes the pose, one matrix entry per lane
//
// Every step of the matching is evaluated in double precision without
// contractions, in a fixed operation order, so that which pixel a point
// matches and whether a pair is kept are decided exactly as the defined
// expressions decide them.
#include <math.h>

#include <mutex>

#include <hip/hip_runtime.h>

#include "tsdf_icp.h"

static_assert(sizeof(tsdf_icp_result) == 600 && sizeof(tsdf_icp_params) == 32, "ICP records in tsdf_icp.h");

namespace tsdf {
namespace {

constexpr int kIcpThreads = 256;
constexpr int kIcpMaxGroups = 512;
// Per-workgroup partials, stored value-major ([kPartial][groups]):
//   0..20 upper triangle of sum g g^T, g = (p x n, n); 21..26 sum g e;
//   27 sum e^2; 28 pair count; 29..31 zero;
//   32..34 -min and 35..37 max of the kept p and q per axis; 38, 39 unused.
constexpr int kPartial = 40;

struct IcpArgs {
    double Rm[9], tm[3];       // model pose, camera to world
    double fx, fy, cx, cy;
    int32_t width, height;
    double dist2;              // dist_max^2
    double cos2;               // cos_min^2
    double theta;
    int32_t shrink;
    double P0[12];             // current pose when the kernels get no device pose
};

// The current pose estimate: the device record or, for a chain's first
// iteration, the host pose passed in the kernel arguments.
__device__ __forceinline__ double pose_at(const double *pose, const IcpArgs &a, int q)
{
    return pose ? pose[q] : a.P0[q];
}

__device__ __forceinline__ bool depth_ok(float d) { return d > 0.0f && isfinite(d); }

struct ReduceLds {
    double s[kIcpThreads / 64][32];
    double x[kIcpThreads / 64][8];
    double tot[kPartial];
};

// Workgroup reduction of 32 sums and 8 maxima per lane into L.tot (visible
// to every thread on return).  Within a wavefront, recursive halving: at
// each exchange a lane keeps one half of its values and sends the other, so
// the sums take 32 exchanges instead of 6 per value.  Afterwards lanes 2m and
// 2m + 1 hold the wavefront's total of sum m, and lanes 8m..8m + 7 its
// maximum m.
__device__ __forceinline__ void block_reduce(const double s[32], const double x[8], ReduceLds &L)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
    double h16[16], h8[8], h4[4], h2[2];
#pragma unroll
    for (int k = 0; k < 16; ++k) h16[k] = (b5 ? s[k + 16] : s[k]) + __shfl_xor(b5 ? s[k] : s[k + 16], 32);
#pragma unroll
    for (int k = 0; k < 8; ++k) h8[k] = (b4 ? h16[k + 8] : h16[k]) + __shfl_xor(b4 ? h16[k] : h16[k + 8], 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) h4[k] = (b3 ? h8[k + 4] : h8[k]) + __shfl_xor(b3 ? h8[k] : h8[k + 4], 8);
#pragma unroll
    for (int k = 0; k < 2; ++k) h2[k] = (b2 ? h4[k + 2] : h4[k]) + __shfl_xor(b2 ? h4[k] : h4[k + 2], 4);
    double h1 = (b1 ? h2[1] : h2[0]) + __shfl_xor(b1 ? h2[0] : h2[1], 2);
    h1 += __shfl_xor(h1, 1);
    if (!(lane & 1)) L.s[wave][lane >> 1] = h1;
    double g4[4], g2[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) g4[k] = fmax(b5 ? x[k + 4] : x[k], __shfl_xor(b5 ? x[k] : x[k + 4], 32));
#pragma unroll
    for (int k = 0; k < 2; ++k) g2[k] = fmax(b4 ? g4[k + 2] : g4[k], __shfl_xor(b4 ? g4[k] : g4[k + 2], 16));
    double g1 = fmax(b3 ? g2[1] : g2[0], __shfl_xor(b3 ? g2[0] : g2[1], 8));
    g1 = fmax(g1, __shfl_xor(g1, 4));
    g1 = fmax(g1, __shfl_xor(g1, 2));
    g1 = fmax(g1, __shfl_xor(g1, 1));
    if (!(lane & 7)) L.x[wave][lane >> 3] = g1;
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 32)
        L.tot[t] = (L.s[0][t] + L.s[1][t]) + (L.s[2][t] + L.s[3][t]);
    else if (t < kPartial)
        L.tot[t] = fmax(fmax(L.x[0][t - 32], L.x[1][t - 32]), fmax(L.x[2][t - 32], L.x[3][t - 32]));
    __syncthreads();
}

__device__ __forceinline__ void init_acc(double s[32], double x[8])
{
#pragma unroll
    for (int k = 0; k < 32; ++k) s[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = -INFINITY;
}

__global__ __launch_bounds__(kIcpThreads) void icp_pairs_kernel(const float *__restrict__ depth,
                                                                const float4 *__restrict__ mvert,
                                                                const float4 *__restrict__ mnorm,
                                                                const double *__restrict__ pose, IcpArgs a,
                                                                double *__restrict__ partial)
{
#pragma clang fp contract(off)
    __shared__ ReduceLds L;
    const int W = a.width, H = a.height;
    double Rc[9], tc[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int c = 0; c < 3; ++c) Rc[3 * r + c] = pose_at(pose, a, 4 * r + c);
        tc[r] = pose_at(pose, a, 4 * r + 3);
    }
    double v[32], bx[8];
    init_acc(v, bx);
    const uint32_t npix = (uint32_t)W * (uint32_t)H;   // at most 16384^2 < 2^32
    const uint32_t stride = gridDim.x * kIcpThreads;
    const uint32_t first = blockIdx.x * kIcpThreads + threadIdx.x;
    // the next pixel's depths are loaded while a pixel waits for its model
    // vertex (indices clamped into the map: what lies past it is not used)
    auto load = [&](uint32_t pix, float d[3]) {
        const uint32_t last = npix - 1u;
        d[0] = depth[min(pix, last)];
        d[1] = depth[min(pix + 1u, last)];
        d[2] = depth[min(pix + (uint32_t)W, last)];
    };
    float next[3];
    load(first, next);
    for (uint32_t pix = first; pix < npix; pix += stride) {
        const float d0 = next[0], dr = next[1], dd = next[2];
        load(pix + stride, next);
        const int j = (int)(pix / (uint32_t)W), i = (int)(pix - (uint32_t)j * (uint32_t)W);
        if (i + 1 >= W || j + 1 >= H) continue;
        if (!(depth_ok(d0) && depth_ok(dr) && depth_ok(dd))) continue;
        // live point and its neighbours through the pixel centres, camera frame
        const double ui = ((double)i - a.cx) / a.fx, ui1 = ((double)(i + 1) - a.cx) / a.fx;
        const double vj = ((double)j - a.cy) / a.fy, vj1 = ((double)(j + 1) - a.cy) / a.fy;
        const double D0 = d0, Dr = dr, Dd = dd;
        const double x0[3] = {ui * D0, vj * D0, D0};
        const double right[3] = {ui1 * Dr - x0[0], vj * Dr - x0[1], Dr - x0[2]};
        const double down[3] = {ui * Dd - x0[0], vj1 * Dd - x0[1], Dd - x0[2]};
        const double nc[3] = {down[1] * right[2] - down[2] * right[1], down[2] * right[0] - down[0] * right[2],
                              down[0] * right[1] - down[1] * right[0]};
        double p[3], nw[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            p[r] = ((Rc[3 * r] * x0[0] + Rc[3 * r + 1] * x0[1]) + Rc[3 * r + 2] * x0[2]) + tc[r];
            nw[r] = (Rc[3 * r] * nc[0] + Rc[3 * r + 1] * nc[1]) + Rc[3 * r + 2] * nc[2];
        }
        // projective match in the model camera
        const double e0 = p[0] - a.tm[0], e1 = p[1] - a.tm[1], e2 = p[2] - a.tm[2];
        const double xm = (a.Rm[0] * e0 + a.Rm[3] * e1) + a.Rm[6] * e2;
        const double ym = (a.Rm[1] * e0 + a.Rm[4] * e1) + a.Rm[7] * e2;
        const double zm = (a.Rm[2] * e0 + a.Rm[5] * e1) + a.Rm[8] * e2;
        if (!(zm > 0.0)) continue;
        const double fu = floor(a.fx * xm / zm + a.cx + 0.5), fv = floor(a.fy * ym / zm + a.cy + 0.5);
        if (!(fu >= 0.0 && fu < (double)W && fv >= 0.0 && fv < (double)H)) continue;
        const long long m = (long long)fv * W + (long long)fu;
        const float4 V = mvert[m], N = mnorm[m];   // in flight together
        if (!(V.w > 0.0f)) continue;
        const double q[3] = {V.x, V.y, V.z}, n[3] = {N.x, N.y, N.z};
        // rejection: distance, then normal deviation
        const double dq[3] = {p[0] - q[0], p[1] - q[1], p[2] - q[2]};
        if (!((dq[0] * dq[0] + dq[1] * dq[1]) + dq[2] * dq[2] <= a.dist2)) continue;
        const double dot = (nw[0] * n[0] + nw[1] * n[1]) + nw[2] * n[2];
        const double nn = (nw[0] * nw[0] + nw[1] * nw[1]) + nw[2] * nw[2];
        const double mm = (n[0] * n[0] + n[1] * n[1]) + n[2] * n[2];
        if (!(dot > 0.0 && dot * dot >= a.cos2 * (nn * mm))) continue;
        // the pair's rows of the normal equations: g = (p x n, n), e = (p - q) . n
        const double g[6] = {p[1] * n[2] - p[2] * n[1], p[2] * n[0] - p[0] * n[2], p[0] * n[1] - p[1] * n[0],
                             n[0], n[1], n[2]};
        const double e = (dq[0] * n[0] + dq[1] * n[1]) + dq[2] * n[2];
        int k = 0;
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int c = r; c < 6; ++c) v[k++] += g[r] * g[c];
#pragma unroll
        for (int r = 0; r < 6; ++r) v[21 + r] += g[r] * e;
        v[27] += e * e;
        v[28] += 1.0;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            bx[r] = fmax(bx[r], fmax(-p[r], -q[r]));
            bx[3 + r] = fmax(bx[3 + r], fmax(p[r], q[r]));
        }
    }
    block_reduce(v, bx, L);
    if (threadIdx.x < kPartial) partial[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = L.tot[threadIdx.x];
}

// Orders a wavefront's LDS accesses (data passed between its lanes).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Plane rotation that zeroes apq: t = tan of its angle from the tangent formula
// in single precision (1e-7) and two Newton steps of t^2 + 2 th t - 1 = 0 with
// FP64 residuals (1e-14, then rounding), c = 1/sqrt(1 + t^2) and s = t c to
// rounding, so that it is orthogonal whatever the accuracy of t.  The chain of
// FP64 latencies is what a sweep costs; the steps' slope is good enough in
// FP32.  Residual |C x - b| / |C| |x| over random systems, median: 8.4e-16 with
// one step, 1.9e-16 with two.
__device__ __forceinline__ void plane_rotation(double app, double aqq, double apq, double &c, double &s, double &t)
{
    double q = __builtin_amdgcn_rcp(apq);
    q = fma(q, fma(-apq, q, 1.0), q);
    q = fma(q, fma(-apq, q, 1.0), q);
    // th = (aqq - app) / (2 apq), t = sign(th) / (|th| + sqrt(th^2 + 1)) (zero in
    // single precision past 1e19: the first step then gives 1 / (2 th)); beyond
    // 1e30 the rotation is the identity
    const double th = 0.5 * (aqq - app) * q;
    const float tf = (float)th, at = fabsf(tf);
    const float t0 = copysignf(__builtin_amdgcn_rcpf(at + __builtin_amdgcn_sqrtf(fmaf(at, at, 1.0f))), tf);
    const double slope = (double)(0.5f * __builtin_amdgcn_rcpf(t0 + tf));
    t = (double)t0;
#pragma unroll
    for (int k = 0; k < 2; ++k) t = fma(-fma(t, fma(2.0, th, t), -1.0), slope, t);
    if (!(fabs(th) < 1e30) || apq == 0.0) t = 0.0;   // (also an undefined th)
    const double x = fma(t, t, 1.0);
    const double y = (double)__builtin_amdgcn_rsqf((float)x);
    const double e = fma(-x * y, y, 1.0);            // 1 - x y^2, about 1e-7
    c = fma(y * e, fma(0.375, e, 0.5), y);           // to e^3
    s = t * c;
}

// Cyclic Jacobi for a symmetric 6x6 matrix on one wavefront.  Every lane holds
// the whole matrix (its upper triangle) and lane r < 6 row r of the
// eigenvector matrix V: nothing is exchanged between lanes.  A sweep is five
// rounds of three disjoint plane rotations: in round k the index x5 = 3k mod 5
// pairs with 5 and the others as (x5 + 1, x5 + 4) and (x5 + 2, x5 + 3) mod 5,
// which covers all 15 pairs.  Disjoint rotations commute and do not touch each
// other's 2x2 blocks, so their chains overlap: A <- J^T A J, V <- V J.
struct Sym6 {
    double a[6][6];   // upper triangle (fully unrolled: registers)
    __device__ __forceinline__ double &operator()(int r, int c) { return r <= c ? a[r][c] : a[c][r]; }
};

template <int kRound>
__device__ __forceinline__ void jacobi_round(Sym6 &A, double v[6])
{
    constexpr int x5 = (3 * kRound) % 5;
    constexpr int P[3] = {x5, (x5 + 1) % 5 < (x5 + 4) % 5 ? (x5 + 1) % 5 : (x5 + 4) % 5,
                          (x5 + 2) % 5 < (x5 + 3) % 5 ? (x5 + 2) % 5 : (x5 + 3) % 5};
    constexpr int Q[3] = {5, (x5 + 1) % 5 < (x5 + 4) % 5 ? (x5 + 4) % 5 : (x5 + 1) % 5,
                          (x5 + 2) % 5 < (x5 + 3) % 5 ? (x5 + 3) % 5 : (x5 + 2) % 5};
    double c[3], s[3], t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) plane_rotation(A(P[i], P[i]), A(Q[i], Q[i]), A(P[i], Q[i]), c[i], s[i], t[i]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int p = P[i], q = Q[i];
        A(p, p) = fma(-t[i], A(p, q), A(p, p));
        A(q, q) = fma(t[i], A(p, q), A(q, q));
        if (t[i] != 0.0) A(p, q) = 0.0;
#pragma unroll
        for (int k = i + 1; k < 3; ++k) {   // the block against another pair
            const int f = P[k], g = Q[k];
            const double pf = A(p, f), pg = A(p, g), qf = A(q, f), qg = A(q, g);
            const double rpf = c[i] * pf - s[i] * qf, rpg = c[i] * pg - s[i] * qg;
            const double rqf = s[i] * pf + c[i] * qf, rqg = s[i] * pg + c[i] * qg;
            A(p, f) = c[k] * rpf - s[k] * rpg;
            A(p, g) = s[k] * rpf + c[k] * rpg;
            A(q, f) = c[k] * rqf - s[k] * rqg;
            A(q, g) = s[k] * rqf + c[k] * rqg;
        }
        const double vp = v[p], vq = v[q];
        v[p] = c[i] * vp - s[i] * vq;
        v[q] = s[i] * vp + c[i] * vq;
    }
}

// Called by the 64 lanes of one wavefront; sA and sV0 (read) and sV, sLam
// (written) in LDS.  sV0 is the rotation the sweeps start from: null for the
// identity, or an orthogonal V0 when sA holds V0^T A V0, so that the
// eigenvectors come out for A itself.
__device__ void jacobi6_wave(const double *sA, const double *sV0, double *sV, double *sLam)
{
    const int lane = threadIdx.x & 63, r = lane < 6 ? lane : 0;
    Sym6 A;
    double v[6];
#pragma unroll
    for (int p = 0; p < 6; ++p) {
#pragma unroll
        for (int q = p; q < 6; ++q) A(p, q) = sA[6 * p + q];
        v[p] = sV0 ? sV0[6 * r + p] : (p == r ? 1.0 : 0.0);
    }
    for (int sweep = 0; sweep < 64; ++sweep) {
        double off = 0.0, diag = 0.0;
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            diag = fma(A(p, p), A(p, p), diag);
#pragma unroll
            for (int q = p + 1; q < 6; ++q) off = fma(A(p, q), A(p, q), off);
        }
        // off-diagonal norm below 1e-13 of the diagonal's (the same in every lane)
        if (!(__builtin_amdgcn_readfirstlane(off > 1e-26 * diag))) break;
        jacobi_round<0>(A, v);
        jacobi_round<1>(A, v);
        jacobi_round<2>(A, v);
        jacobi_round<3>(A, v);
        jacobi_round<4>(A, v);
    }
    if (lane < 6) {
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            sV[6 * lane + p] = v[p];
            if (p == lane) sLam[p] = A(p, p);
        }
    }
    wave_sync();
}

// Scratch of the solve kernel.
struct SolveLds {
    double tot[kPartial];           // the reduced sums and maxima
    double A[36], b[6];             // the system solved (scaled when shrink is set)
    double V0[36], B[36];           // warm start: previous eigenvectors, V0^T A V0
    double V[36], lam[6];           // eigenvectors (columns) and eigenvalues
    double w[6], xh[6];             // coefficients of the kept directions, solution
    double sc[6];                   // sines and cosines of the increment's angles
    double P[12];                   // the current pose
};

// Entry (r, c) of the 6x6 sum g g^T from its upper triangle.
__device__ __forceinline__ double sum_gg(const double *tot, int r, int c)
{
    const int i = min(r, c), j = max(r, c);
    return tot[6 * i - i * (i - 1) / 2 + (j - i)];
}

// Adds up (or takes the maximum of) ten values over the 64 lanes by recursive
// halving: at each exchange a lane keeps one half of its values and sends the
// other.  Lane 4 k holds the total of value k.
template <bool kMax>
__device__ __forceinline__ double wave_total10(const double v[10])
{
    const int lane = threadIdx.x & 63;
    auto op = [](double x, double y) { return kMax ? fmax(x, y) : x + y; };
    const double none = kMax ? -INFINITY : 0.0;
    double h8[8], h4[4], h2[2];
    const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double up = k + 8 < 10 ? v[k + 8] : none;
        h8[k] = op(b5 ? up : v[k], __shfl_xor(b5 ? v[k] : up, 32));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) h4[k] = op(b4 ? h8[k + 4] : h8[k], __shfl_xor(b4 ? h8[k] : h8[k + 4], 16));
#pragma unroll
    for (int k = 0; k < 2; ++k) h2[k] = op(b3 ? h4[k + 2] : h4[k], __shfl_xor(b3 ? h4[k] : h4[k + 2], 8));
    double h = op(b2 ? h2[1] : h2[0], __shfl_xor(b2 ? h2[0] : h2[1], 4));
    h = op(h, __shfl_xor(h, 2));
    return op(h, __shfl_xor(h, 1));
}

// warm: start the eigen-decomposition from the previous iteration's
// eigenvectors (kept in vwork): the system changes little from one iteration
// to the next, so V^T A V is nearly diagonal and a sweep or two finish it.
//
// One workgroup: what it costs is the length of its chain of FP64 operations
// and LDS round trips.  Each wavefront adds up ten of the sums (the last the
// maxima); from there on one wavefront works with a lane per matrix entry.  A
// single thread for the system, the back-substitution and the pose, and an
// eigen-decomposition that exchanged the matrix between lanes: 14.3 us at
// 160x120 and 15.9 at 640x480, now 11.0 and 11.5 (means over chains of ten
// iterations from a nearby pose; 15 us at 640x480 between frames 7.5 cm apart).
__global__ __launch_bounds__(kIcpThreads) void icp_solve_kernel(const double *__restrict__ partial, int groups,
                                                                const double *__restrict__ pose, IcpArgs a,
                                                                tsdf_icp_result *__restrict__ res,
                                                                double *__restrict__ vwork, int warm)
{
    __shared__ SolveLds L;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (wave < 3) {
        double v[10];
#pragma unroll
        for (int k = 0; k < 10; ++k) v[k] = 0.0;
#pragma unroll 2
        for (int g = lane; g < groups; g += 64)
#pragma unroll
            for (int k = 0; k < 10; ++k) v[k] += partial[(size_t)(10 * wave + k) * groups + g];
        const double s = wave_total10<false>(v);
        if (!(lane & 3) && lane < 40) L.tot[10 * wave + (lane >> 2)] = s;
    } else {
        if (warm && lane < 36) L.V0[lane] = vwork[lane];
        double v[10];
#pragma unroll
        for (int k = 0; k < 10; ++k) v[k] = -INFINITY;
#pragma unroll 2
        for (int g = lane; g < groups; g += 64)
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] = fmax(v[k], partial[(size_t)(32 + k) * groups + g]);
        const double s = wave_total10<true>(v);
        if (!(lane & 3) && lane < 24) L.tot[32 + (lane >> 2)] = s;
    }
    const double pose_mine = wave == 0 && lane < 12 ? pose_at(pose, a, lane) : 0.0;
    __syncthreads();
    if (wave) return;

    // The scaled system by the change of variables c^ = S^-1 (c - M n), M n =
    // m x n: row r of the transform of (c, n) is D_r (e_r - sum_l M_rl e_3+l),
    // D = (S^-1, 1), so an entry of T A T^T is a sum of nine.
    const double N = L.tot[28];
    double m[3] = {0.0, 0.0, 0.0}, S[3] = {1.0, 1.0, 1.0};
    const bool scaled = a.shrink && N > 0.0;
    if (scaled) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double lo = -L.tot[32 + q], hi = L.tot[35 + q];
            m[q] = 0.5 * (lo + hi);
            const double ext = hi - lo;
            S[q] = ext > 0.0 ? ext : 1.0;
        }
    }
    const bool own = lane < 36;
    const int r = own ? lane / 6 : (lane - 36) % 6, c = own ? lane % 6 : 0;   // lanes 36..41: the right-hand side
    auto at3 = [](const double x[3], int q) { return q == 0 ? x[0] : q == 1 ? x[1] : x[2]; };
    auto row = [&](int q, int idx[3], double w[3]) {   // the transform's row q, unscaled
        const int q1 = (q + 1) % 3, q2 = (q + 2) % 3;
        idx[0] = q;
        idx[1] = 3 + q1;
        idx[2] = 3 + q2;
        w[0] = 1.0;
        w[1] = q < 3 ? at3(m, q2) : 0.0;
        w[2] = q < 3 ? -at3(m, q1) : 0.0;
    };
    int ri[3], ci[3];
    double rw[3], cw[3];
    row(r, ri, rw);
    row(c, ci, cw);
    const double Sr = r < 3 ? at3(S, r) : 1.0, Sc = c < 3 ? at3(S, c) : 1.0;
    // (the terms in M are left out where there is no M, not multiplied by zero:
    // an infinite normal makes some sums infinite and must not reach the others)
    const bool rm = scaled && r < 3, cm = scaled && c < 3;
    double A = 0.0, b = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double x = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) x += j == 0 || cm ? cw[j] * sum_gg(L.tot, ri[i], ci[j]) : 0.0;
        A += i == 0 || rm ? rw[i] * x : 0.0;
        b += i == 0 || rm ? rw[i] * L.tot[21 + ri[i]] : 0.0;
    }
    A /= Sr * Sc;
    b = -b / Sr;
    if (own) L.A[lane] = A;
    else if (lane < 42) L.b[lane - 36] = b;
    wave_sync();
    // (r, c) and (c, r) are the same sum in another order
    if (own) A = 0.5 * (A + L.A[6 * c + r]);
    wave_sync();
    if (own) L.A[lane] = A;
    wave_sync();
    const bool use_warm = warm && N > 0.0;
    if (use_warm) {   // B = V0^T A V0, symmetrised
        double x = 0.0;
        for (int l = 0; l < 6; ++l) x += L.A[6 * r + l] * L.V0[6 * l + c];
        if (own) L.V[lane] = x;
        wave_sync();
        x = 0.0;
        for (int k = 0; k < 6; ++k) x += L.V0[6 * k + r] * L.V[6 * k + c];
        if (own) L.B[lane] = x;
        wave_sync();
        x = 0.5 * (x + L.B[6 * c + r]);
        wave_sync();
        if (own) L.B[lane] = x;
        wave_sync();
    }
    if (N > 0.0) jacobi6_wave(use_warm ? L.B : L.A, use_warm ? L.V0 : nullptr, L.V, L.lam);
    if (own) vwork[lane] = N > 0.0 ? L.V[lane] : (r == c ? 1.0 : 0.0);

    // the directions above the threshold: lane e < 6 has eigenvalue e
    const int e = lane < 6 ? lane : 0;
    const double lam = N > 0.0 ? L.lam[e] : 0.0;
    const bool keep = lane < 6 && N > 0.0 && lam > 0.0 && (a.theta >= 0.0 ? lam / N > a.theta : true);
    const int kept = __popcll(__ballot(keep));
    if (lane < 6) {
        double vb = 0.0;
        for (int q = 0; q < 6; ++q) vb += L.V[6 * q + e] * L.b[q];
        L.w[e] = keep ? vb / lam : 0.0;
    }
    wave_sync();
    if (lane < 6) {
        double x = 0.0;
        for (int q = 0; q < 6; ++q)
            if (L.w[q] != 0.0) x += L.V[6 * e + q] * L.w[q];
        L.xh[e] = x;
    }
    wave_sync();
    // back to the unscaled increment: r = S^-1 r^, t = t^ - r x m
    double x[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (N > 0.0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) x[q] = L.xh[q] / S[q];
        x[3] = L.xh[3] - (x[1] * m[2] - x[2] * m[1]);
        x[4] = L.xh[4] - (x[2] * m[0] - x[0] * m[2]);
        x[5] = L.xh[5] - (x[0] * m[1] - x[1] * m[0]);
    }
    // R_inc = Rz(gamma) Ry(beta) Rx(alpha); pose' = R_inc pose + t_inc
    if (lane < 3) sincos(at3(x, lane), &L.sc[lane], &L.sc[3 + lane]);
    if (lane < 12) L.P[lane] = pose_mine;
    wave_sync();
    if (lane < 12) {
        const int pr = lane >> 2, pc = lane & 3;
        double P = pose_mine;
        if (N > 0.0) {
            const double sa = L.sc[0], sb = L.sc[1], sg = L.sc[2], ca = L.sc[3], cb = L.sc[4], cg = L.sc[5];
            const double y0 = pr == 0 ? cg * cb : pr == 1 ? sg * cb : -sb;
            const double y1 = pr == 0 ? cg * (sb * sa) - sg * ca : pr == 1 ? sg * (sb * sa) + cg * ca : cb * sa;
            const double y2 = pr == 0 ? cg * (sb * ca) + sg * sa : pr == 1 ? sg * (sb * ca) - cg * sa : cb * ca;
            P = y0 * L.P[pc] + y1 * L.P[4 + pc] + y2 * L.P[8 + pc];
            if (pc == 3) P += at3(x + 3, pr);
        }
        res->pose[lane] = P;   // (may be the current pose's own record: read before)
    }
    // eigenvalues per pair, ascending, by an insertion sort in every lane: all six
    // are written whatever they are (a rank by comparisons has gaps with NaN)
    if (lane < 6) L.lam[e] = N > 0.0 ? lam / N : 0.0;
    wave_sync();
    if (lane < 6) {
        double o[6], mine = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) o[q] = L.lam[q];
#pragma unroll
        for (int q = 1; q < 6; ++q)
#pragma unroll
            for (int f = q; f > 0; --f) {
                const bool swap = o[f - 1] > o[f];
                const double lo = swap ? o[f] : o[f - 1], hi = swap ? o[f - 1] : o[f];
                o[f - 1] = lo;
                o[f] = hi;
            }
#pragma unroll
        for (int q = 0; q < 6; ++q) mine = q == lane ? o[q] : mine;
        res->lambda[lane] = mine;
        res->b[lane] = L.b[lane];
        res->x[lane] = lane < 3 ? at3(x, lane) : at3(x + 3, lane - 3);
    }
    if (lane < 3) {
        res->m[lane] = at3(m, lane);
        res->S[lane] = at3(S, lane);
    }
    if (own) res->C[lane] = A;
    if (lane == 0) {
        res->residual2 = L.tot[27];
        res->pairs = (int64_t)N;
        res->kept = kept;
        res->pad = 0;
    }
}

int icp_groups(int32_t width, int32_t height)
{
    const long long npix = (long long)width * height;
    const long long g = (npix + kIcpThreads - 1) / kIcpThreads;
    return (int)(g < kIcpMaxGroups ? g : kIcpMaxGroups);
}

bool icp_pose_ok(const double *p)
{
    for (int q = 0; q < 12; ++q)
        if (!isfinite(p[q])) return false;
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) {
            const double dot = p[4 * r] * p[4 * c] + p[4 * r + 1] * p[4 * c + 1] + p[4 * r + 2] * p[4 * c + 2];
            if (fabs(dot - (r == c ? 1.0 : 0.0)) > 1e-6) return false;
        }
    const double det = p[0] * (p[5] * p[10] - p[6] * p[9]) - p[1] * (p[4] * p[10] - p[6] * p[8]) +
                       p[2] * (p[4] * p[9] - p[5] * p[8]);
    return det > 0;
}

}  // namespace

// Scratch memory of tsdf_icp_run_noalloc: the per-workgroup partial sums of
// at most kIcpMaxGroups workgroups (the cap of icp_groups, whatever the frame
// size) followed by the 36 warm-start eigenvector entries, the layout the
// caller's workspace has in tsdf_icp_run.  Each device holds its own copy
// from the first call on it until the process ends.
constexpr int kScratchDoubles = kIcpMaxGroups * kPartial + 36;
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[kMaxDevices];

// Device address of the current device's `scratch` (in host code the name
// stands for a host-side shadow, never for device memory); looked up once
// per device with that device current.  nullptr on failure.
double *scratch_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        g_scratch_ptr[dev] = (double *)ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace tsdf

using namespace tsdf;

extern "C" {

uint64_t tsdf_icp_workspace_bytes(int32_t width, int32_t height)
{
    if (width < 1 || height < 1 || width > 16384 || height > 16384) return 0;
    // partials, then the last eigenvectors (36 doubles) for a warm start
    return (uint64_t)icp_groups(width, height) * kPartial * sizeof(double) + 36 * sizeof(double);
}

}  // extern "C"

namespace {

// Validates the arguments shared by the ICP entry points (all but the
// workspace) and fills the kernel arguments.
tsdf_status icp_args(const float *depth_dev, const tsdf_intrinsics *K, const float *model_vertex_dev,
                     const float *model_normal_dev, const double *model_pose_c2w, const tsdf_icp_params *params,
                     const void *result_dev, IcpArgs &a)
{
    if (!depth_dev || !K || !model_vertex_dev || !model_normal_dev || !model_pose_c2w || !params || !result_dev)
        return TSDF_EINVAL;
    if (!(isfinite(K->fx) && isfinite(K->fy) && isfinite(K->cx) && isfinite(K->cy) && K->fx > 0 && K->fy > 0))
        return TSDF_EINVAL;
    if (tsdf_icp_workspace_bytes(K->width, K->height) == 0) return TSDF_EINVAL;
    if (!icp_pose_ok(model_pose_c2w)) return TSDF_EINVAL;
    if (!(isfinite(params->dist_max) && params->dist_max > 0) ||
        !(isfinite(params->cos_min) && params->cos_min >= -1.0 && params->cos_min <= 1.0) ||
        !isfinite(params->theta) || (params->shrink != 0 && params->shrink != 1))
        return TSDF_EINVAL;
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) a.Rm[3 * r + c] = model_pose_c2w[4 * r + c];
        a.tm[r] = model_pose_c2w[4 * r + 3];
    }
    a.fx = K->fx;
    a.fy = K->fy;
    a.cx = K->cx;
    a.cy = K->cy;
    a.width = K->width;
    a.height = K->height;
    a.dist2 = params->dist_max * params->dist_max;
    a.cos2 = params->cos_min * params->cos_min;
    a.theta = params->theta;
    a.shrink = params->shrink;
    for (int q = 0; q < 12; ++q) a.P0[q] = 0.0;
    return TSDF_OK;
}

void icp_enqueue(const float *depth_dev, const float *mv, const float *mn, const double *pose_dev, const IcpArgs &a,
                 void *workspace_dev, tsdf_icp_result *result_dev, int warm, hipStream_t stream)
{
    const int groups = icp_groups(a.width, a.height);
    double *partial = (double *)workspace_dev;
    double *vwork = partial + (size_t)groups * kPartial;
    hipLaunchKernelGGL(icp_pairs_kernel, dim3(groups), dim3(kIcpThreads), 0, stream, depth_dev, (const float4 *)mv,
                       (const float4 *)mn, pose_dev, a, partial);
    hipLaunchKernelGGL(icp_solve_kernel, dim3(1), dim3(kIcpThreads), 0, stream, partial, groups, pose_dev, a,
                       result_dev, vwork, warm);
}

}  // namespace

extern "C" {

tsdf_status tsdf_icp_step(const float *depth_dev, const tsdf_intrinsics *K, const float *model_vertex_dev,
                          const float *model_normal_dev, const double model_pose_c2w[12], const double *pose_dev,
                          const tsdf_icp_params *params, void *workspace_dev, uint64_t workspace_bytes,
                          tsdf_icp_result *result_dev, hipStream_t stream)
{
    IcpArgs a;
    if (!pose_dev) return TSDF_EINVAL;
    const tsdf_status st = icp_args(depth_dev, K, model_vertex_dev, model_normal_dev, model_pose_c2w, params,
                                    result_dev, a);
    if (st != TSDF_OK) return st;
    if (!workspace_dev || workspace_bytes < tsdf_icp_workspace_bytes(K->width, K->height)) return TSDF_EINVAL;
    icp_enqueue(depth_dev, model_vertex_dev, model_normal_dev, pose_dev, a, workspace_dev, result_dev, 0, stream);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

}  // extern "C"

namespace {

// Validates the arguments of a chain of iterations (all but the workspace).
tsdf_status icp_run_args(const float *depth_dev, const tsdf_intrinsics *K, const float *model_vertex_dev,
                         const float *model_normal_dev, const double *model_pose_c2w, const double *pose_init_c2w,
                         const tsdf_icp_params *params, int32_t iters, const void *results_dev, IcpArgs &a)
{
    if (!pose_init_c2w || iters < 1 || iters > 1024 || !icp_pose_ok(pose_init_c2w)) return TSDF_EINVAL;
    const tsdf_status st = icp_args(depth_dev, K, model_vertex_dev, model_normal_dev, model_pose_c2w, params,
                                    results_dev, a);
    if (st != TSDF_OK) return st;
    for (int q = 0; q < 12; ++q) a.P0[q] = pose_init_c2w[q];
    return TSDF_OK;
}

tsdf_status icp_run_enqueue(const float *depth_dev, const float *mv, const float *mn, const IcpArgs &a, int32_t iters,
                            void *workspace_dev, tsdf_icp_result *results_dev, hipStream_t stream)
{
    for (int k = 0; k < iters; ++k)
        icp_enqueue(depth_dev, mv, mn, k == 0 ? nullptr : results_dev[k - 1].pose, a, workspace_dev, results_dev + k,
                    k > 0, stream);
    return hipGetLastError() == hipSuccess ? TSDF_OK : TSDF_EHIP;
}

}  // namespace

extern "C" {

tsdf_status tsdf_icp_run(const float *depth_dev, const tsdf_intrinsics *K, const float *model_vertex_dev,
                         const float *model_normal_dev, const double model_pose_c2w[12],
                         const double pose_init_c2w[12], const tsdf_icp_params *params, int32_t iters,
                         void *workspace_dev, uint64_t workspace_bytes, tsdf_icp_result *results_dev,
                         hipStream_t stream)
{
    IcpArgs a;
    const tsdf_status st = icp_run_args(depth_dev, K, model_vertex_dev, model_normal_dev, model_pose_c2w,
                                        pose_init_c2w, params, iters, results_dev, a);
    if (st != TSDF_OK) return st;
    if (!workspace_dev || workspace_bytes < tsdf_icp_workspace_bytes(K->width, K->height)) return TSDF_EINVAL;
    return icp_run_enqueue(depth_dev, model_vertex_dev, model_normal_dev, a, iters, workspace_dev, results_dev,
                           stream);
}

tsdf_status tsdf_icp_run_noalloc(const float *depth_dev, const tsdf_intrinsics *K, const float *model_vertex_dev,
                                 const float *model_normal_dev, const double model_pose_c2w[12],
                                 const double pose_init_c2w[12], const tsdf_icp_params *params, int32_t iters,
                                 tsdf_icp_result *results_dev, hipStream_t stream)
{
    IcpArgs a;
    const tsdf_status st = icp_run_args(depth_dev, K, model_vertex_dev, model_normal_dev, model_pose_c2w,
                                        pose_init_c2w, params, iters, results_dev, a);
    if (st != TSDF_OK) return st;
    // the frame-size check above bounds the workgroups at kIcpMaxGroups, so
    // the partials always fit; checked again against the array itself
    if (tsdf_icp_workspace_bytes(K->width, K->height) > sizeof(double) * (uint64_t)kScratchDoubles)
        return TSDF_EINVAL;
    double *ws = scratch_address();
    if (!ws) return TSDF_EHIP;
    return icp_run_enqueue(depth_dev, model_vertex_dev, model_normal_dev, a, iters, ws, results_dev, stream);
}

}  // extern "C"

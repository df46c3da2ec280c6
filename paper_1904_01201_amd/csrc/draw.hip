// The direct path: triangles are drawn into the z-keys of a screen tile held
// in LDS, cluster by cluster from near to far, without triangle lists.
//
//   k_zclear     clear the views' counters (and z-keys, where tiles are shared)
//   k_zcull      per (view, 64-triangle cluster): frustum test; the visible
//                clusters go to the view's distance buckets with their pixel
//                rectangle and the largest 1/w any of their fragments can have
//   k_tile<TS>   a block per TS x TS tile (or per tile and share of the
//                clusters): lists the clusters whose rectangle meets the tile,
//                nearest buckets first; its waves take them one by one, drop
//                those whose part of the tile already holds nearer fragments
//                everywhere, set up the others' triangles and merge their
//                fragments in LDS by a 64-bit max (1/w bits above the
//                complemented key).  A block that owns its tile shades and
//                writes it; shares of a tile merge their z-keys in memory
//   k_zresolve   shared tiles only: per band of 32 x 2 pixels, shade and write
//
// Coverage, keys and shading are those of the tile-list path, operation by
// operation, and the maximum is independent of order: the outputs are the
// same bits.
//
// This is the path of small launches (runtime.cpp, direct_launch), which the
// tile lists leave waiting on a chain of eight kernels, and on a raster whose
// few long lists fall to few blocks.  One 256 x 256 view of 200k triangles
// took 0.1 ms there: 51 us raster, 12 us setup, 20 us binning, 15 us the rest
// and 5 us between kernels; here 57 us, 35 of them k_tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "device_util.h"
#include "dtypes.h"
#include "kernels.h"
#include "raster_math.h"
#include "shade.h"

#pragma clang fp contract(off)

namespace habmi {

typedef unsigned long long u64;

// DESC: the launch's descriptor block comes as an argument and is written here.
// Copied from pinned memory instead, it held the first kernel back by 7 us: a
// 128 x 128 frame of 2k triangles took 42 us, 36 so; a 256 x 256 frame of 200k
// triangles 62 and 56, a 203 x 117 one on the static scratch 40 and 33.
template <bool DESC>
__global__ __launch_bounds__(256) void k_zclear(typename std::conditional<DESC, InlineDesc, uint32_t>::type desc,
                                                uint4 *__restrict__ views, uint32_t n16, DViewCounters *__restrict__ ctr, uint32_t nviews,
                                                uint4 *__restrict__ z, size_t nz)
{
    const size_t stride = (size_t)gridDim.x * 256u;
    const size_t i = blockIdx.x * 256u + threadIdx.x;
    if constexpr (DESC) {
        if (i < n16) views[i] = reinterpret_cast<const uint4 *>(desc.bytes)[i];
    }
    for (size_t k = i; k < nz; k += stride) z[k] = make_uint4(0, 0, 0, 0);
    for (size_t k = i; k < (size_t)nviews * (sizeof(DViewCounters) / 16); k += stride)
        reinterpret_cast<uint4 *>(ctr)[k] = make_uint4(0, 0, 0, 0);
}

// ------------------------------------------------------------ k_zcull
// Is any of the cluster's box in sight of view v?  The test is box_outside's
// (kernels.hip states why it drops nothing the exact path would draw).  For
// a box wholly in front of the near plane, r also gets the pixel rectangle
// that holds every pixel its triangles can cover and an upper bound of any
// fragment's 1/w; else 1/w is unbounded (r.rho = inf) and the cluster is
// always drawn.  In fp32 a camera coordinate is off by less than
// 2^-20 |d|_1, so a projected coordinate is by less than
// (f + |x|) 2^-20 |d|_1 / w pixels (plus the snap): the rectangle is grown by
// four times that and two pixels, and rectangles whose margin or extent is
// out of all proportion are not used.  A box that passes all of this has no
// vertex outside the fixed-point domain, so dropping it hides no range error.
__device__ __forceinline__ bool box_in_sight(const DView &v, float4 mn, float4 mx, ClusterRec &r, float &wn)
{
    const double fS = (double)v.fS;
    const double Kx = (double)((v.cxS + 1024.0f) * 1.0000152587890625f);
    const double Ky = (double)((v.cyS + 1024.0f) * 1.0000152587890625f);
    double X[8], Y[8], W[8], l1 = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const double dx = (double)((c & 1) ? mx.x : mn.x) - (double)v.p[0];
        const double dy = (double)((c & 2) ? mx.y : mn.y) - (double)v.p[1];
        const double dz = (double)((c & 4) ? mx.z : mn.z) - (double)v.p[2];
        X[c] = (double)v.R[0] * dx + (double)v.R[3] * dy + (double)v.R[6] * dz;
        Y[c] = (double)v.R[1] * dx + (double)v.R[4] * dy + (double)v.R[7] * dz;
        W[c] = -((double)v.R[2] * dx + (double)v.R[5] * dy + (double)v.R[8] * dz);
        l1 = fmax(l1, fabs(dx) + fabs(dy) + fabs(dz));
    }
    const double mg = (fS + fmax(Kx, Ky)) * 0x1p-18 * l1, mz = 0x1p-18 * l1;
    bool rt = true, lt = true, up = true, dn = true, nr = true;
    double wmin = W[0];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        rt = rt && X[c] * fS - Kx * W[c] > mg;
        lt = lt && -X[c] * fS - Kx * W[c] > mg;
        up = up && Y[c] * fS - Ky * W[c] > mg;
        dn = dn && -Y[c] * fS - Ky * W[c] > mg;
        nr = nr && W[c] < (double)v.zn - mz;
        wmin = fmin(wmin, W[c]);
    }
    if (rt || lt || up || dn || nr) return false;
    wn = (float)wmin;
    r.lo = r.hi = 0;
    r.rho = __uint_as_float(0x7F800000u);
    const float ws = (float)(wmin - mz);
    if (ws > 1.001f * v.zn) {
        const float f = v.fS * (1.0f / 256.0f);
        float x0 = 1e30f, x1 = -1e30f, y0 = 1e30f, y1 = -1e30f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float s = f / (float)W[c];
            const float x = (float)X[c] * s, y = (float)Y[c] * s;
            x0 = fminf(x0, x);
            x1 = fmaxf(x1, x);
            y0 = fminf(y0, y);
            y1 = fmaxf(y1, y);
        }
        const float ext = fmaxf(fmaxf(-x0, x1), fmaxf(-y0, y1));
        const float m = 2.0f + (f + ext) * 0x1p-18f * (float)l1 / ws;
        if (ext < 65536.0f && m < 64.0f) {
            const float cx = 0.5f * (float)v.W, cy = 0.5f * (float)v.H;
            const int i0 = max((int)floorf(cx + x0 - m), 0), i1 = min((int)ceilf(cx + x1 + m), (int)v.W - 1);
            const int j0 = max((int)floorf(cy - y1 - m), 0), j1 = min((int)ceilf(cy - y0 + m), (int)v.H - 1);
            if (i0 > i1 || j0 > j1) return false;
            r.lo = (uint32_t)i0 | ((uint32_t)j0 << 16);
            r.hi = (uint32_t)i1 | ((uint32_t)j1 << 16);
            r.rho = (1.0f / ws) * 1.000030517578125f;
        }
    }
    return true;
}

// Distance bucket of a cluster whose nearest corner has planar depth w: half
// octaves from 0.25 m (the last one open), from the float's exponent and
// leading mantissa bit.
__device__ __forceinline__ uint32_t dist_bucket(float w)
{
    if (!(w > 0.25f)) return 0;
    return min((__float_as_uint(w) >> 22) - (__float_as_uint(0.25f) >> 22), kBuckets - 1);
}

constexpr int kZCullBlock = 256;

__global__ __launch_bounds__(kZCullBlock) void k_zcull(const DView *__restrict__ views,
                                                       DViewCounters *__restrict__ ctr,
                                                       ClusterRec *__restrict__ recs)
{
    __shared__ uint32_t cnt[kBuckets], base[kBuckets];
    const uint32_t vi = blockIdx.y;
    const DView &v = views[vi];
    const uint32_t ncl = (v.T + kCluster - 1) / kCluster;
    const uint32_t c0 = blockIdx.x * kZCullBlock;
    if (c0 >= ncl) return;
    if (threadIdx.x < kBuckets) cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t c = c0 + threadIdx.x;
    ClusterRec r;
    r.c = c;
    float wn = 0.0f;
    uint32_t b = 0, rank = 0;
    bool vis = c < ncl;
    if (vis) {
        const auto *p = gmem(reinterpret_cast<const float *>(v.cbox)) + 8ull * c;
        vis = box_in_sight(v, make_float4(p[0], p[1], p[2], p[3]), make_float4(p[4], p[5], p[6], p[7]), r, wn);
    }
    if (vis) {
        b = dist_bucket(wn);
        rank = atomicAdd(&cnt[b], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kBuckets) {
        const uint32_t n = cnt[threadIdx.x];
        base[threadIdx.x] = n ? atomicAdd(&ctr[vi].bucket[threadIdx.x], n) : 0u;
    }
    __syncthreads();
    if (vis) recs[(size_t)v.pair_base * kBuckets + (size_t)b * ncl + base[b] + rank] = r;
}

// ------------------------------------------------------------ rasterisation
// A block's tile: its z-keys in LDS and its pixels [oi, oi + TS) x [oj, oj + TS).
template <int TS>
struct Tile {
    u64 *z;
    int oi, oj;
    __device__ __forceinline__ uint32_t at(int i, int j) const { return (uint32_t)((j - oj) * TS + (i - oi)); }
    __device__ __forceinline__ void put(uint32_t off, u64 key) const
    {
        (void)__hip_atomic_fetch_max(z + off, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

__device__ __forceinline__ u64 zkey(float num, float invA, uint32_t nkey)
{
    const float rho = num * invA;
    return ((u64)__float_as_uint(rho) << 32) | (u64)nkey;
}

// (float)A, from int32 when it fits: the same rounding.
__device__ __forceinline__ float area_f(long long A)
{
    return A == (long long)(int)A ? (float)(int)A : (float)A;
}

__device__ __forceinline__ int rl(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ float rlf(float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); }

// Draw up to one triangle per lane (`live`: oriented a, b, c with twice-area
// A > 0), each in its pixel box's part of the tile.  Small parts: every lane
// walks its own, pixel by pixel; larger ones: the whole wave draws one
// triangle after another.
template <int TS>
__device__ __forceinline__ void draw_lanes(const DView &v, const Tile<TS> &zt, bool live, const SVtx<0> &a,
                                           const SVtx<0> &b, const SVtx<0> &c, long long A, uint32_t key)
{
    PixBox pb = pix_box(v, a, b, c);
    pb.i0 = max(pb.i0, zt.oi);
    pb.j0 = max(pb.j0, zt.oj);
    pb.i1 = min(pb.i1, zt.oi + TS - 1);
    pb.j1 = min(pb.j1, zt.oj + TS - 1);
    live = live && pb.i0 <= pb.i1 && pb.j0 <= pb.j1;
    if (!__ballot(live)) return;
    const uint32_t w = (uint32_t)(pb.i1 - pb.i0 + 1), h = (uint32_t)(pb.j1 - pb.j0 + 1);
    const uint32_t area = live ? w * h : 0u;
    // edge functions at the box's first pixel centre
    const int dx0 = c.X - b.X, dx1 = a.X - c.X, dx2 = b.X - a.X;
    const int dy0 = c.Y - b.Y, dy1 = a.Y - c.Y, dy2 = b.Y - a.Y;
    const int Ox = 256 * pb.i0 + 128, Oy = 256 * pb.j0 + 128;
    const int rx0 = b.X - Ox, rx1 = c.X - Ox, rx2 = a.X - Ox;
    const int ry0 = b.Y - Oy, ry1 = c.Y - Oy, ry2 = a.Y - Oy;
    constexpr int kNear = 1 << 14;
    const bool near = abs(rx0) < kNear && abs(rx1) < kNear && abs(rx2) < kNear && abs(ry0) < kNear &&
                      abs(ry1) < kNear && abs(ry2) < kNear;
    // how far the lanes walk: a step of the lane loop costs the wave about
    // 30 instructions, a triangle drawn by the wave about 80
    const uint32_t n24 = (uint32_t)__popcll(__ballot(area > 24)), n48 = (uint32_t)__popcll(__ballot(area > 48));
    const uint32_t n96 = (uint32_t)__popcll(__ballot(area > 96));
    uint32_t most = 24;
    if (n24 - n48 > 9) most = 48;
    if (n48 - n96 > 18) most = 96;
    const bool walk = live && near && area <= most;
    const bool med = live && !walk;
    // 24-bit products: |d| < 2^15, |r| < 2^14 (used where near)
    const int E0 = __mul24(dy0, rx0) - __mul24(dx0, ry0);
    const int E1 = __mul24(dy1, rx1) - __mul24(dx1, ry1);
    const int E2 = __mul24(dy2, rx2) - __mul24(dx2, ry2);
    const int n0 = owned(dx0, dy0) ? 0 : 1, n1 = owned(dx1, dy1) ? 0 : 1, n2 = owned(dx2, dy2) ? 0 : 1;
    const float invA = recip_rn(area_f(A));
    const uint32_t nkey = ~key;
    const uint32_t off0 = zt.at(pb.i0, pb.j0);
    if (walk) {
        const int wm = (int)w - 1;
        // to the next pixel of the row, and from a row's last pixel to the
        // next row's first
        const int cx0 = -256 * dy0, cx1 = -256 * dy1, cx2 = -256 * dy2;
        const int cr0 = 256 * (dx0 + __mul24(dy0, wm)), cr1 = 256 * (dx1 + __mul24(dy1, wm)),
                  cr2 = 256 * (dx2 + __mul24(dy2, wm));
        int F0 = E0, F1 = E1, F2 = E2;
        uint32_t off = off0;
        int x = 0;
        for (uint32_t k = 0; k < area; ++k) {
            if (F0 >= n0 && F1 >= n1 && F2 >= n2) {
                const float w0 = (float)F0 * a.rw, w1 = (float)F1 * b.rw, w2 = (float)F2 * c.rw;
                zt.put(off, zkey((w0 + w1) + w2, invA, nkey));
            }
            const bool wrap = x == wm;
            F0 += wrap ? cr0 : cx0;
            F1 += wrap ? cr1 : cx1;
            F2 += wrap ? cr2 : cx2;
            off += wrap ? TS - (uint32_t)wm : 1u;
            x = wrap ? 0 : x + 1;
        }
    }
    for (u64 m = __ballot(med); m; m &= m - 1) {
        const int l = __ffsll((long long)m) - 1;
        const int wl = rl((int)w, l), al = rl((int)area, l);
        const int d0 = rl(dx0, l), d1 = rl(dx1, l), d2 = rl(dx2, l), y0 = rl(dy0, l), y1 = rl(dy1, l), y2 = rl(dy2, l);
        const int o0 = rl(n0, l), o1 = rl(n1, l), o2 = rl(n2, l);
        const float r0 = rlf(a.rw, l), r1 = rlf(b.rw, l), r2 = rlf(c.rw, l), ia = rlf(invA, l);
        const uint32_t kl = (uint32_t)rl((int)nkey, l), ol = (uint32_t)rl((int)off0, l);
        const float iw = 1.0f / (float)wl;
        if (rl(near ? 1 : 0, l)) {
            // vertices within 64 px of the box: int32 arithmetic is exact
            const int e0 = rl(E0, l), e1 = rl(E1, l), e2 = rl(E2, l);
            for (int p = (int)lane_id(); p < al; p += 64) {
                const int y = (int)(((float)p + 0.5f) * iw), x = p - __mul24(y, wl);
                const int F0 = e0 + 256 * (__mul24(d0, y) - __mul24(y0, x));
                const int F1 = e1 + 256 * (__mul24(d1, y) - __mul24(y1, x));
                const int F2 = e2 + 256 * (__mul24(d2, y) - __mul24(y2, x));
                if (F0 >= o0 && F1 >= o1 && F2 >= o2) {
                    const float w0 = (float)F0 * r0, w1 = (float)F1 * r1, w2 = (float)F2 * r2;
                    zt.put(ol + (uint32_t)(y * TS + x), zkey((w0 + w1) + w2, ia, kl));
                }
            }
            continue;
        }
        const long long e0 = (long long)y0 * rl(rx0, l) - (long long)d0 * rl(ry0, l);
        const long long e1 = (long long)y1 * rl(rx1, l) - (long long)d1 * rl(ry1, l);
        const long long e2 = (long long)y2 * rl(rx2, l) - (long long)d2 * rl(ry2, l);
        for (int p = (int)lane_id(); p < al; p += 64) {
            const int y = (int)(((float)p + 0.5f) * iw), x = p - __mul24(y, wl);
            const long long F0 = e0 + (long long)d0 * (256 * y) - (long long)y0 * (256 * x);
            const long long F1 = e1 + (long long)d1 * (256 * y) - (long long)y1 * (256 * x);
            const long long F2 = e2 + (long long)d2 * (256 * y) - (long long)y2 * (256 * x);
            if (F0 >= o0 && F1 >= o1 && F2 >= o2) {
                const float w0 = (float)F0 * r0, w1 = (float)F1 * r1, w2 = (float)F2 * r2;
                zt.put(ol + (uint32_t)(y * TS + x), zkey((w0 + w1) + w2, ia, kl));
            }
        }
    }
}

// Set up and draw triangle t (per lane) of view v.
template <int TS>
__device__ __forceinline__ void draw_triangles(const DView &v, const Tile<TS> &zt, const float P[9], bool valid,
                                               uint32_t t, bool &rerr)
{
    Vtx<0> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    const float zn = v.zn;
    const bool allin = c0.w >= zn && c1.w >= zn && c2.w >= zn;
    bool live = valid && (c0.w >= zn || c1.w >= zn || c2.w >= zn);
    if (allin) {
        // conservative frustum rejection before any division (as in setup)
        const float Kx = (v.cxS + 1024.0f) * 1.0000152587890625f;
        const float Ky = (v.cyS + 1024.0f) * 1.0000152587890625f;
        const float x0 = c0.x * v.fS, x1 = c1.x * v.fS, x2 = c2.x * v.fS;
        const float y0 = c0.y * v.fS, y1 = c1.y * v.fS, y2 = c2.y * v.fS;
        const float kx0 = Kx * c0.w, kx1 = Kx * c1.w, kx2 = Kx * c2.w;
        const float ky0 = Ky * c0.w, ky1 = Ky * c1.w, ky2 = Ky * c2.w;
        if ((x0 > kx0 && x1 > kx1 && x2 > kx2) || (x0 < -kx0 && x1 < -kx1 && x2 < -kx2) ||
            (y0 > ky0 && y1 > ky1 && y2 > ky2) || (y0 < -ky0 && y1 < -ky1 && y2 < -ky2))
            live = false;
    }
    if (!__ballot(live)) return;
    SVtx<0> a = {}, b = {}, c = {};
    long long A = 0;
    bool ok = false;
    if (live && allin) {
        bool in = snap(v, c0, a);
        in &= snap(v, c1, b);
        in &= snap(v, c2, c);
        if (!in) rerr = true;
        A = area2(a, b, c);
        if (A < 0) {
            const SVtx<0> s = b;
            b = c;
            c = s;
            A = -A;
        }
        ok = in && A != 0;
    }
    // triangles that cross the near plane have up to two sub-triangles
    const bool clip = live && !allin;
    const int nsub = __ballot(clip) ? 2 : 1;
#pragma unroll 1
    for (int sub = 0; sub < nsub; ++sub) {
        if (clip) ok = setup_sub(v, c0, c1, c2, sub, a, b, c, A, rerr);
        else if (sub) ok = false;
        draw_lanes<TS>(v, zt, ok, a, b, c, A, 2u * t + (uint32_t)sub);
    }
}

// Does every pixel of the cluster's part of the tile (w x h from (i, j))
// already hold a fragment nearer than any of the cluster's can be?  The keys
// only grow: a key read early can only keep a cluster that could be dropped.
template <int TS>
__device__ __forceinline__ bool hidden(const Tile<TS> &zt, int i, int j, int w, int h, float rho)
{
    const uint32_t *zh = reinterpret_cast<const uint32_t *>(zt.z + zt.at(i, j)) + 1;
    const float iw = 1.0f / (float)w;
    for (int p0 = 0; p0 < w * h; p0 += 64) {
        const int p = p0 + (int)lane_id();
        bool shows = false;
        if (p < w * h) {
            const int y = (int)(((float)p + 0.5f) * iw), x = p - y * w;
            shows = !(__uint_as_float(__hip_atomic_load(zh + 2 * (y * TS + x), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP)) > rho);
        }
        if (__ballot(shows)) return false;
    }
    return true;
}

// ------------------------------------------------------------ k_tile
// Bound by latency: in a small launch a wave draws a cluster or two, about
// 900 instructions each behind three dependent loads (record, positions, the
// list before them), with a wave or two per SIMD.  So the clusters of a tile
// are spread over as many blocks as fill the chip; what a share costs beside
// its clusters is its part of the record list and merging its touched pixels
// by memory atomics (about 27 G 64-byte sectors/s on this part, whatever a
// sector holds).  Drawing straight into memory with those atomics, without a
// tile in LDS, took 75 us instead of 35 on the same view (5.4 sectors per wave
// and step); writing every pixel after a look at its key 110 us (each look
// waits for the atomics before it).
template <int TS>
struct TileCfg {
    static constexpr int NW = TS == 64 ? 8 : 4;           // waves per block
    static constexpr int NT = NW * 64;
    static constexpr uint32_t list = TS == 64 ? 2048 : 1024;   // clusters listed at once
    static constexpr int BW = TS < kBandW ? TS : kBandW, BH = 64 / BW;
};

template <int TS>
__global__ __launch_bounds__(TileCfg<TS>::NT) __attribute__((amdgpu_waves_per_eu(4))) void k_tile(
    const DView *__restrict__ views, const uint32_t *__restrict__ lview, const uint32_t *__restrict__ tpre, uint32_t nl,
    uint32_t shares, const DViewCounters *__restrict__ ctr, const ClusterRec *__restrict__ recs,
    u64 *__restrict__ zbuf, uint32_t *__restrict__ err)
{
    using C = TileCfg<TS>;
    __shared__ u64 zt_[TS * TS];
    __shared__ uint32_t list[C::list];
    __shared__ uint32_t wtot[C::NW], cursor;
    __shared__ __align__(16) uint8_t s_rgb[C::NW][kBandRgb];
    uint32_t lo = 0, hi = nl - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (tpre[mid] <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t vi = uniform(lview[uniform(lo)]);
    const DView &v = views[vi];
    const uint32_t in_view = blockIdx.x - uniform(tpre[uniform(lo)]);
    const uint32_t share = in_view % shares, tile = in_view / shares;
    const uint32_t ntx = (v.W + TS - 1) / TS;
    const int ty = (int)(tile / ntx), tx = (int)(tile % ntx);
    const Tile<TS> zt = {zt_, tx * TS, ty * TS};
    const int ti1 = min(zt.oi + TS, (int)v.W) - 1, tj1 = min(zt.oj + TS, (int)v.H) - 1;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    for (uint32_t i = tid; i < TS * TS; i += C::NT) zt_[i] = 0;
    // this share's clusters: ranks share, share + shares, ... of the buckets
    // in order
    uint32_t ex[kBuckets], nvis = 0;
#pragma unroll
    for (uint32_t b = 0; b < kBuckets; ++b) {
        ex[b] = nvis;
        nvis += ctr[vi].bucket[b];
    }
    const uint32_t mine = nvis > share ? (nvis - share + shares - 1) / shares : 0u;
    const uint32_t ncl = (v.T + kCluster - 1) / kCluster;
    const ClusterRec *const vr = recs + (size_t)v.pair_base * kBuckets;
    bool rerr = false;
    constexpr uint32_t kPer = 1024 / C::NT;   // records a thread tests per round
    for (uint32_t base = 0; base < mine;) {
        // list the clusters that meet the tile
        uint32_t count = 0;
        while (base < mine && count + 1024 <= C::list) {
            uint32_t at[kPer], got = 0;
            bool meets[kPer];
#pragma unroll
            for (uint32_t q = 0; q < kPer; ++q) {
                // consecutive records per thread keep the order
                const uint32_t k = base + tid * kPer + q;
                meets[q] = false;
                at[q] = 0;
                if (k < mine) {
                    const uint32_t rank = k * shares + share;
                    uint32_t b = 0, eb = 0;
#pragma unroll
                    for (uint32_t j = 1; j < kBuckets; ++j)
                        if (ex[j] <= rank) {
                            b = j;
                            eb = ex[j];
                        }
                    at[q] = b * ncl + (rank - eb);
                    const ClusterRec r = vr[at[q]];
                    const int i0 = (int)(r.lo & 0xFFFFu), j0 = (int)(r.lo >> 16);
                    const int i1 = (int)(r.hi & 0xFFFFu), j1 = (int)(r.hi >> 16);
                    meets[q] = !(r.rho < 3.0e38f) || (i0 <= ti1 && i1 >= zt.oi && j0 <= tj1 && j1 >= zt.oj);
                }
                got += meets[q] ? 1u : 0u;
            }
            uint32_t tot;
            uint32_t o = count + block_excl_scan<C::NT>(got, wtot, &tot);
#pragma unroll
            for (uint32_t q = 0; q < kPer; ++q)
                if (meets[q]) list[o++] = at[q];
            count += tot;
            base += 1024;
        }
        if (tid == 0) cursor = 0;
        __syncthreads();
        // the waves draw them in order
        for (;;) {
            uint32_t k = 0;
            if (lane == 0) k = atomicAdd(&cursor, 1u);
            k = uniform(k);
            if (k >= count) break;
            const ClusterRec r = vr[uniform(list[k])];
            const float rho = __uint_as_float(uniform(__float_as_uint(r.rho)));
            const uint32_t rlo = uniform(r.lo), rhi = uniform(r.hi);
            if (rho < 3.0e38f) {
                const int i0 = max((int)(rlo & 0xFFFFu), zt.oi), j0 = max((int)(rlo >> 16), zt.oj);
                const int i1 = min((int)(rhi & 0xFFFFu), ti1), j1 = min((int)(rhi >> 16), tj1);
                if (hidden<TS>(zt, i0, j0, i1 - i0 + 1, j1 - j0 + 1, rho)) continue;
            }
            const uint32_t t = uniform(r.c) * kCluster + lane;
            const bool valid = t < v.T;
            float P[9] = {};
            if (valid) load_pos(v, t, P);
            draw_triangles<TS>(v, zt, P, valid, t, rerr);
        }
        __syncthreads();
    }
    if (rerr) atomicOr(err, kErrRange);
    if (mine == 0) __syncthreads();   // the cleared keys
    const uint32_t px = lane % C::BW, py = lane / C::BW;
    constexpr uint32_t kBandsX = TS / C::BW, kBands = kBandsX * (TS / C::BH);
    for (uint32_t band = wave; band < kBands; band += C::NW) {
        const uint32_t bx = (band % kBandsX) * C::BW, by = (band / kBandsX) * C::BH;
        const int pi = zt.oi + (int)(bx + px), pj = zt.oj + (int)(by + py);
        if (zt.oi + (int)bx > ti1 || zt.oj + (int)by > tj1) continue;
        const bool in = pi <= ti1 && pj <= tj1;
        const u64 z = zt_[(by + py) * TS + bx + px];
        if (shares == 1) {
            shade_band<C::BW, C::BH>(v, (uint32_t)zt.oi + bx, (uint32_t)zt.oj + by, pi, pj, in,
                                     __uint_as_float((uint32_t)(z >> 32)), ~(uint32_t)z, s_rgb[wave], err);
        } else if (in && z) {
            u64 *zv = zbuf + (((u64)v.zoff_hi << 32) | v.zoff_lo);
            (void)__hip_atomic_fetch_max(zv + ((uint32_t)pj * v.W + (uint32_t)pi), z, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ------------------------------------------------------------ k_zresolve
__global__ __launch_bounds__(kBandThreads) void k_zresolve(const DView *__restrict__ views,
                                                           const uint32_t *__restrict__ lview,
                                                           const uint32_t *__restrict__ bpre, uint32_t nl,
                                                           const u64 *__restrict__ zbuf, uint32_t *__restrict__ err)
{
    __shared__ __align__(16) uint8_t s_rgb[kBandRgb];
    uint32_t lo = 0, hi = nl - 1;
    const uint32_t blk = blockIdx.x;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (bpre[mid] <= blk) lo = mid;
        else hi = mid - 1;
    }
    const DView &v = views[uniform(lview[uniform(lo)])];
    const uint32_t W = v.W, H = v.H;
    const uint32_t nbx = (W + kBandW - 1) / kBandW;
    const uint32_t band = blk - bpre[lo];
    const uint32_t x0 = (band % nbx) * kBandW, y0 = (band / nbx) * kBandH;
    const uint32_t lane = lane_id();
    const int pi = (int)(x0 + lane % kBandW), pj = (int)(y0 + lane / kBandW);
    const bool in = pi < (int)W && pj < (int)H;
    float best_rho = 0.0f;
    uint32_t best_key = kNone;
    if (in) {
        const u64 z = zbuf[(((u64)v.zoff_hi << 32) | v.zoff_lo) + (u64)((uint32_t)pj * W + (uint32_t)pi)];
        best_rho = __uint_as_float((uint32_t)(z >> 32));
        best_key = ~(uint32_t)z;
    }
    shade_band<kBandW, kBandH>(v, x0, y0, pi, pj, in, best_rho, best_key, s_rgb, err);
}

// ------------------------------------------------------------ host side
static inline uint32_t cdiv(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

static inline void mark(const LaunchPlan &L, int ev, hipStream_t s)
{
    if (L.prof && ((L.prof_mask >> (ev >> 1)) & 1u)) (void)hipEventRecord(L.prof[ev], s);
}

template <int TS>
static void launch_tile(const LaunchPlan &L, const RasterLaunch &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile<TS>, dim3(L.tile_grid), dim3(TileCfg<TS>::NT), 0, s, L.views, R.lview, L.tpre, R.nl,
                       L.shares, L.ctr, L.recs, L.zbuf, L.err);
}

hipError_t launch_direct(const LaunchPlan &L, hipStream_t s)
{
    const RasterLaunch &R = L.raster[0];
    const size_t nz = L.shares > 1 ? L.znum / 2 : 0;   // 16-byte pairs of z-keys
    const size_t nc = (size_t)L.nviews * (sizeof(DViewCounters) / 16);
    const size_t nclear = nz > nc ? nz : nc;
    mark(L, 0, s);
    const dim3 grid((uint32_t)(nclear / 256 + 1 < 4096 ? nclear / 256 + 1 : 4096));
    uint4 *const views = reinterpret_cast<uint4 *>(const_cast<DView *>(L.views)), *const z = reinterpret_cast<uint4 *>(L.zbuf);
    if (L.desc)
        hipLaunchKernelGGL(k_zclear<true>, grid, dim3(256), 0, s, *L.desc, views, L.desc_bytes / 16, L.ctr, L.nviews, z, nz);
    else
        hipLaunchKernelGGL(k_zclear<false>, grid, dim3(256), 0, s, 0u, views, 0u, L.ctr, L.nviews, z, nz);
    mark(L, 1, s);
    mark(L, 2, s);
    hipLaunchKernelGGL(k_zcull, dim3(L.cull_blocks, L.nviews), dim3(kZCullBlock), 0, s, L.views, L.ctr, L.recs);
    mark(L, 3, s);
    const int ph = R.ts == 8 ? 5 : R.ts == 16 ? 6 : 7;
    mark(L, 2 * ph, s);
    switch (L.tile_edge) {
    case 16: launch_tile<16>(L, R, s); break;
    case 32: launch_tile<32>(L, R, s); break;
    case 64: launch_tile<64>(L, R, s); break;
    default: return hipErrorInvalidValue;
    }
    mark(L, 2 * ph + 1, s);
    mark(L, 2 * kPhaseResolve, s);
    if (L.shares > 1)
        hipLaunchKernelGGL(k_zresolve, dim3(R.bands), dim3(kBandThreads), 0, s, L.views, R.lview, R.bpre, R.nl, L.zbuf,
                           L.err);
    mark(L, 2 * kPhaseResolve + 1, s);
    return hipGetLastError();
}

}  // namespace habmi

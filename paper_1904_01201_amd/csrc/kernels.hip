// HIP kernels of the renderer for gfx950 (CDNA4, wave64).
//
// One launch sequence renders a batch of views (any mix of scenes,
// resolutions and output sets):
//   k_reset      zero the per-view, per-tile and work-queue counters
//   k_cull       per (view, 64-triangle cluster): conservative frustum test
//                of the cluster's box; the visible clusters are listed
//   k_setup      per (view, run of visible clusters): fetch each triangle,
//                transform, clip, snap, orient and cull it; survivors (key,
//                pixel bbox) go to the run's slots with wave-level
//                compaction (the views of a scene are consecutive, so its
//                triangles are re-read from L2/MALL)
//   k_bin<count> per chunk of runs: LDS histogram of the screen tiles
//                their boxes touch, one global add per touched tile
//   k_bin_scan   per view: exclusive scans of the tile counts (list offsets;
//                tiles over capacity take the lossless overflow path) and of
//                the tiles' segment counts; the (tile, segment) work items
//                are appended to the queue of the view's tile size
//   k_bin<scatter> per chunk of runs: write each key into every touched
//                tile's list (LDS ranks, one global reservation per tile)
//   k_raster<TS> persistent blocks pull (tile, segment) items from the queue
//                (an atomic counter used for work distribution only).  The
//                segment's triangles are staged through LDS (each lane
//                rebuilds one edge setup relative to the tile, with the
//                pixel blocks its box and edges leave), then the wave lists
//                the (triangle, block) pairs and each step gives every lane
//                group one pair: the group's lanes test that block's pixels
//                and keep the nearest candidate (largest 1/w, smaller key on
//                ties) by an LDS atomic max per pixel; the segment's
//                per-pixel winner goes to scratch
//   k_raster_wave the same for 16-pixel tiles, a wave per work item; its
//                z-keys stay in one place per tile (k_resolve_wave reads them)
//   k_resolve<TS> per band of 32 x 2 pixels (one wave): merge the segments'
//                winners with the same rule, rebuild the winner, write
//                colour (through LDS, as words), planar depth and index:
//                whole 32-byte sectors.
// Coverage and visibility are decided by exact integer edge functions and
// one fixed sequence of fp32 operations (the key), so outputs do not depend
// on batching, tile size, capacity, segmenting or scheduling order.
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

// ------------------------------------------------------------ k_scene
// A wave per cluster, a lane per triangle.  A lane has read its triangle's indices
// before it writes the colours, which may take their place.
__global__ __launch_bounds__(256) void k_scene(MeshSource m, uint32_t T, float *__restrict__ tpos, uint32_t *attr,
                                               float4 *__restrict__ cbox, float3 size, float grow,
                                               SpreadSums *__restrict__ spread)
{
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (uniform(t & ~63u) >= T) return;
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (t < T) {
        size_t vid[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) vid[k] = m.idx[3ull * t + k];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float x = m.pos[3 * vid[k] + a];
                tpos[9ull * t + 3 * k + a] = x;
                mn[a] = fminf(mn[a], x);
                mx[a] = fmaxf(mx[a], x);
            }
            if (m.uv) {
                attr[6ull * t + 2 * k] = __float_as_uint(m.uv[2 * vid[k]]);
                attr[6ull * t + 2 * k + 1] = __float_as_uint(m.uv[2 * vid[k] + 1]);
            } else {
                const uint8_t *c = m.col ? m.col + 3 * vid[k] : nullptr;
                attr[3ull * t + k] = c ? (uint32_t)c[0] | ((uint32_t)c[1] << 8) | ((uint32_t)c[2] << 16) : 0xFFFFFFu;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            mn[a] = fminf(mn[a], __shfl_xor(mn[a], d));
            mx[a] = fmaxf(mx[a], __shfl_xor(mx[a], d));
        }
    if (lane_id() == 0) {
        cbox[2 * (t / kCluster)] = make_float4(mn[0], mn[1], mn[2], 0.0f);
        cbox[2 * (t / kCluster) + 1] = make_float4(mx[0], mx[1], mx[2], 0.0f);
        // in whole units: the sum does not depend on the order
        const float part = (mx[0] - mn[0] + grow) / (size.x + grow) * ((mx[1] - mn[1] + grow) / (size.y + grow)) *
                           ((mx[2] - mn[2] + grow) / (size.z + grow));
        atomicAdd(&spread->sum[blockIdx.x % 32u][0], (unsigned long long)(fminf(part, 1.0f) * 16777216.0f));
    }
}

// ------------------------------------------------------------ k_reset
__global__ __launch_bounds__(256) void k_reset(DViewCounters *__restrict__ ctr, uint32_t nviews,
                                               uint32_t *__restrict__ tile_count,
                                               uint32_t *__restrict__ tile_cursor, uint32_t ntiles,
                                               DQueue *__restrict__ q)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < nviews) {
        ctr[i].vis_clusters = 0;
        ctr[i].vis_tail = 0;
        ctr[i].surv_count = 0;
        ctr[i].bin_used = 0;
        ctr[i].bbox_tests = 0;
        ctr[i].covered = 0;
    }
    if (i < ntiles) {
        tile_count[i] = 0;
        tile_cursor[i] = 0;
    }
    if (i < 4) q->total[i] = 0;
    if (i < 3 * kQueues) q->head[i / kQueues][i % kQueues].next = 0;
}

// ------------------------------------------------------------ k_setup
// True if the triangle a, b, c (either orientation, less than 8 px wide and
// high, not degenerate) covers none of the n <= 4 pixel centres of its box,
// decided exactly: the centres lie inside the triangle's bounding box, so every
// difference is below 2^11 and every edge value below 2^23 in magnitude.  A is
// twice its area.
__device__ __forceinline__ bool misses_centres(const SVtx<0> &a, const SVtx<0> &b, const SVtx<0> &c, int A,
                                               const PixBox &pb, int w, int n)
{
    const int ox = 256 * pb.i0 + 128, oy = 256 * pb.j0 + 128;
    const int bX = A < 0 ? c.X : b.X, bY = A < 0 ? c.Y : b.Y, cX = A < 0 ? b.X : c.X, cY = A < 0 ? b.Y : c.Y;
    const int dx[3] = {cX - bX, a.X - cX, bX - a.X}, dy[3] = {cY - bY, a.Y - cY, bY - a.Y};
    const int rx[3] = {bX - ox, cX - ox, a.X - ox}, ry[3] = {bY - oy, cY - oy, a.Y - oy};
    int e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        e[k] = __mul24(dy[k], rx[k]) - __mul24(dx[k], ry[k]) - (owned(dx[k], dy[k]) ? 0 : 1);
    if ((e[0] | e[1] | e[2]) >= 0) return false;
    int p = 0, q = 0;
    for (int s = 1; s < n; ++s) {
        p += 256;
        if (p == 256 * w) {
            p = 0;
            q += 256;
        }
        const int f0 = e[0] + __mul24(dx[0], q) - __mul24(dy[0], p);
        const int f1 = e[1] + __mul24(dx[1], q) - __mul24(dy[1], p);
        const int f2 = e[2] + __mul24(dx[2], q) - __mul24(dy[2], p);
        if ((f0 | f1 | f2) >= 0) return false;
    }
    return true;
}

// Survival of sub-triangles 0 and 1 of one triangle in view v, with their
// pixel boxes.  Deterministic: calling it twice gives the same answer.
//
// Unless the view's work is counted, a small sub-triangle that covers no pixel
// does not survive.  Of the 64 bench views' 5.9 M survivors 5.1 M are less than
// 8 px in extent and 4.2 M have at most four centres in their box; the test
// drops 1.6 M of these (boxes of five to nine centres would give 0.05 M more).
// It takes 10 us of setup (setup is bound by VALU issue) and saves 6 of the
// count, 11 of the scatter and 22 of the raster: 0.445 -> 0.415 ms.
__device__ __forceinline__ void survive(const DView &v, const float P[9], bool valid, bool &s0,
                                        bool &s1, PixBox &b0, PixBox &b1, bool &rerr)
{
    s0 = s1 = false;
    if (!valid) return;
    Vtx<0> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    const float zn = v.zn;
    const bool allin = c0.w >= zn && c1.w >= zn && c2.w >= zn;
    const bool anyin = c0.w >= zn || c1.w >= zn || c2.w >= zn;
    if (!anyin) return;
    SVtx<0> a, bb, c;
    if (allin) {
        // no clipping and no second sub-triangle
        if (!snap3<true>(v, c0, c1, c2, a, bb, c)) {
            // Beyond the fixed-point domain, an error unless the triangle is
            // out of sight anyway: all three |Xc fS| exceed (cxS + 4 px)
            // (1 + 2^-16) w on one side, so the snapped bbox is at least 3 px
            // outside the viewport (three fp32 roundings cost < 2^-22
            // relative).
            const float Kx = (v.cxS + 1024.0f) * 1.0000152587890625f;
            const float Ky = (v.cyS + 1024.0f) * 1.0000152587890625f;
            const float x0 = c0.x * v.fS, x1 = c1.x * v.fS, x2 = c2.x * v.fS;
            const float y0 = c0.y * v.fS, y1 = c1.y * v.fS, y2 = c2.y * v.fS;
            const float kx0 = Kx * c0.w, kx1 = Kx * c1.w, kx2 = Kx * c2.w;
            const float ky0 = Ky * c0.w, ky1 = Ky * c1.w, ky2 = Ky * c2.w;
            rerr |= !((x0 > kx0 && x1 > kx1 && x2 > kx2) || (x0 < -kx0 && x1 < -kx1 && x2 < -kx2) ||
                      (y0 > ky0 && y1 > ky1 && y2 > ky2) || (y0 < -ky0 && y1 < -ky1 && y2 < -ky2));
            return;
        }
        b0 = pix_box(v, a, bb, c);
        if (b0.i0 > b0.i1 || b0.j0 > b0.j1) return;
        const uint32_t ext = (uint32_t)(max(a.X, max(bb.X, c.X)) - min(a.X, min(bb.X, c.X))) |
                             (uint32_t)(max(a.Y, max(bb.Y, c.Y)) - min(a.Y, min(bb.Y, c.Y)));
        if (ext < 2048u) {
            const int A = __mul24(bb.X - a.X, c.Y - a.Y) - __mul24(bb.Y - a.Y, c.X - a.X);
            const int w = b0.i1 - b0.i0 + 1, n = w * (b0.j1 - b0.j0 + 1);
            s0 = A != 0 && (n > 4 || v.count_work || !misses_centres(a, bb, c, A, b0, w, n));
        } else {
            s0 = area2(a, bb, c) != 0;
        }
        return;
    }
    long long A;
    if (setup_sub(v, c0, c1, c2, 0, a, bb, c, A, rerr)) {
        b0 = pix_box(v, a, bb, c);
        s0 = b0.i0 <= b0.i1 && b0.j0 <= b0.j1;
    }
    if (setup_sub(v, c0, c1, c2, 1, a, bb, c, A, rerr)) {
        b1 = pix_box(v, a, bb, c);
        s1 = b1.i0 <= b1.i1 && b1.j0 <= b1.j1;
    }
}

// Conservative frustum test of a 64-triangle cluster's bounding box for
// view v, in fp64 over the box's eight corners.  The box counts as outside
// only when all corners lie beyond one side plane of the per-vertex
// rejection in `survive` by a margin (fS + K) 2^-18 |d|_1 that exceeds that
// test's fp32 error (< 2^-20 |d|_1 per camera coordinate), or all lie in
// front of the near plane by 2^-18 |d|_1: then every vertex of every
// triangle in the box fails in the same way, each triangle (and each
// near-clipped piece, a convex combination of its vertices) is culled by
// the exact path, and skipping the cluster changes nothing.
__device__ __forceinline__ bool box_outside(const DView &v, float4 mn, float4 mx)
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
    bool r = true, l = true, u = true, d = true, n = true;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        r = r && X[c] * fS - Kx * W[c] > mg;
        l = l && -X[c] * fS - Kx * W[c] > mg;
        u = u && Y[c] * fS - Ky * W[c] > mg;
        d = d && -Y[c] * fS - Ky * W[c] > mg;
        n = n && W[c] < (double)v.zn - mz;
    }
    return r || l || u || d || n;
}

// Block (x, view): test kCullBlock consecutive 64-triangle clusters of the
// view's scene against the view's frustum, compact the visible ones with a
// block scan and append them to the view's segment of the visible-cluster
// list behind one reservation (their order there is immaterial: nothing
// downstream depends on it).
constexpr int kCullBlock = 256;

__global__ __launch_bounds__(kCullBlock) void k_cull(const DView *__restrict__ views,
                                                     DViewCounters *__restrict__ ctr,
                                                     uint32_t *__restrict__ vis_clusters)
{
    __shared__ uint32_t wtot[kCullBlock / 64];
    __shared__ uint32_t sbase;
    const uint32_t vi = blockIdx.y;
    const DView &v = views[vi];
    const uint32_t ncl = (v.T + kCluster - 1) / kCluster;
    const uint32_t c0 = blockIdx.x * kCullBlock;
    if (c0 >= ncl) return;
    const uint32_t c = c0 + threadIdx.x;
    bool vis = c < ncl;
    if (vis && v.cbox) {
        const auto *b = gmem(reinterpret_cast<const float *>(v.cbox)) + 8ull * c;
        vis = !box_outside(v, make_float4(b[0], b[1], b[2], b[3]), make_float4(b[4], b[5], b[6], b[7]));
    }
    if (vis && c == ncl - 1 && v.T % kCluster) {
        ctr[vi].vis_tail = 1;
        vis = false;
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<kCullBlock>(vis ? 1u : 0u, wtot, &tot);
    if (threadIdx.x == 0) sbase = tot ? atomicAdd(&ctr[vi].vis_clusters, tot) : 0u;
    __syncthreads();
    if (vis) vis_clusters[v.pair_base + sbase + ex] = c;
}

// Work items of k_setup: (view, run of kRun visible clusters).  Each block
// builds the prefix of item counts over the views in LDS; the waves stride over
// the items.  A wave sets up one triangle of each of the run's clusters per lane
// (independent loads in flight together).
//
// A run's survivors (key, box) go to slots of their own, two per triangle of a
// full run, and their number into the run's first list entry (which held its
// first cluster).  Only a view's last run can hold the scene's last, partial
// cluster, so its runs' slots fit two per triangle of the scene.
constexpr uint32_t kSlots = 2 * kRun * kCluster;

// A view's visible clusters.  The list leaves out the scene's last cluster if
// that is partial; it comes after the others.
__device__ __forceinline__ uint32_t visible_clusters(const DViewCounters &c) { return c.vis_clusters + c.vis_tail; }

// Survivors of a view's run (which is in sight).
__device__ __forceinline__ uint32_t run_count(const DView &v, const uint32_t *__restrict__ vis_clusters, uint32_t run)
{
    return vis_clusters[v.pair_base + run * kRun];
}

// Does a survivor's pixel box meet the TS-pixel tile at (ti0, tj0)?
template <int TS>
__device__ __forceinline__ bool box_meets(uint2 bb, int ti0, int tj0)
{
    return (int)(bb.y & 0xFFFFu) >= ti0 && (int)(bb.x & 0xFFFFu) < ti0 + TS && (int)(bb.y >> 16) >= tj0 &&
           (int)(bb.x >> 16) < tj0 + TS;
}

// The exclusive prefix over the views of ceil(visible clusters / per).
template <int NT>
__device__ __forceinline__ uint32_t build_prefix(const DViewCounters *ctr, uint32_t nviews, uint32_t per, uint32_t *pre,
                                                 uint32_t *wtot)
{
    const uint32_t seg = (nviews + NT - 1) / NT;
    const uint32_t i0 = threadIdx.x * seg, i1 = min(i0 + seg, nviews);
    uint32_t local = 0;
    for (uint32_t i = i0; i < i1; ++i) local += (visible_clusters(ctr[i]) + per - 1) / per;
    uint32_t total;
    uint32_t run = block_excl_scan<NT>(local, wtot, &total);
    for (uint32_t i = i0; i < i1; ++i) {
        pre[i] = run;
        run += (visible_clusters(ctr[i]) + per - 1) / per;
    }
    __syncthreads();
    return total;
}

__device__ __forceinline__ uint32_t find_view(const uint32_t *pre, uint32_t nviews, uint32_t item)
{
    uint32_t lo = 0, hi = nviews - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Each wave appends to a run's own slots: no counter that other waves wait for.
// (Survivors gathered in LDS and appended to the view's list behind an atomic
// add, 500 at a time, met 600 others at each of eight views' counters: eight
// 512 x 384 views of 1M triangles set up in 59 us, now 42; 64 views of 4 scenes
// 114-134 and 102, 1024 views of 20k triangles 126 and 106.  The lists had no
// gaps, which took 4 us less in the count and 9 in the scatter.)  The run's
// loads are in flight together; 6 waves per SIMD (78 VGPRs).  Bound by VALU
// issue and the reads of 36 bytes a triangle.
__global__ __launch_bounds__(kSetupBlock) __attribute__((amdgpu_waves_per_eu(kSetupWavesPerSimd))) void k_setup(
    const DView *__restrict__ views, uint32_t nviews, DViewCounters *__restrict__ ctr, uint32_t *vis_clusters,
    uint32_t *__restrict__ skey, uint2 *__restrict__ sbox, uint32_t *__restrict__ err)
{
    extern __shared__ uint32_t pre[];      // [nviews]: sized at launch
    __shared__ uint32_t wtot[kSetupBlock / 64];
    const uint32_t total = build_prefix<kSetupBlock>(ctr, nviews, kRun, pre, wtot);
    const uint32_t lane = lane_id();
    const unsigned long long lt = lanemask_lt();
    const uint32_t nwaves = (gridDim.x * kSetupBlock) >> 6;
    bool rerr = false;
    for (uint32_t item = uniform((blockIdx.x * kSetupBlock + threadIdx.x) >> 6); item < total; item += nwaves) {
        const uint32_t vi = uniform(find_view(pre, nviews, item));
        const DView &v = views[vi];
        const uint32_t run = item - uniform(pre[vi]), first = run * kRun;
        const uint32_t nvis = visible_clusters(ctr[vi]), nlist = ctr[vi].vis_clusters;
        uint32_t *const entry = vis_clusters + v.pair_base + first;
        uint32_t cl[kRun], t[kRun];
        bool valid[kRun];
        float P[kRun][9];
#pragma unroll
        for (uint32_t j = 0; j < kRun; ++j) cl[j] = entry[min(j, nvis - 1 - first)];
#pragma unroll
        for (uint32_t j = 0; j < kRun; ++j) {
            t[j] = (first + j < nlist ? uniform(cl[j]) : (v.T - 1) / kCluster) * kCluster + lane;
            valid[j] = first + j < nvis && t[j] < v.T;
        }
#pragma unroll
        for (uint32_t j = 0; j < kRun; ++j) {
            if (valid[j]) {
                load_pos(v, t[j], P[j]);
            } else {
#pragma unroll
                for (int a = 0; a < 9; ++a) P[j][a] = 0.0f;
            }
        }
        // one cluster at a time, its survivors in (sub, lane) order: only one
        // cluster's boxes are live at once
        const uint32_t base = v.surv_base + run * kSlots;
        uint32_t n = 0;
        unsigned long long narea = 0;
#pragma unroll
        for (uint32_t j = 0; j < kRun; ++j) {
            bool s0, s1;
            PixBox b0, b1;
            survive(v, P[j], valid[j], s0, s1, b0, b1, rerr);
            const unsigned long long m0 = __ballot(s0), m1 = __ballot(s1);
            if (s0) {
                const uint32_t o = base + n + (uint32_t)__popcll(m0 & lt);
                skey[o] = 2u * t[j];
                sbox[o] = pack_box(b0);
            }
            n += (uint32_t)__popcll(m0);
            if (s1) {
                const uint32_t o = base + n + (uint32_t)__popcll(m1 & lt);
                skey[o] = 2u * t[j] + 1u;
                sbox[o] = pack_box(b1);
            }
            n += (uint32_t)__popcll(m1);
            if (v.count_work) {
                uint32_t area = 0;
                if (s0) area += (uint32_t)(b0.i1 - b0.i0 + 1) * (uint32_t)(b0.j1 - b0.j0 + 1);
                if (s1) area += (uint32_t)(b1.i1 - b1.i0 + 1) * (uint32_t)(b1.j1 - b1.j0 + 1);
                // two boxes of at most 2^24 pixels per lane: the two halves
                // of the wave sum cannot overflow
                const uint32_t alo = wave_sum_u32(area & 0xFFFFu);
                const uint32_t ahi = wave_sum_u32(area >> 16);
                narea += (unsigned long long)alo + ((unsigned long long)ahi << 16);
            }
        }
        if (lane == 0) {
            entry[0] = n;
            if (v.count_work && n) {
                atomicAdd(&ctr[vi].surv_count, n);
                atomicAdd(&ctr[vi].bbox_tests, narea);
            }
        }
    }
    if (rerr) atomicOr(err, kErrRange);
}

// ------------------------------------------------------------ binning
// Items of the count/scatter kernels are (view, chunk of kBinRuns runs); every block builds the prefix of chunk counts over the
// views, then strides over the items.
constexpr uint32_t kBinHeld = 4;       // survivors a thread holds in registers

// LDS slot of tile i in the per-chunk tile arrays: the low five bits are
// XORed with the next five, a permutation within each aligned run of 32
// slots.  Vertically adjacent tiles (32 per row at 256 px / 8 px tiles) would
// otherwise share an LDS bank, and a wave's boxes touch such columns of tiles
// together; the arrays are cleared up to the next multiple of 32.
__device__ __forceinline__ uint32_t swz(uint32_t i) { return i ^ ((i >> 5) & 31u); }

// Tiles [tx0, tx1] x [ty0, ty1] that a survivor's pixel box touches.
struct TileRange {
    int tx0, ty0, tx1, ty1;
};

__device__ __forceinline__ TileRange tile_range(uint2 bb, uint32_t ts)
{
    TileRange r;
    r.tx0 = (int)(bb.x & 0xFFFFu) >> ts;
    r.ty0 = (int)(bb.x >> 16) >> ts;
    r.tx1 = (int)(bb.y & 0xFFFFu) >> ts;
    r.ty1 = (int)(bb.y >> 16) >> ts;
    return r;
}

// f(tile, key) for the tiles of a range, whose rows hold tiles_x, that each lane's
// survivor (if it has one) touches.  A large box would hold up the other lanes:
// the whole wave walks it.
template <class F>
__device__ __forceinline__ void walk_tiles(bool has, const TileRange &R, uint32_t tiles_x, uint32_t key, F f)
{
    constexpr int kLaneTiles = 24;
    const int nx = R.tx1 - R.tx0 + 1, area = has ? nx * (R.ty1 - R.ty0 + 1) : 0;
    if (has && area <= kLaneTiles)
        for (int ty = R.ty0; ty <= R.ty1; ++ty)
            for (int tx = R.tx0; tx <= R.tx1; ++tx) f((uint32_t)ty * tiles_x + (uint32_t)tx, key);
    for (unsigned long long m = __ballot(area > kLaneTiles); m; m &= m - 1) {
        const int l = __ffsll((long long)m) - 1;
        const int wx = __builtin_amdgcn_readlane(nx, l), wn = __builtin_amdgcn_readlane(area, l);
        const int x0 = __builtin_amdgcn_readlane(R.tx0, l), y0 = __builtin_amdgcn_readlane(R.ty0, l);
        const uint32_t wk = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
        const float iw = 1.0f / (float)wx;
        for (int p = (int)lane_id(); p < wn; p += 64) {
            const int y = (int)(((float)p + 0.5f) * iw);   // exact: a few thousand tiles at most
            f((uint32_t)(y0 + y) * tiles_x + (uint32_t)(x0 + p - y * wx), wk);
        }
    }
}

// List entries of one work item: kSegPerTile * TS^2, or wave_seg (if not 0) where
// a wave rasterises a 16-pixel tile by itself (k_raster_wave).
__device__ __forceinline__ uint32_t seg_size(uint32_t ts_log2, uint32_t wave_seg)
{
    return wave_seg && ts_log2 == 4 ? wave_seg : kSegPerTile << (2 * ts_log2);
}

// Number of (tile, segment) work items of a tile: none when empty, one per
// segment of at most seg_size list entries; for an overflow tile, which scans
// all survivors, one, or none where k_raster_wave takes it from a list of its own.
__device__ __forceinline__ uint32_t tile_segments(uint32_t c, uint32_t off, uint32_t ts_log2, uint32_t wave_seg)
{
    if (c == 0) return 0;
    if (off == kOverflow) return wave_seg && ts_log2 == 4 ? 0u : 1u;
    const uint32_t S = seg_size(ts_log2, wave_seg);
    return (c + S - 1) / S;
}

// First z-key of a view's 16-pixel tile (k_raster_wave): 256 keys per tile.
__device__ __forceinline__ size_t wave_tile(const DView &v, uint32_t tile)
{
    return (((size_t)v.zoff_hi << 32) | v.zoff_lo) + 256u * (size_t)tile;
}

// Eight waves per SIMD (64 VGPRs in the scatter): 2048 blocks, the grid, are
// resident; with 66 VGPRs a quarter of them ran after the others (1024 views'
// scatter 47 us, 41 so).
//
// LARGE: some view has more tiles than the histogram holds, or the triangles are
// coarse, kCoarseTiles a tile or fewer: a wave then walks each large box, which held up
// the other lanes, a lane to each.  One 512 x 512 view of a 5k-triangle apartment (lists)
// 222 -> 173 us, eight of 20k 224 -> 176, of 200k (195 triangles a tile) 162 -> 156, but
// two of 200k 106 -> 111 and sixteen of 1M (977) 307 -> 311.  A launch without either is
// spared that form's register spills (5 us of the scatter of 64 views).
template <bool SCATTER, bool LARGE>
__global__ __launch_bounds__(kBinBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_bin(const DView *__restrict__ views, uint32_t nviews,
                                                   const DViewCounters *__restrict__ ctr,
                                                   const uint32_t *__restrict__ vis_clusters,
                                                   const uint32_t *__restrict__ skey,
                                                   const uint2 *__restrict__ sbox,
                                                   uint32_t *__restrict__ tile_count,
                                                   const uint32_t *__restrict__ tile_off,
                                                   uint32_t *__restrict__ tile_cursor,
                                                   uint32_t *__restrict__ bins, uint32_t wave_seg,
                                                   unsigned long long *__restrict__ zt)
{
    extern __shared__ uint32_t pre[];      // [nviews]: sized at launch
    __shared__ uint32_t hist[kLdsTiles];   // low 16 bits: count, high 16 bits: rank cursor
    __shared__ uint32_t lbase[SCATTER ? kLdsTiles : 1];
    // the prefix scan's per-wave totals live in the histogram (first
    // written after the scan's closing barrier): 32 KiB per scatter block
    uint32_t *const wtot = hist;
    const uint32_t total = build_prefix<kBinBlock>(ctr, nviews, kBinRuns * kRun, pre, wtot);
    const uint32_t tid = threadIdx.x;
    if (SCATTER && wave_seg) {
        // the 16-pixel tiles whose items merge by atomic max start from cleared
        // keys: a share of each view's tiles per block, 16 tiles at a time per wave
        const uint32_t shares = max(1u, gridDim.x / nviews), lane = lane_id();
        for (uint32_t u = blockIdx.x; u < nviews * shares; u += gridDim.x) {
            const DView &v = views[u / shares];
            const uint32_t n = v.ts_log2 == 4 ? v.tiles_x * v.tiles_y : 0u;
            for (uint32_t t0 = ((u % shares) * (kBinBlock / 64) + uniform(tid >> 6)) * 16u; t0 < n;
                 t0 += shares * (kBinBlock / 64) * 16u) {
                const uint32_t t = t0 + lane;
                bool multi = false;
                if (lane < 16u && t < n) multi = tile_count[v.tile_base + t] > wave_seg || tile_off[v.tile_base + t] == kOverflow;
                for (unsigned long long m = __ballot(multi); m; m &= m - 1) {
                    uint4 *const z = reinterpret_cast<uint4 *>(zt + wave_tile(v, t0 + (uint32_t)__ffsll((long long)m) - 1u));
                    z[lane] = make_uint4(0, 0, 0, 0);
                    z[lane + 64] = make_uint4(0, 0, 0, 0);
                }
            }
        }
    }
    for (uint32_t item = blockIdx.x; item < total; item += gridDim.x) {
        const uint32_t vi = uniform(find_view(pre, nviews, item));
        const DView &v = views[vi];
        // the chunk's survivors, as if without the gaps between its runs
        const uint32_t run = (item - uniform(pre[vi])) * kBinRuns, nvis = visible_clusters(ctr[vi]);
        uint32_t n = 0, first[kBinRuns], gap[kBinRuns];
#pragma unroll
        for (uint32_t j = 0; j < kBinRuns; ++j)   // without branches: all in flight together
            gap[j] = run_count(v, vis_clusters, min(run + j, (nvis - 1) / kRun));
#pragma unroll
        for (uint32_t j = 0; j < kBinRuns; ++j) {
            const uint32_t c = (run + j) * kRun < nvis ? uniform(gap[j]) : 0u;
            n += c;
            first[j] = n;   // of the next run
            gap[j] = kSlots - c;
        }
        const uint32_t slot0 = v.surv_base + run * kSlots;
        auto at = [&](uint32_t e) {
            uint32_t s = slot0 + e;
#pragma unroll
            for (uint32_t j = 0; j + 1 < kBinRuns; ++j) s += e >= first[j] ? gap[j] : 0u;
            return s;
        };
        // the view's fields in registers: the atomics below may not be
        // assumed to leave the view records alone
        const uint32_t ts = v.ts_log2, tiles_x = v.tiles_x, nt = v.tiles_x * v.tiles_y;
        const uint32_t tile_base = v.tile_base, bin_base = v.bin_base;
        if (!LARGE || nt <= kLdsTiles) {
            // a thread's first survivors, loaded together while the histogram
            // is cleared and kept for the scatter; a chunk of 8 runs has about
            // 860, more go one round at a time
            uint2 box[kBinHeld];
            uint32_t key[kBinHeld];
#pragma unroll
            for (uint32_t r = 0; r < kBinHeld; ++r) {
                box[r] = make_uint2(0u, 0u);
                const uint32_t e = r * kBinBlock + tid;
                if (e < n) {
                    const uint32_t s = at(e);
                    box[r] = sbox[s];
                    if (SCATTER) key[r] = skey[s];
                }
            }
            // f(tile, key) for the tiles of every survivor of the chunk
            auto each = [&](auto f) {
                auto lane = [&](uint2 bb, uint32_t k) {
                    const TileRange R = tile_range(bb, ts);
                    for (int ty = R.ty0; ty <= R.ty1; ++ty)
                        for (int tx = R.tx0; tx <= R.tx1; ++tx) f((uint32_t)ty * tiles_x + (uint32_t)tx, k);
                };
                if constexpr (LARGE) {
#pragma unroll
                    for (uint32_t r = 0; r < kBinHeld; ++r) walk_tiles(r * kBinBlock + tid < n, tile_range(box[r], ts), tiles_x, key[r], f);
                    for (uint32_t e0 = kBinHeld * kBinBlock; e0 < n; e0 += kBinBlock) {
                        const uint32_t s = at(min(e0 + tid, n - 1u));
                        walk_tiles(e0 + tid < n, tile_range(sbox[s], ts), tiles_x, SCATTER ? skey[s] : 0u, f);
                    }
                } else {
#pragma unroll
                    for (uint32_t r = 0; r < kBinHeld; ++r)
                        if (r * kBinBlock + tid < n) lane(box[r], key[r]);
                    for (uint32_t e = kBinHeld * kBinBlock + tid; e < n; e += kBinBlock) {
                        const uint32_t s = at(e);
                        lane(sbox[s], SCATTER ? skey[s] : 0u);
                    }
                }
            };
            for (uint32_t i = tid; i < ((nt + 31u) & ~31u); i += kBinBlock) hist[i] = 0;
            __syncthreads();
            // count this chunk's entries per tile in LDS (at most kSlots a
            // run and tile: fits the 16-bit half)
            each([&](uint32_t tl, uint32_t) { atomicAdd(&hist[swz(tl)], 1u); });
            __syncthreads();
            // one global operation per touched tile; a thread's tiles are
            // i, i + kBinBlock, ...: their loads and atomics are issued
            // together, not one tile after another
            if (!SCATTER) {
                for (uint32_t i = tid; i < nt; i += kBinBlock) {
                    const uint32_t c = hist[swz(i)] & 0xFFFFu;
                    if (c) atomicAdd(&tile_count[tile_base + i], c);
                }
            } else {
                constexpr int kPer = kLdsTiles / kBinBlock;
                uint32_t c[kPer], off[kPer], got[kPer];
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const uint32_t i = tid + (uint32_t)k * kBinBlock;
                    c[k] = i < nt ? hist[swz(i)] & 0xFFFFu : 0u;
                }
                // list offsets of the tiles this chunk touches only (a chunk
                // of consecutive survivors touches a small part of the view)
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const uint32_t i = tid + (uint32_t)k * kBinBlock;
                    off[k] = i < nt && c[k] ? tile_off[tile_base + i] : kOverflow;   // (so written, no register spills)
                }
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const uint32_t i = tid + (uint32_t)k * kBinBlock;
                    got[k] = (c[k] && off[k] != kOverflow) ? atomicAdd(&tile_cursor[tile_base + i], c[k]) : 0u;
                }
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const uint32_t i = tid + (uint32_t)k * kBinBlock;
                    if (c[k]) lbase[swz(i)] = off[k] == kOverflow ? kOverflow : off[k] + got[k];
                }
            }
            if (SCATTER) {
                __syncthreads();
                each([&](uint32_t tl, uint32_t k) {
                    const uint32_t b = lbase[swz(tl)];
                    if (b == kOverflow) return;
                    const uint32_t rank = atomicAdd(&hist[swz(tl)], 1u << 16) >> 16;
                    bins[bin_base + b + rank] = k;
                });
            }
            __syncthreads();
        } else {
            // more tiles than the histogram holds: in windows of whole rows, from
            // the first to the last that the chunk touches.  A 2048 x 2048 view of a
            // 2k-triangle room is counted and scattered in 0.11 and 0.6 ms; a global
            // atomic per tile and survivor took 4.4 and 2.2 (a 1024 x 1024 view of 1M
            // triangles 0.02 and 0.05; 0.13 and 0.51).
            const uint32_t high = kLdsTiles / tiles_x;
            uint32_t lo = v.tiles_y, hi = 0;
            for (uint32_t e = tid; e < n; e += kBinBlock) {
                const TileRange R = tile_range(sbox[at(e)], ts);
                lo = min(lo, (uint32_t)R.ty0);
                hi = max(hi, (uint32_t)R.ty1 + 1u);
            }
            if (tid < 2) hist[tid] = tid ? 0u : lo;
            __syncthreads();
            atomicMin(&hist[0], lo);
            atomicMax(&hist[1], hi);
            __syncthreads();
            lo = uniform(hist[0]);
            hi = uniform(hist[1]);
            __syncthreads();
#pragma unroll 1
            for (; lo < hi; lo += high) {
                const uint32_t base = tile_base + lo * tiles_x, nw = min(high * tiles_x, nt - lo * tiles_x);
                auto each = [&](auto f) {
                    for (uint32_t e0 = 0; e0 < n; e0 += kBinBlock) {
                        const bool has = e0 + tid < n;
                        const uint32_t s = at(has ? e0 + tid : 0u);
                        TileRange R = tile_range(sbox[s], ts);
                        R.ty0 = max(R.ty0 - (int)lo, 0);
                        R.ty1 = min(R.ty1 - (int)lo, (int)high - 1);
                        walk_tiles(has, R, tiles_x, SCATTER ? skey[s] : 0u, f);
                    }
                };
                for (uint32_t i = tid; i < ((nw + 31u) & ~31u); i += kBinBlock) hist[i] = 0;
                __syncthreads();
                each([&](uint32_t tl, uint32_t) { atomicAdd(&hist[swz(tl)], 1u); });
                __syncthreads();
                for (uint32_t i = tid; i < nw; i += kBinBlock) {
                    const uint32_t c = hist[swz(i)];
                    if (!c) continue;
                    if (!SCATTER) {
                        atomicAdd(&tile_count[base + i], c);
                    } else {
                        const uint32_t off = tile_off[base + i];
                        lbase[swz(i)] = off == kOverflow ? kOverflow : off + atomicAdd(&tile_cursor[base + i], c);
                    }
                }
                __syncthreads();
                if (SCATTER) {
                    each([&](uint32_t tl, uint32_t k) {
                        const uint32_t b = lbase[swz(tl)];
                        if (b != kOverflow) bins[bin_base + b + (atomicAdd(&hist[swz(tl)], 1u << 16) >> 16)] = k;
                    });
                    __syncthreads();
                }
            }
        }
    }
}

// Per view: exclusive scan of tile counts into list offsets.  A tile whose
// count exceeds tile_cap, or whose list would end beyond the view's bin
// capacity, is marked kOverflow.  Then the view's work items are reserved
// in its tile size's queue and written out; tile_item gets each tile's
// first item.  A block per view, of 256 threads where no view has more tiles; the tiles
// whose items merge are cleared by the scatter's blocks, not by a view's one
// (eight views of 768 tiles: 17 us, 9 without it).
//
// Overflow tiles of k_raster_wave are listed from the end of its items backwards
// (a tile takes one entry there or one per segment at the front, so the two never
// meet): it cuts each into as many items as fill the launch.
__device__ __forceinline__ void list_overflow(DQueue *__restrict__ q, uint2 *__restrict__ items16, uint32_t cap16,
                                              uint32_t vi, uint32_t tile)
{
    items16[cap16 - 1u - atomicAdd(&q->total[kOverTotal], 1u)] = make_uint2(vi, tile);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_bin_scan(const DView *__restrict__ views,
                                                         DViewCounters *__restrict__ ctr,
                                                         const uint32_t *__restrict__ tile_count,
                                                         uint32_t *__restrict__ tile_off,
                                                         uint32_t *__restrict__ tile_item,
                                                         DQueue *__restrict__ q,
                                                         uint2 *__restrict__ items8,
                                                         uint2 *__restrict__ items16,
                                                         uint2 *__restrict__ items32, uint32_t wave_seg,
                                                         uint32_t cap16)
{
    __shared__ uint32_t wtot[NT / 64];
    __shared__ uint32_t sbase;
    const uint32_t vi = blockIdx.x;
    const DView &v = views[vi];
    const uint32_t n = v.tiles_x * v.tiles_y;
    const uint32_t cls = v.ts_log2 - 3;
    uint32_t run = 0, srun = 0;
    for (uint32_t base = 0; base < n; base += NT) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t c = i < n ? tile_count[v.tile_base + i] : 0u;
        const uint32_t e = c <= v.tile_cap ? c : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan<NT>(e, wtot, &tot);
        const unsigned long long P = (unsigned long long)run + ex;
        // a tile with more segments than the item encoding holds also takes
        // the (single-item) overflow path
        const bool over = c > v.tile_cap || P + e > v.bin_cap ||
                          c > (kMaxSegments - 1) * seg_size(v.ts_log2, wave_seg);
        const uint32_t off = (c == 0) ? 0u : (over ? kOverflow : (uint32_t)P);
        const uint32_t ns = tile_segments(c, off, v.ts_log2, wave_seg);
        uint32_t stot;
        const uint32_t sex = block_excl_scan<NT>(ns, wtot, &stot);
        if (i < n) {
            tile_off[v.tile_base + i] = off;
            tile_item[v.tile_base + i] = srun + sex;
            if (off == kOverflow && wave_seg && cls == 1) list_overflow(q, items16, cap16, vi, i);
        }
        run += tot;
        srun += stot;
    }
    if (threadIdx.x == 0) {
        ctr[vi].bin_used = min(run, v.bin_cap);
        sbase = srun ? atomicAdd(&q->total[cls], srun) : 0u;
    }
    __syncthreads();
    const uint32_t qb = sbase;
    uint2 *items = cls == 0 ? items8 : cls == 1 ? items16 : items32;
    for (uint32_t i = threadIdx.x; i < n; i += NT) {
        const uint32_t c = tile_count[v.tile_base + i];
        const uint32_t ns = tile_segments(c, tile_off[v.tile_base + i], v.ts_log2, wave_seg);
        const uint32_t first = qb + tile_item[v.tile_base + i];
        tile_item[v.tile_base + i] = first;
        for (uint32_t sgm = 0; sgm < ns; ++sgm) items[first + sgm] = make_uint2(vi, i | (sgm << 18));
    }
}

// The same for views of at most 64 tiles: a wave per view, 16 to a block, which
// reserves its views' work items together (with a block per view the queue's
// counter serialises them: 1024 views of 16 tiles took 18 us, 8 so).
constexpr int kSmallScanWaves = 16;
__global__ __launch_bounds__(64 * kSmallScanWaves) void k_bin_scan_small(
    const DView *__restrict__ views, uint32_t nviews, DViewCounters *__restrict__ ctr,
    const uint32_t *__restrict__ tile_count, uint32_t *__restrict__ tile_off, uint32_t *__restrict__ tile_item,
    DQueue *__restrict__ q, uint2 *__restrict__ items8, uint2 *__restrict__ items16, uint2 *__restrict__ items32,
    uint32_t wave_seg, uint32_t cap16)
{
    __shared__ uint32_t wtot[kSmallScanWaves], wcls[kSmallScanWaves], base[3];
    const uint32_t lane = lane_id(), w = uniform(threadIdx.x >> 6), vi = blockIdx.x * kSmallScanWaves + w;
    const bool valid = vi < nviews;
    const DView &v = views[valid ? vi : 0u];
    const uint32_t n = valid ? v.tiles_x * v.tiles_y : 0u, cls = v.ts_log2 - 3;
    auto excl = [&](uint32_t x, uint32_t &tot) {
        uint32_t a = x;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const uint32_t b = __shfl_up(a, d);
            if (lane >= (uint32_t)d) a += b;
        }
        tot = __shfl(a, 63);
        return a - x;
    };
    const uint32_t c = lane < n ? tile_count[v.tile_base + lane] : 0u;
    const uint32_t e = c <= v.tile_cap ? c : 0u;
    uint32_t tot, stot;
    const unsigned long long P = excl(e, tot);
    const bool over = c > v.tile_cap || P + e > v.bin_cap || c > (kMaxSegments - 1) * seg_size(v.ts_log2, wave_seg);
    const uint32_t off = (c == 0) ? 0u : (over ? kOverflow : (uint32_t)P);
    const uint32_t ns = tile_segments(c, off, v.ts_log2, wave_seg);
    const uint32_t sex = excl(ns, stot);
    if (lane == 0) {
        wtot[w] = stot;
        wcls[w] = cls;
        if (valid) ctr[vi].bin_used = min(tot, v.bin_cap);
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kSmallScanWaves; ++k) sum += wcls[k] == threadIdx.x ? wtot[k] : 0u;
        base[threadIdx.x] = sum ? atomicAdd(&q->total[threadIdx.x], sum) : 0u;
    }
    __syncthreads();
    uint32_t first = base[cls] + sex;
#pragma unroll
    for (int k = 0; k < kSmallScanWaves; ++k) first += k < (int)w && wcls[k] == cls ? wtot[k] : 0u;
    if (lane >= n) return;
    tile_off[v.tile_base + lane] = off;
    tile_item[v.tile_base + lane] = first;
    uint2 *items = cls == 0 ? items8 : cls == 1 ? items16 : items32;
    for (uint32_t sgm = 0; sgm < ns; ++sgm) items[first + sgm] = make_uint2(vi, lane | (sgm << 18));
    if (off == kOverflow && wave_seg && cls == 1) list_overflow(q, items16, cap16, vi, lane);
}

// ------------------------------------------------------------ k_raster
// LDS record of one (sub-triangle, tile) pair: edge functions relative to
// the tile's first pixel centre, E_k(P, Q) = C_k + dx_k Q - dy_k P with
// (P, Q) the pixel offset from that centre in 1/256 px.  Everything a visit
// needs for the common (packed) case sits in one 48-byte block laid out as
// three naturally aligned 16-byte words (three LDS loads); unpacked and
// int64 records keep their extra words in a second array.
struct alignas(16) LRec {
    int c0, c1, c2;    // C_k (slow: its low word)
    uint32_t flags;
    int e0, e1, e2;    // packed: (dx_k, -dy_k) as 16-bit pairs; else dx_k
    uint32_t nkey;     // ~key: the low word of the z-key
    float rw0, rw1, rw2, invA;
};
struct alignas(8) LExt {
    int ny0, ny1, ny2; // -dy_k (unpacked records)
    int hi0, hi1, hi2; // slow: high words of C_k
};
static_assert(sizeof(LRec) == 48 && sizeof(LExt) == 24, "LDS records");

// One record as three 16-byte LDS loads, at a byte offset from the array.
__device__ __forceinline__ LRec lds_rec_at(const char *base, uint32_t off)
{
    const uint4 *p = reinterpret_cast<const uint4 *>(base + off);
    const uint4 a = p[0], b = p[1], c = p[2];
    LRec r;
    r.c0 = (int)a.x;
    r.c1 = (int)a.y;
    r.c2 = (int)a.z;
    r.flags = a.w;
    r.e0 = (int)b.x;
    r.e1 = (int)b.y;
    r.e2 = (int)b.z;
    r.nkey = b.w;
    r.rw0 = __uint_as_float(c.x);
    r.rw1 = __uint_as_float(c.y);
    r.rw2 = __uint_as_float(c.z);
    r.invA = __uint_as_float(c.w);
    return r;
}

// flags: byte k (k = 0, 1, 2) is 1 when edge k is not owned (the pixel needs
// E_k > 0; a byte of its own lets a compare read it directly), bit 24 slow
// (int64 edge values), bit 25 packed (every edge delta fits int16)
constexpr uint32_t kSlow = 1u << 24;
constexpr uint32_t kPacked = 1u << 25;

typedef short short2_t __attribute__((ext_vector_type(2)));

// The raster's lanes test their pixels block by block: an 8-pixel tile
// (one wave) is cut into eight blocks of 4 columns x 2 rows, larger tiles
// into 4x4-pixel quarters.  A record carries the mask of the tile's blocks
// (row-major, NX per row) that its pixel box touches: 8, 16 or 64 bits.
template <int TS>
struct Blk {
    static constexpr int WL = 2, HL = TS == 8 ? 1 : 2;   // log2 of the block's width, height
    static constexpr int W = 1 << WL, H = 1 << HL, NX = TS / W, NY = TS / H;
};
template <int TS>
using QMask = typename std::conditional<TS == 32, unsigned long long,
                                        typename std::conditional<TS == 8, uint8_t, uint32_t>::type>::type;

// The bits a raster pair entry carries for block b of a wave's 8 x 8 pixels
// (bx = b % 2, by = b / 2): the block's offset in the packed (Q, P) pair of
// 1/256-pixel coordinates (Q in the low half, P in the high half) and in
// the wave's z-keys (8 bytes per pixel, row-major), both placed so that an
// OR with the lane's own offsets adds them; the record's offset sits in bits
// 12..23 and touches neither.
template <int TS>
__host__ __device__ constexpr uint32_t pair_bits(int b)
{
    using B = Blk<TS>;
    const uint32_t bx = (uint32_t)(b & 1), by = (uint32_t)(b >> 1);
    return (by * B::H * 256u) | ((bx * B::W * 256u) << 16) | ((by * B::H * 8u + bx * B::W) * 8u);
}
template <int TS>
__host__ __device__ constexpr uint32_t pair_bits_all()
{
    uint32_t m = 0;
    for (int b = 0; b < 2 * (8 / Blk<TS>::H); ++b) m |= pair_bits<TS>(b);
    return m;
}
// the z-key offsets are below 512 bytes, the (Q, P) offsets at or above
template <int TS>
constexpr uint32_t kPairZ = pair_bits_all<TS>() & 0x1FFu;
template <int TS>
constexpr uint32_t kPairQP = pair_bits_all<TS>() & ~0x1FFu;
static_assert(kPairZ<8> == 0x1A0u && kPairQP<8> == 0x04000600u, "pair bits, 8-pixel tiles");
static_assert(kPairZ<16> == 0x120u && kPairQP<16> == 0x04000400u, "pair bits, larger tiles");
static_assert(((kPairZ<8> | kPairQP<8>) & 0x00FFF000u) == 0 && ((kPairZ<32> | kPairQP<32>) & 0x00FFF000u) == 0,
              "record offset bits");

// The record of sub-triangle `key` relative to the TS-pixel tile at (ti0, tj0),
// with its edges (dx, dy), its owned flags and its pixel box in the tile; false
// if there is none.
template <int TS>
__device__ __forceinline__ bool edge_rec(const DView &v, uint32_t key, int ti0, int tj0, LRec &r, LExt &x, int box[4],
                                         int dx[3], int dy[3], uint32_t &notown, bool &packed, bool &rerr)
{
    const uint32_t t = key >> 1;
    const int sub = (int)(key & 1u);
    float P[9];
    load_pos(v, t, P);
    Vtx<0> c0, c1, c2;
    cam_xform(v, P[0], P[1], P[2], c0);
    cam_xform(v, P[3], P[4], P[5], c1);
    cam_xform(v, P[6], P[7], P[8], c2);
    SVtx<0> a, b, c;
    long long A = 0;
    const bool front = c0.w >= v.zn && c1.w >= v.zn && c2.w >= v.zn;
    if (front) {
        // all three vertices in front of the near plane (the common case):
        // clipping returns them unchanged and there is no second
        // sub-triangle, so this is the setup of sub-triangle 0 without the
        // polygon bookkeeping, which it survived
        if (sub != 0) return false;
        (void)snap3<false>(v, c0, c1, c2, a, b, c);
    } else if (!setup_sub(v, c0, c1, c2, sub, a, b, c, A, rerr)) {
        return false;
    }
    const PixBox pb = pix_box(v, a, b, c);
    box[0] = max(pb.i0 - ti0, 0);
    box[1] = min(pb.i1 - ti0, TS - 1);
    box[2] = max(pb.j0 - tj0, 0);
    box[3] = min(pb.j1 - tj0, TS - 1);
    if (box[0] > box[1] || box[2] > box[3]) return false;
    // the tile's first pixel centre, and whether every vertex lies within 64 px
    // of it (|X| < 2^29: differences fit int32)
    const int Ox = 256 * ti0 + 128, Oy = 256 * tj0 + 128;
    constexpr int kNear = 1 << 14;
    const bool small = abs(a.X - Ox) < kNear && abs(b.X - Ox) < kNear && abs(c.X - Ox) < kNear &&
                       abs(a.Y - Oy) < kNear && abs(b.Y - Oy) < kNear && abs(c.Y - Oy) < kNear;
    // twice the area, made positive by the order of b and c (a clipped piece
    // comes oriented); its float has the same rounding from either width
    float fA;
    if (small) {
        const int A32 = __mul24(b.X - a.X, c.Y - a.Y) - __mul24(b.Y - a.Y, c.X - a.X);   // |.| < 2^31
        fA = (float)A32;
    } else {
        if (front) A = area2(a, b, c);
        fA = (float)A;
    }
    if (fA < 0.0f) {
        const SVtx<0> tmp = b;
        b = c;
        c = tmp;
        fA = -fA;
    }
    // edge k runs from vertex k+1 to vertex k+2
    dx[0] = c.X - b.X;
    dx[1] = a.X - c.X;
    dx[2] = b.X - a.X;
    dy[0] = c.Y - b.Y;
    dy[1] = a.Y - c.Y;
    dy[2] = b.Y - a.Y;
    const int ax[3] = {b.X, c.X, a.X};
    const int ay[3] = {b.Y, c.Y, a.Y};
    notown = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (!owned(dx[k], dy[k])) notown |= 1u << (8 * k);
    // C_k = E_k at the tile's first pixel centre, as low and high words
    int clo[3], chi[3];
    bool fast = true;
    packed = true;
    // edge start points relative to that centre
    const int rx[3] = {ax[0] - Ox, ax[1] - Ox, ax[2] - Ox};
    const int ry[3] = {ay[0] - Oy, ay[1] - Oy, ay[2] - Oy};
    if (small) {
        // |d| < 2^15, 24-bit products,
        // |C| < 2^30, every pixel value of the tile < 2^31 in magnitude:
        // the packed form, without 64-bit arithmetic
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            clo[k] = __mul24(dy[k], rx[k]) - __mul24(dx[k], ry[k]);
            chi[k] = clo[k] >> 31;
        }
    } else {
        constexpr unsigned long long PM = 256ull * (TS - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            // C_k = dy r_x - dx r_y from 32 x 32 -> 64-bit products (|r| < 2^30)
            const long long C = (long long)dy[k] * rx[k] - (long long)dx[k] * ry[k];
            clo[k] = (int)(uint32_t)(unsigned long long)C;
            chi[k] = (int)(C >> 32);
            // the largest and smallest E_k over the tile's pixel centres: C_k
            // plus PM times the positive (negative) parts of dx_k and -dy_k
            // (each part below 2^30 in magnitude, their sum below 2^31)
            const uint32_t up = (uint32_t)max(dx[k], 0) + (uint32_t)(-min(dy[k], 0));
            const uint32_t dn = (uint32_t)(-min(dx[k], 0)) + (uint32_t)max(dy[k], 0);
            const long long emax = C + (long long)((unsigned long long)up * PM);
            const long long emin = C - (long long)((unsigned long long)dn * PM);
            // every pixel value of the tile within +-2^29, so each product
            // term (a difference of two such values) stays within +-2^30: no
            // int32 intermediate can overflow
            fast = fast && emax <= (1ll << 29) && emin >= -(1ll << 29) && dx[k] < (1 << 22) &&
                   dx[k] > -(1 << 22) && dy[k] < (1 << 22) && dy[k] > -(1 << 22);
        }
        packed = fast;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            packed = packed && dx[k] < 32768 && dx[k] > -32768 && dy[k] < 32768 && dy[k] > -32768;
    }
    r.c0 = clo[0];
    r.c1 = clo[1];
    r.c2 = clo[2];
    x.hi0 = chi[0];
    x.hi1 = chi[1];
    x.hi2 = chi[2];
    if (packed) {
        r.e0 = (int)(((uint32_t)dx[0] & 0xFFFFu) | ((uint32_t)(-dy[0]) << 16));
        r.e1 = (int)(((uint32_t)dx[1] & 0xFFFFu) | ((uint32_t)(-dy[1]) << 16));
        r.e2 = (int)(((uint32_t)dx[2] & 0xFFFFu) | ((uint32_t)(-dy[2]) << 16));
    } else {
        r.e0 = dx[0];
        r.e1 = dx[1];
        r.e2 = dx[2];
    }
    x.ny0 = -dy[0];
    x.ny1 = -dy[1];
    x.ny2 = -dy[2];
    r.invA = recip_rn(fA);
    r.rw0 = a.rw;
    r.rw1 = b.rw;
    r.rw2 = c.rw;
    r.nkey = ~key;
    r.flags = notown | (fast ? 0u : kSlow) | (packed ? kPacked : 0u);
    return true;
}

template <int TS>
__device__ __forceinline__ bool build_rec(const DView &v, uint32_t key, int ti0, int tj0, LRec &r, LExt &x,
                                          QMask<TS> &qm, bool &rerr)
{
    int box[4], dx[3], dy[3];
    uint32_t notown;
    bool packed;
    if (!edge_rec<TS>(v, key, ti0, tj0, r, x, box, dx, dy, notown, packed, rerr)) return false;
    using B = Blk<TS>;
    using Q = QMask<TS>;
    const int qx0 = box[0] >> B::WL, qx1 = box[1] >> B::WL, qy0 = box[2] >> B::HL, qy1 = box[3] >> B::HL;
    const Q row = (Q)(((Q)2 << qx1) - ((Q)1 << qx0));
    qm = 0;
#pragma unroll
    for (int qy = 0; qy < B::NY; ++qy)
        if (qy >= qy0 && qy <= qy1) qm |= row << (qy * B::NX);

    if constexpr (TS == 8) {
        // Drop the blocks that hold no pixel centre the triangle can cover:
        // an edge whose largest value over a block's centres is below its
        // threshold (1 if not owned, else 0) excludes the block.  E_k peaks
        // at the block corner that dx_k and -dy_k favour; g_k is that peak
        // for block (0, 0) less the threshold, and moves by dx_k 256 H per
        // block row and by -dy_k 256 W per block column.  A block stays
        // while every such value is >= 0, i.e. while the sign bit of their
        // OR is clear.  Every value is E_k at a pixel centre of the tile,
        // minus 0 or 1: exact in int32 for packed records (|E| < 2^31).
        if (packed) {
            constexpr int PW = 256 * (B::W - 1), QH = 256 * (B::H - 1);
            int g[3], sp[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                g[k] = (k == 0 ? r.c0 : k == 1 ? r.c1 : r.c2) + (dx[k] > 0 ? __mul24(dx[k], QH) : 0) - (dy[k] < 0 ? __mul24(dy[k], PW) : 0) -
                       (int)((notown >> (8 * k)) & 1u);
                sp[k] = dy[k] * (256 * B::W);
            }
            QMask<TS> keep = 0;
#pragma unroll
            for (int qy = 0; qy < B::NY; ++qy) {
#pragma unroll
                for (int qx = 0; qx < B::NX; ++qx) {
                    const int e = (g[0] - qx * sp[0]) | (g[1] - qx * sp[1]) | (g[2] - qx * sp[2]);
                    keep |= (QMask<TS>)((uint32_t)~e >> 31) << (qy * B::NX + qx);
                }
                if (qy + 1 < B::NY) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) g[k] += dx[k] * (256 * B::H);
                }
            }
            qm &= keep;
            if (!qm) return false;
        }
    }
    return true;
}

__device__ __forceinline__ long long join64(int hi, int lo)
{
    return (long long)(((unsigned long long)(uint32_t)hi << 32) | (unsigned long long)(uint32_t)lo);
}

// ------------------------------------------------------------ k_raster_wave
// A wave rasterises a work item of a 16-pixel tile by itself: the balanced
// form of k_raster (which see) over the tile's 32 blocks of 4 x 2 pixels, the
// tile's 256 z-keys in LDS block by block.  Against 8-pixel tiles a survivor
// meets 1.4 tiles instead of 1.9, and lists are long enough to fill the staging
// lanes; against a 256-thread block per 16-pixel tile no wave tests another's
// records and nothing waits at barriers.
//
// Records whose edges do not fit the packed form (a vertex far from the tile)
// are tested one after another by the whole wave.
//
// An overflow tile's scan is shared by several items, each gathering the survivors
// that meet the tile a wave's lanes full before it rebuilds them: few do.  Eight
// 256 x 256 views of 200k triangles with every tile over its cap take 0.19 ms;
// one item a tile over the slots with their gaps took 2.0, a 256-thread block over
// a list without gaps 0.83.
//
// Bound by VALU issue, half of it rebuilding the entries' setup: 79 M wave
// instructions for the 64 bench views (99 M before the setup dropped triangles
// that cover no pixel), 65 % busy in a launch of half of them, which ends short
// of waves.  0.146 ms alone for the 64 views; with the same lists 8-pixel tiles
// took 0.222 where this took 0.203, a 256-thread block per 16-pixel tile 0.289;
// eight 512 x 384 views of 1M triangles 0.096 ms (0.156 ms in blocks).
constexpr uint32_t kWavePairs = 512;   // (record, block) pairs listed at once: eight blocks a record

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaveWavesPerSimd))) void k_raster_wave(
    const DView *__restrict__ views, const uint2 *__restrict__ items, uint32_t cap, uint32_t seg, DQueue *__restrict__ q,
    DViewCounters *__restrict__ ctr, const uint32_t *__restrict__ vis_clusters, const uint32_t *__restrict__ skey,
    const uint2 *__restrict__ sbox, const uint32_t *__restrict__ tile_count, const uint32_t *__restrict__ tile_off, const uint32_t *__restrict__ bins,
    unsigned long long *__restrict__ zt, uint32_t *__restrict__ err)
{
    constexpr int TS = 16;
    constexpr uint32_t cls = 1;
    __shared__ LRec srec[64];
    __shared__ __align__(16) unsigned long long zk[256];
    __shared__ __align__(8) uint32_t slist[kWavePairs + 16];   // padded for the last double step's read
    const uint32_t lane = lane_id();
    const unsigned long long lt = lanemask_lt();
    for (uint32_t i = lane; i < kWavePairs + 16; i += 64) slist[i] = 0;
    // the lane's place (pxl, pyl) in its group's block; its packed (Q, P) pair
    // in block 0 and its byte offset among the block's z-keys
    const uint32_t gi = lane >> 3, pxl = lane & 3u, pyl = (lane >> 2) & 1u;
    const uint32_t QPl = (256u * pyl) | ((256u * pxl) << 16), zl = (lane & 7u) * 8u;
    // overflow tiles come first, each as `parts` items that share its scan by
    // runs: about two items a resident wave in all
    const uint32_t nover = uniform(q->total[kOverTotal]);
    if (blockIdx.x >= cap && !nover) return;
    const uint32_t parts = nover ? max(1u, min(2u * gridDim.x / nover, 64u)) : 1u;
    const uint32_t nfirst = nover * parts, total = nfirst + q->total[cls];
    const uint32_t nq = min(kQueues, gridDim.x), x = blockIdx.x % nq;
    const char *const rb = reinterpret_cast<const char *>(srec);
    bool rerr = false;
    for (;;) {
        uint32_t k = 0;
        if (lane == 0) k = atomicAdd(&q->head[cls][x].next, 1u);
        k = uniform(k);
        const uint32_t item = ((k / kQueueGroup) * nq + x) * kQueueGroup + k % kQueueGroup;
        if (item >= total) break;
        const bool over = item < nfirst;
        const uint2 it = items[over ? cap - 1u - item / parts : item - nfirst];
        const uint32_t vi = uniform(it.x), itile = uniform(it.y);
        const uint32_t tile = itile & 0x3FFFFu, sgm = itile >> 18;
        const DView &v = views[vi];
        const int ti0 = (int)(tile % v.tiles_x) * TS, tj0 = (int)(tile / v.tiles_x) * TS;
        const bool count = v.count_work != 0;
        const uint32_t cnt = uniform(tile_count[v.tile_base + tile]);
        uint4 *const z4 = reinterpret_cast<uint4 *>(zk);
        z4[lane] = make_uint4(0, 0, 0, 0);
        z4[lane + 64] = make_uint4(0, 0, 0, 0);
        uint32_t ncov = 0;
        // merge a covered fragment's key at byte offset zo of the tile's keys
        auto put = [&](uint32_t zo, float num, float invA, uint32_t nkey) {
            const float rho = num * invA;
            atomicMax(reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(zk) + zo),
                      ((unsigned long long)__float_as_uint(rho) << 32) | (unsigned long long)nkey);
        };
        // test up to 64 entries, one a lane
        auto entries = [&](bool have, uint32_t key) {
            LRec r;
            LExt rx;
            int box[4], dx[3], dy[3];
            uint32_t notown = 0, m = 0;
            bool packed = true;
            have = have && edge_rec<TS>(v, key, ti0, tj0, r, rx, box, dx, dy, notown, packed, rerr);
            if (have && packed) {
                srec[lane] = r;
                // the blocks that the box touches, less those that an edge
                // excludes: E_k peaks at the block corner that dx_k and -dy_k
                // favour, g_k is that peak in block (0, 0) less the threshold
                const int qx0 = box[0] >> 2, qx1 = box[1] >> 2, qy0 = box[2] >> 1, qy1 = box[3] >> 1;
                const uint32_t row = (2u << qx1) - (1u << qx0);
                const uint32_t hi8 = 0x11111111u >> (28 - 4 * qy1), lo8 = 0x11111111u << (4 * qy0);
                m = (hi8 & lo8) * row;
                int g[3];
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    g[j] = (j == 0 ? r.c0 : j == 1 ? r.c1 : r.c2) + (dx[j] > 0 ? dx[j] * 256 : 0) -
                           (dy[j] < 0 ? dy[j] * 768 : 0) - (int)((notown >> (8 * j)) & 1u);
                for (uint32_t t = m; t; t &= t - 1) {
                    const int b = __ffs((int)t) - 1, bx = b & 3, by = b >> 2;
                    const int e0 = g[0] + __mul24(dx[0], by << 9) - __mul24(dy[0], bx << 10);
                    const int e1 = g[1] + __mul24(dx[1], by << 9) - __mul24(dy[1], bx << 10);
                    const int e2 = g[2] + __mul24(dx[2], by << 9) - __mul24(dy[2], bx << 10);
                    if ((e0 | e1 | e2) < 0) m &= ~(1u << b);
                }
            }
            // the packed records' pairs, up to eight a record at a time: entry =
            // block, record offset (16-byte units, bits 12..19), the block's
            // (Q, P) in 1/256 pixel (bits 9..11 and 26..27)
            const uint32_t eb = (lane * (uint32_t)(sizeof(LRec) / 16)) << 12;
            while (__ballot(m != 0)) {
                const uint32_t np = min((uint32_t)__popc(m), kWavePairs / 64);
                uint32_t pos = 0, tot = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned long long bk = __ballot((np >> j) & 1u);
                    pos += (uint32_t)__popcll(bk & lt) << j;
                    tot += (uint32_t)__popcll(bk) << j;
                }
                tot = uniform(tot);
                for (uint32_t j = 0; j < np; ++j) {
                    const uint32_t b = (uint32_t)__ffs((int)m) - 1u;
                    m &= m - 1;
                    slist[pos + j] = eb | b | ((b >> 2) << 9) | ((b & 3u) << 26);
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                auto visit = [&](uint32_t en, bool act) {
                    const LRec R = lds_rec_at(rb, ((en >> 12) & 0xFFu) << 4);
                    const uint32_t qp = (en & 0x0C000E00u) | QPl;
                    const short2_t QPq = __builtin_bit_cast(short2_t, qp);
                    const uint32_t fl = R.flags;
                    const int n0 = (int)(fl & 0xFFu), n1 = (int)((fl >> 8) & 0xFFu), n2 = (int)((fl >> 16) & 0xFFu);
                    const int F0 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e0), QPq, R.c0, false);
                    const int F1 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e1), QPq, R.c1, false);
                    const int F2 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e2), QPq, R.c2, false);
                    const bool cov = act && F0 >= n0 && F1 >= n1 && F2 >= n2;
                    if (!__ballot(cov)) return;
                    if (count) {
                        // pixels outside the view do not count
                        const bool inv =
                            ti0 + (int)(qp >> 24) < (int)v.W && tj0 + (int)((qp & 0xFFFFu) >> 8) < (int)v.H;
                        ncov += (uint32_t)__popcll(__ballot(cov && inv));
                    }
                    const float w0 = (float)F0 * R.rw0, w1 = (float)F1 * R.rw1, w2 = (float)F2 * R.rw2;
                    if (cov) put(((en & 31u) << 6) | zl, (w0 + w1) + w2, R.invA, R.nkey);
                };
                uint32_t p = 0;
                // two steps per list read (one 8-byte LDS load) while more
                // than eight pairs remain
                for (; p + 8 < tot; p += 16) {
                    const uint32_t pi = p + 2 * gi;
                    const uint2 e2 = *reinterpret_cast<const uint2 *>(slist + pi);
                    visit(e2.x, pi < tot);
                    visit(e2.y, pi + 1 < tot);
                }
                if (p < tot) visit(slist[p + gi], p + gi < tot);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
            // the other records, one at a time: 64 pixels a step, block by block
            for (unsigned long long u = __ballot(have && !packed); u; u &= u - 1) {
                const int l = __ffsll((long long)u) - 1;
                auto from = [&](int y) { return __builtin_amdgcn_readlane(y, l); };
                auto fromf = [&](float y) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), l)); };
                const int x0 = from(dx[0]), x1 = from(dx[1]), x2 = from(dx[2]);
                const int y0 = from(dy[0]), y1 = from(dy[1]), y2 = from(dy[2]);
                const uint32_t fl = (uint32_t)from((int)r.flags), nkey = (uint32_t)from((int)r.nkey);
                const float w0 = fromf(r.rw0), w1 = fromf(r.rw1), w2 = fromf(r.rw2), ia = fromf(r.invA);
                const int s0 = from(box[2]) >> 2, s1 = from(box[3]) >> 2;   // of four rows: eight blocks
                const int px = (int)((gi & 3u) * 4u + pxl), py = 4 * s0 + (int)((gi >> 2) * 2u + pyl);
                // E: this lane's edge values in the first step, D: on to the next
                auto steps = [&](auto E0, auto E1, auto E2, auto D0, auto D1, auto D2) {
#pragma unroll 1
                    for (int s = s0, y = py; s <= s1; ++s, y += 4) {
                        const bool cov = E0 >= (int)(fl & 0xFFu) && E1 >= (int)((fl >> 8) & 0xFFu) &&
                                         E2 >= (int)((fl >> 16) & 0xFFu);
                        if (count) ncov += (uint32_t)__popcll(__ballot(cov && ti0 + px < (int)v.W && tj0 + y < (int)v.H));
                        if (cov)
                            put((uint32_t)s * 512u + lane * 8u, ((float)E0 * w0 + (float)E1 * w1) + (float)E2 * w2, ia, nkey);
                        E0 += D0;
                        E1 += D1;
                        E2 += D2;
                    }
                };
                const int c0 = from(r.c0), c1 = from(r.c1), c2 = from(r.c2), P = 256 * px, Q = 256 * py;
                if (!(fl & kSlow)) {
                    // every edge value in the tile lies within +-2^29, so a step is
                    // less than 2^29 and the one behind the last fits as well
                    auto at = [&](int c, int dX, int dY) {
                        return (int)((uint32_t)c + (uint32_t)__mul24(dX, Q) - (uint32_t)__mul24(dY, P));
                    };
                    steps(at(c0, x0, y0), at(c1, x1, y1), at(c2, x2, y2), x0 * 1024, x1 * 1024, x2 * 1024);
                } else {
                    auto at = [&](int hi, int c, int dX, int dY) {
                        return join64(hi, c) + (long long)dX * Q - (long long)dY * P;
                    };
                    steps(at(from(rx.hi0), c0, x0, y0), at(from(rx.hi1), c1, x1, y1), at(from(rx.hi2), c2, x2, y2),
                          (long long)x0 * 1024, (long long)x1 * 1024, (long long)x2 * 1024);
                }
            }
        };
        if (!over) {
            const uint32_t begin = sgm * seg, end = min(begin + seg, cnt);
            const uint32_t *const list = bins + v.bin_base + uniform(tile_off[v.tile_base + tile]);
            for (uint32_t base = begin; base < end; base += 64) {
                const uint32_t e = base + lane;
                const bool have = e < end;
                entries(have, have ? list[e] : 0u);
            }
        } else {
            // this part's runs (their counts loaded 64 at a time); the survivors
            // that meet the tile are gathered a wave's lanes full before they are
            // tested
            const uint32_t nruns = (uniform(visible_clusters(ctr[vi])) + kRun - 1) / kRun;
            uint32_t held = 0, key = 0;
            for (uint32_t run0 = item % parts; run0 < nruns; run0 += 64 * parts) {
                const uint32_t mine = run0 + lane * parts;
                const uint32_t counts = mine < nruns ? run_count(v, vis_clusters, mine) : 0u;
                for (uint32_t j = 0; j < 64 && run0 + j * parts < nruns; ++j) {
                    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)counts, (int)j);
                    const uint32_t slot0 = v.surv_base + (run0 + j * parts) * kSlots;
                    // two steps' boxes in flight together
                    for (uint32_t e0 = 0; e0 < n; e0 += 128) {
                        const uint32_t ea = e0 + lane, eb = ea + 64;
                        const uint2 ba = sbox[slot0 + min(ea, n - 1)];
                        const uint2 bb = sbox[slot0 + min(eb, n - 1)];
                        bool meets = ea < n && box_meets<TS>(ba, ti0, tj0);
                        const bool next = eb < n && box_meets<TS>(bb, ti0, tj0);
#pragma unroll 1
                        for (uint32_t e = ea;;) {
                            const unsigned long long mm = __ballot(meets);
                            const uint32_t got = (uint32_t)__popcll(mm);
                            if (got) {
                                // hits go to the lanes behind those held, the
                                // others' (junk) behind them: each lane gets one
                                const uint32_t rank = (uint32_t)__popcll(mm & lt), to = held + (meets ? rank : got + lane - rank);
                                uint32_t found = 0;
                                if (meets) found = skey[slot0 + e];
                                found = (uint32_t)__builtin_amdgcn_ds_permute((int)((to & 63u) << 2), (int)found);
                                if (lane >= held) key = found;
                                held += got;
                                if (held >= 64) {
                                    entries(true, key);
                                    held -= 64;
                                    key = found;
                                }
                            }
                            if (e == eb) break;
                            e = eb;
                            meets = next;
                        }
                    }
                }
            }
            if (held) entries(lane < held, key);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        unsigned long long *const z = zt + wave_tile(v, tile);
        if (!over && cnt <= seg) {
            uint4 *const zo = reinterpret_cast<uint4 *>(z);
            zo[lane] = z4[lane];
            zo[lane + 64] = z4[lane + 64];
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const unsigned long long b = zk[64 * j + lane];
                if (b) (void)__hip_atomic_fetch_max(z + 64 * j + lane, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (count && lane == 0 && ncov) atomicAdd(&ctr[vi].covered, (unsigned long long)ncov);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    if (rerr) atomicOr(err, kErrRange);
}

// LO: lane-owned pixels with an atomic-free z-test in registers; else
// balanced steps over (record, block) pairs with the z-keys in LDS.
template <int TS, bool LO>
// 6 waves per SIMD: the register budget (80 VGPRs) that lets enough
// waves hide the LDS and staging latency (the LDS of an 8-pixel tile,
// 7.3 KB, allows 22 blocks per CU); a 32-pixel tile's LDS allows 4.
__global__ __launch_bounds__(TS *TS) __attribute__((amdgpu_waves_per_eu(TS == 32 ? 4 : 6))) void k_raster(const DView *__restrict__ views,
                                                   const uint2 *__restrict__ items,
                                                   DQueue *__restrict__ q,
                                                   DViewCounters *__restrict__ ctr,
                                                   const uint32_t *__restrict__ vis_clusters,
                                                   const uint32_t *__restrict__ skey,
                                                   const uint2 *__restrict__ sbox,
                                                   const uint32_t *__restrict__ tile_count,
                                                   const uint32_t *__restrict__ tile_off,
                                                   const uint32_t *__restrict__ bins,
                                                   uint2 *__restrict__ partial,
                                                   uint32_t *__restrict__ err)
{
    constexpr int NT = TS * TS;
    constexpr int NS = TS / 8;
    constexpr uint32_t cls = TS == 8 ? 0u : TS == 16 ? 1u : 2u;
    constexpr uint32_t S = kSegPerTile * NT;
    using B = Blk<TS>;
    // a wave's 8x8 pixels hold NL blocks: 2 columns of 8 / H rows
    constexpr int NL = 2 * (8 / B::H);
    using QM = QMask<TS>;
    __shared__ LRec srec[NT];
    __shared__ LExt sext[NT];
    __shared__ QM sqm[NT];
    // lane groups of one block's size; a step gives each group one (record,
    // block) pair
    constexpr uint32_t GS = B::W * B::H, NG = 64 / GS;
    static_assert(NG == NL, "one lane group per block of a wave");
    // per wave, lane-owned pixels: per block, byte offsets in srec of the
    // chunk's records that touch the block ([NL][64]); balanced steps: the
    // chunk's (record, block) pairs, record by record, padded for the last
    // double step's read (zeroed once, so a stale entry is still a record
    // or a pair)
    constexpr uint32_t kList = LO ? NL * 64 : NL * 64 + 2 * NG;
    __shared__ __align__(8) uint32_t slist[NT / 64][kList];
    // per wave, balanced steps: the best z-key of each of its 64 pixels
    // (row-major 8 x 8)
    __shared__ unsigned long long szb[NT / 64][LO ? 1 : 64];
    __shared__ uint32_t s_item;
    // an overflow tile's scan: has a wave staged any in this step (two, in turn)
    constexpr uint32_t NW = NT / 64;
    __shared__ uint32_t s_more[2];

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const unsigned long long lt = lanemask_lt();
    for (uint32_t i = lane; i < kList; i += 64) slist[wave][i] = 0;
    const int sx = (int)(wave % NS), sy = (int)(wave / NS);
    // lane-owned pixels: lane (li, lj) of the wave's 8 x 8 pixels, at (P, Q)
    // in 1/256 pixel from the tile's first pixel centre; (Q, P) as a 16-bit
    // pair for the packed edge records (dot2 gives dx Q - dy P)
    const int li = (int)(lane & 7u), lj = (int)(lane >> 3);
    const int P = 256 * (sx * 8 + li), Q = 256 * (sy * 8 + lj);
    const short2_t QP = __builtin_bit_cast(short2_t, (uint32_t)Q | ((uint32_t)P << 16));
    // balanced steps: a lane's place in its group's block: (pxl, pyl); the
    // group's block b (bx = b % 2, by = b / 2 in the wave's 8 x 8 pixels)
    // comes with the pair.  QPl: (Q, P) of that place in block 0 as a
    // 16-bit pair; zl: its byte offset in the wave's z-keys.
    const uint32_t pxl = lane % B::W, pyl = (lane % GS) / B::W;
    const uint32_t QPl = (256u * (uint32_t)(sy * 8 + (int)pyl)) | ((256u * (uint32_t)(sx * 8 + (int)pxl)) << 16);
    const uint32_t zl = (pyl * 8 + pxl) * 8;
    unsigned long long *const zw = &szb[wave][0];
    const uint32_t total = q->total[cls];
    bool rerr = false;

    // nq queues (at most one per block); this block drains queue x, whose
    // k-th grab is item ((k / G) nq + x) G + k % G with G = kQueueGroup:
    // every item belongs to exactly one (queue, grab), in increasing order
    const uint32_t nq = min(kQueues, gridDim.x), x = blockIdx.x % nq;
    for (;;) {
        if (tid == 0) {
            if (NW > 1) s_more[0] = s_more[1] = 0;
            const uint32_t k = atomicAdd(&q->head[cls][x].next, 1u);
            s_item = ((k / kQueueGroup) * nq + x) * kQueueGroup + k % kQueueGroup;
        }
        __syncthreads();
        const uint32_t item = uniform(s_item);
        __syncthreads();
        if (item >= total) break;
        const uint2 it = items[item];
        const uint32_t vi = it.x;
        const uint32_t tile = it.y & 0x3FFFFu, sgm = it.y >> 18;
        const DView &v = views[vi];
        const int tx = (int)(tile % v.tiles_x), ty = (int)(tile / v.tiles_x);
        const int ti0 = tx * TS, tj0 = ty * TS;
        const bool count = v.count_work != 0;
        // lane-owned pixels: the lanes whose pixel is in view
        unsigned long long inmask = 0ull;
        if constexpr (LO) inmask = __ballot(ti0 + sx * 8 + li < (int)v.W && tj0 + sy * 8 + lj < (int)v.H);

        const uint32_t tglob = v.tile_base + tile;
        const uint32_t cnt = tile_count[tglob];
        const uint32_t off = tile_off[tglob];
        const bool over = off == kOverflow;
        const uint32_t *list = bins + v.bin_base + (over ? 0u : off);

        // z-key of the best fragment so far: 1/w bits above the complemented
        // triangle key.  A covered fragment has 1/w > 0 (positive weights,
        // positive twice-area), so one unsigned max orders by largest 1/w,
        // then smaller key; 0 means no fragment.  Lane-owned pixels keep it
        // in the owning lane's registers (atomic-free); balanced steps, where
        // any lane group may test any pixel block, keep it in LDS and merge
        // by atomic max.
        unsigned long long best = 0ull;
        if constexpr (!LO) {
            zw[lane] = 0ull;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
        uint32_t ncov = 0;

        // the list's segment, a block's threads at a time; of an overflow tile the
        // survivors of all visible runs, each wave through runs of its own, 64 at
        // a time, for the whole block
        const uint32_t nruns = over ? (uniform(visible_clusters(ctr[vi])) + kRun - 1) / kRun : 0u;
        uint32_t base = over ? 0u : sgm * S, stop = over ? 0u : min(base + S, cnt), run = uniform(wave);
        for (uint32_t step = 0;; ++step) {
            if (over) {
                while (base >= stop && run < nruns) {
                    base = run * kSlots;
                    stop = base + uniform(run_count(v, vis_clusters, run));
                    run += NW;
                }
                if (NW == 1 && base >= stop) break;
                if (NW > 1 && lane == 0 && base < stop) s_more[step & 1u] = 1;
            } else if (base >= stop) {
                break;
            }
            // stage: each thread rebuilds one list entry's edge setup for this tile
            {
                const uint32_t e = base + (over ? lane : tid);
                QM qm = 0;
                LRec r;
                LExt rx;
                bool go = e < stop;
                uint32_t key = 0;
                if (go) {
                    if (over) {
                        go = box_meets<TS>(sbox[v.surv_base + e], ti0, tj0);
                        if (go) key = skey[v.surv_base + e];
                    } else {
                        key = list[e];
                    }
                }
                if (NW == 1 && over && !__ballot(go)) {
                    base += 64;
                    continue;
                }
                if (go && !build_rec<TS>(v, key, ti0, tj0, r, rx, qm, rerr)) qm = 0;
                sqm[tid] = qm;
                if (qm) {
                    srec[tid] = r;
                    if (!(r.flags & kPacked)) sext[tid] = rx;
                }
            }
            __syncthreads();
            const uint32_t m = over ? (uint32_t)NT : min((uint32_t)NT, stop - base);
            base += over ? 64u : (uint32_t)NT;
            if (NW > 1 && over) {
                if (!s_more[step & 1u]) break;   // no wave had any
                if (tid == 0) s_more[~step & 1u] = 0;
            }
            if constexpr (LO) {
                // z-test of this lane's pixel against fragment weights w_k where
                // covered (cov) and the wave's coverage ballot cm
                auto zkeep = [&](const LRec &R, bool cov, float w0, float w1, float w2) {
                    const float num = (w0 + w1) + w2;
                    const float rho = num * R.invA;
                    const unsigned long long cand =
                        ((unsigned long long)__float_as_uint(rho) << 32) | (unsigned long long)R.nkey;
                    if (count) ncov += (uint32_t)__popcll(__ballot(cov) & inmask);
                    best = (cov && cand > best) ? cand : best;
                };
                // one step: every active lane tests its pixel against record R
                // (index k) of its block under the top-left rule (an edge not
                // owned needs E > 0)
                auto visit = [&](const LRec &R, uint32_t k, bool act, auto allpk) {
                    const uint32_t fl = R.flags;
                    const int n0 = (int)(fl & 0xFFu), n1 = (int)((fl >> 8) & 0xFFu), n2 = (int)((fl >> 16) & 0xFFu);
                    if (decltype(allpk)::value || !__ballot(act && !(fl & kPacked))) {
                        // every active lane's record is packed
                        const int F0 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e0), QP, R.c0, false);
                        const int F1 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e1), QP, R.c1, false);
                        const int F2 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e2), QP, R.c2, false);
                        const bool cov = act && F0 >= n0 && F1 >= n1 && F2 >= n2;
                        if (!__ballot(cov)) return;
                        zkeep(R, cov, (float)F0 * R.rw0, (float)F1 * R.rw1, (float)F2 * R.rw2);
                        return;
                    }
                    bool cov = false;
                    float w0 = 0.0f, w1 = 0.0f, w2 = 0.0f;
                    if (act && (fl & kPacked)) {
                        const int F0 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e0), QP, R.c0, false);
                        const int F1 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e1), QP, R.c1, false);
                        const int F2 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e2), QP, R.c2, false);
                        cov = F0 >= n0 && F1 >= n1 && F2 >= n2;
                        w0 = (float)F0 * R.rw0;
                        w1 = (float)F1 * R.rw1;
                        w2 = (float)F2 * R.rw2;
                    } else if (act && !(fl & kSlow)) {
                        const LExt &X = sext[k];
                        const int F0 = (int)((uint32_t)R.c0 + (uint32_t)__mul24(R.e0, Q) + (uint32_t)__mul24(X.ny0, P));
                        const int F1 = (int)((uint32_t)R.c1 + (uint32_t)__mul24(R.e1, Q) + (uint32_t)__mul24(X.ny1, P));
                        const int F2 = (int)((uint32_t)R.c2 + (uint32_t)__mul24(R.e2, Q) + (uint32_t)__mul24(X.ny2, P));
                        cov = F0 >= n0 && F1 >= n1 && F2 >= n2;
                        w0 = (float)F0 * R.rw0;
                        w1 = (float)F1 * R.rw1;
                        w2 = (float)F2 * R.rw2;
                    } else if (act) {
                        const LExt &X = sext[k];
                        const long long E0 = join64(X.hi0, R.c0) + (long long)R.e0 * Q + (long long)X.ny0 * P;
                        const long long E1 = join64(X.hi1, R.c1) + (long long)R.e1 * Q + (long long)X.ny1 * P;
                        const long long E2 = join64(X.hi2, R.c2) + (long long)R.e2 * Q + (long long)X.ny2 * P;
                        cov = E0 >= (long long)n0 && E1 >= (long long)n1 && E2 >= (long long)n2;
                        w0 = (float)E0 * R.rw0;
                        w1 = (float)E1 * R.rw1;
                        w2 = (float)E2 * R.rw2;
                    }
                    if (!__ballot(cov)) return;
                    zkeep(R, cov, w0, w1, w2);
                };
                // the wave's NL blocks (8 or 16 lanes each) walk their own lists
                // of records whose box touches them: one step tests up to NL
                // records.  Block b of this wave is bit qb + (b / 2) NX + b % 2
                // of a record's block mask.  Per chunk of 64 records, each
                // block's relevant records are compacted into its LDS list; step
                // i then tests entry i of every block's list.
                const uint32_t qb = (uint32_t)(sy * (8 / B::H) * B::NX + 2 * sx);
                const uint32_t lq = ((lane >> (3 + B::HL)) << 1) | ((lane >> 2) & 1u);
                uint32_t *const wl = &slist[wave][0];
                for (uint32_t g = 0; g < m; g += 64) {
                    const bool in = g + lane < m;
                    const QM qm = in ? sqm[g + lane] : (QM)0;
                    bool rl[NL];
                    unsigned long long mk[NL], any = 0;
#pragma unroll
                    for (int b = 0; b < NL; ++b) {
                        rl[b] = (qm >> (qb + (uint32_t)((b >> 1) * B::NX + (b & 1)))) & 1u;
                        mk[b] = __ballot(rl[b]);
                        any |= mk[b];
                    }
                    if (!any) continue;
                    const uint32_t off = (g + lane) * (uint32_t)sizeof(LRec);
                    bool rel = false;
                    uint32_t nsteps = 0, myc = 0;
#pragma unroll
                    for (int b = 0; b < NL; ++b) {
                        if (rl[b]) wl[b * 64 + __popcll(mk[b] & lt)] = off;
                        rel = rel || rl[b];
                        const uint32_t c = (uint32_t)__popcll(mk[b]);
                        nsteps = max(nsteps, c);
                        myc = lq == (uint32_t)b ? c : myc;
                    }
                    nsteps = uniform(nsteps);
                    // does every record this wave will test have the packed form?
                    const bool allpk = !__ballot(rel && !(srec[g + lane].flags & kPacked));
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    const uint32_t *const myl = wl + lq * 64;
                    const char *const rb = reinterpret_cast<const char *>(srec);
                    if (allpk) {
                        // two steps per list read (one 8-byte LDS load)
                        uint32_t i = 0;
                        for (; i + 1 < nsteps; i += 2) {
                            const uint2 o2 = *reinterpret_cast<const uint2 *>(myl + i);
                            visit(lds_rec_at(rb, o2.x), o2.x / (uint32_t)sizeof(LRec), i < myc, std::true_type());
                            visit(lds_rec_at(rb, o2.y), o2.y / (uint32_t)sizeof(LRec), i + 1 < myc, std::true_type());
                        }
                        if (i < nsteps) {
                            const uint32_t o = myl[i];
                            visit(lds_rec_at(rb, o), o / (uint32_t)sizeof(LRec), i < myc, std::true_type());
                        }
                    } else {
                        for (uint32_t i = 0; i < nsteps; ++i) {
                            const uint32_t o = myl[i];
                            visit(lds_rec_at(rb, o), o / (uint32_t)sizeof(LRec), i < myc, std::false_type());
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                }
            } else {
                // z-test of the pixel of pair entry `en` against fragment weights
                // w_k where covered (cov)
                auto zkeep = [&](const LRec &R, uint32_t en, uint32_t qp, bool cov, float w0, float w1, float w2) {
                    const float num = (w0 + w1) + w2;
                    const float rho = num * R.invA;
                    const unsigned long long cand =
                        ((unsigned long long)__float_as_uint(rho) << 32) | (unsigned long long)R.nkey;
                    if (count) {
                        // pixels outside the view do not count
                        const bool inv = ti0 + (int)(qp >> 24) < (int)v.W && tj0 + (int)((qp & 0xFFFFu) >> 8) < (int)v.H;
                        ncov += (uint32_t)__popcll(__ballot(cov && inv));
                    }
                    if (cov) {
                        unsigned long long *z = reinterpret_cast<unsigned long long *>(
                            reinterpret_cast<char *>(zw) + ((en & kPairZ<TS>) | zl));
                        atomicMax(z, cand);
                    }
                };
                // one step: every active lane tests the pixel its pair entry
                // names against the pair's record under the top-left rule (an
                // edge not owned needs E > 0)
                const char *const rb = reinterpret_cast<const char *>(srec);
                auto visit = [&](uint32_t en, bool act, auto allpk) {
                    const uint32_t off = ((en >> 12) & 0xFFFu) << 4;
                    const LRec R = lds_rec_at(rb, off);
                    const uint32_t qp = (en & kPairQP<TS>) | QPl;
                    const short2_t QPq = __builtin_bit_cast(short2_t, qp);
                    const uint32_t fl = R.flags;
                    const int n0 = (int)(fl & 0xFFu), n1 = (int)((fl >> 8) & 0xFFu), n2 = (int)((fl >> 16) & 0xFFu);
                    if (decltype(allpk)::value || !__ballot(act && !(fl & kPacked))) {
                        // every active lane's record is packed
                        const int F0 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e0), QPq, R.c0, false);
                        const int F1 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e1), QPq, R.c1, false);
                        const int F2 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e2), QPq, R.c2, false);
                        const bool cov = act && F0 >= n0 && F1 >= n1 && F2 >= n2;
                        if (!__ballot(cov)) return;
                        zkeep(R, en, qp, cov, (float)F0 * R.rw0, (float)F1 * R.rw1, (float)F2 * R.rw2);
                        return;
                    }
                    const int Pq = (int)(qp >> 16), Qq = (int)(qp & 0xFFFFu);
                    bool cov = false;
                    float w0 = 0.0f, w1 = 0.0f, w2 = 0.0f;
                    if (act && (fl & kPacked)) {
                        const int F0 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e0), QPq, R.c0, false);
                        const int F1 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e1), QPq, R.c1, false);
                        const int F2 = __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, R.e2), QPq, R.c2, false);
                        cov = F0 >= n0 && F1 >= n1 && F2 >= n2;
                        w0 = (float)F0 * R.rw0;
                        w1 = (float)F1 * R.rw1;
                        w2 = (float)F2 * R.rw2;
                    } else if (act && !(fl & kSlow)) {
                        const LExt &X = sext[off / (uint32_t)sizeof(LRec)];
                        const int F0 = (int)((uint32_t)R.c0 + (uint32_t)__mul24(R.e0, Qq) + (uint32_t)__mul24(X.ny0, Pq));
                        const int F1 = (int)((uint32_t)R.c1 + (uint32_t)__mul24(R.e1, Qq) + (uint32_t)__mul24(X.ny1, Pq));
                        const int F2 = (int)((uint32_t)R.c2 + (uint32_t)__mul24(R.e2, Qq) + (uint32_t)__mul24(X.ny2, Pq));
                        cov = F0 >= n0 && F1 >= n1 && F2 >= n2;
                        w0 = (float)F0 * R.rw0;
                        w1 = (float)F1 * R.rw1;
                        w2 = (float)F2 * R.rw2;
                    } else if (act) {
                        const LExt &X = sext[off / (uint32_t)sizeof(LRec)];
                        const long long E0 = join64(X.hi0, R.c0) + (long long)R.e0 * Qq + (long long)X.ny0 * Pq;
                        const long long E1 = join64(X.hi1, R.c1) + (long long)R.e1 * Qq + (long long)X.ny1 * Pq;
                        const long long E2 = join64(X.hi2, R.c2) + (long long)R.e2 * Qq + (long long)X.ny2 * Pq;
                        cov = E0 >= (long long)n0 && E1 >= (long long)n1 && E2 >= (long long)n2;
                        w0 = (float)E0 * R.rw0;
                        w1 = (float)E1 * R.rw1;
                        w2 = (float)E2 * R.rw2;
                    }
                    if (!__ballot(cov)) return;
                    zkeep(R, en, qp, cov, w0, w1, w2);
                };
                // Per 64 records, the wave lists the (record, block) pairs of the
                // records whose block mask has its blocks (block b of this wave
                // is bit qb + (b / 2) NX + b % 2 of the mask), record by record;
                // step i gives lane group g pair i NG + g, so every step tests
                // NG pairs whatever blocks they fall in.  A pair entry carries
                // the record's offset in srec (in 16-byte units, bits 12..23)
                // and its block's pixel offsets: for the packed (Q, P) pair and
                // for the z-keys (kPairQP, kPairZ bits).
                const uint32_t qb = (uint32_t)(sy * (8 / B::H) * B::NX + 2 * sx);
                uint32_t *const wl = &slist[wave][0];
                const uint32_t gi = lane / GS;
                for (uint32_t g = 0; g < m; g += 64) {
                    const bool in = g + lane < m;
                    const QM qm = in ? sqm[g + lane] : (QM)0;
                    uint32_t mb = 0;
#pragma unroll
                    for (int b = 0; b < NL; ++b)
                        mb |= (uint32_t)((qm >> (qb + (uint32_t)((b >> 1) * B::NX + (b & 1)))) & 1u) << b;
                    // exclusive prefix of the pair counts over the wave, by bit
                    // planes (a count is at most NL <= 8)
                    const uint32_t np = (uint32_t)__popc(mb);
                    uint32_t pos = 0, tot = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned long long bk = __ballot((np >> k) & 1u);
                        pos += (uint32_t)__popcll(bk & lt) << k;
                        tot += (uint32_t)__popcll(bk) << k;
                    }
                    tot = uniform(tot);
                    if (!tot) continue;
                    const uint32_t eb = ((g + lane) * (uint32_t)(sizeof(LRec) / 16)) << 12;
#pragma unroll
                    for (int b = 0; b < NL; ++b) {
                        if ((mb >> b) & 1u) wl[pos++] = eb | pair_bits<TS>(b);
                    }
                    // does every record this wave will test have the packed form?
                    const bool allpk = !__ballot(mb && !(srec[g + lane].flags & kPacked));
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    uint32_t p = 0;
                    if (allpk) {
                        // two steps per list read (one 8-byte LDS load) while
                        // more than NG pairs remain
                        for (; p + NG < tot; p += 2 * NG) {
                            const uint32_t pi = p + 2 * gi;
                            const uint2 e2 = *reinterpret_cast<const uint2 *>(wl + pi);
                            visit(e2.x, pi < tot, std::true_type());
                            visit(e2.y, pi + 1 < tot, std::true_type());
                        }
                        if (p < tot) visit(wl[p + gi], p + gi < tot, std::true_type());
                    } else {
                        for (; p < tot; p += NG) visit(wl[p + gi], p + gi < tot, std::false_type());
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                }
            }
            __syncthreads();
        }
        if constexpr (!LO) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            best = zw[lane];
        }
        partial[(size_t)item * NT + tid] = make_uint2((uint32_t)(best >> 32), ~(uint32_t)best);
        if (v.count_work && lane == 0 && ncov) atomicAdd(&ctr[vi].covered, (unsigned long long)ncov);
    }
    if (rerr) atomicOr(err, kErrRange);
}

// Resolve bands: 32 x 2 pixels of one view per wave (one lane per pixel,
// four 8-pixel tiles side by side).  Each lane merges its pixel's segment
// winners (largest 1/w, smaller key on a tie: the same order-free rule) and
// shades it.
template <int TS>
__global__ __launch_bounds__(kBandThreads) void k_resolve(const DView *__restrict__ views,
                                                          const uint32_t *__restrict__ lview,
                                                          const uint32_t *__restrict__ bpre, uint32_t nl,
                                                          const uint32_t *__restrict__ tile_count,
                                                          const uint32_t *__restrict__ tile_off,
                                                          const uint32_t *__restrict__ tile_item,
                                                          const uint2 *__restrict__ partial,
                                                          uint32_t *__restrict__ err)
{
    constexpr int NT = TS * TS;
    constexpr int NS = TS / 8;
    __shared__ __align__(16) uint8_t s_rgb[kBandRgb];
    uint32_t lo = 0, hi = nl - 1;
    const uint32_t blk = blockIdx.x;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (bpre[mid] <= blk) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t vi = uniform(lview[uniform(lo)]);
    const DView &v = views[vi];
    const uint32_t W = v.W, H = v.H;
    const uint32_t nbx = (W + kBandW - 1) / kBandW;
    const uint32_t band = blk - bpre[lo];
    const uint32_t x0 = (band % nbx) * kBandW, y0 = (band / nbx) * kBandH;
    const uint32_t lane = lane_id();
    const uint32_t cx = lane % kBandW, cy = lane / kBandW;   // position in the band
    const int pi = (int)(x0 + cx), pj = (int)(y0 + cy);
    const bool in = pi < (int)W && pj < (int)H;
    float best_rho = 0.0f;
    uint32_t best_key = kNone;
    if (in) {
        const uint32_t tile = (uint32_t)(pj / TS) * v.tiles_x + (uint32_t)(pi / TS);
        const uint32_t sub = (uint32_t)(((pj % TS) / 8) * NS + (pi % TS) / 8);
        const uint32_t tglob = v.tile_base + tile;
        const uint32_t ns = tile_segments(tile_count[tglob], tile_off[tglob], v.ts_log2, 0);
        const uint32_t first = tile_item[tglob];
        const uint32_t slot = sub * 64u + (uint32_t)((pj % 8) * 8 + (pi % 8));
        for (uint32_t s = 0; s < ns; ++s) {
            const uint2 pr = partial[(size_t)(first + s) * NT + slot];
            const float rho = __uint_as_float(pr.x);
            if (pr.y != kNone && (rho > best_rho || (rho == best_rho && pr.y < best_key))) {
                best_rho = rho;
                best_key = pr.y;
            }
        }
    }
    shade_band<kBandW, kBandH>(v, x0, y0, pi, pj, in, best_rho, best_key, s_rgb, err);
}

// As k_resolve, from the tiles' z-keys that k_raster_wave left (a tile without
// entries has none).  A wave shades STACK bands, one below the other: STACK is
// 1, 2 or 4, so they lie in one row of tiles.  256 mixed 128 / 256 / 512 px
// views, 29 M pixels: 1.25 ms a step with one band a wave and the winner read
// through its indices, 1.08 with four and its attributes by triangle.  (A 64-byte
// record of both, half a cache line, took the same and twice a scene's memory.)
// Bound by the latency of the winner's read and by VALU issue (280 instructions a
// band, 70 % busy).
template <int STACK>
__global__ __launch_bounds__(kBandThreads) void k_resolve_wave(const DView *__restrict__ views,
                                                               const uint32_t *__restrict__ lview,
                                                               const uint32_t *__restrict__ bpre, uint32_t nl,
                                                               const uint32_t *__restrict__ tile_count,
                                                               const unsigned long long *__restrict__ zt,
                                                               uint32_t *__restrict__ err)
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
    const uint32_t x0 = (band % nbx) * kBandW, y0 = (band / nbx) * (kBandH * STACK);
    const uint32_t lane = lane_id();
    const uint32_t pi = x0 + lane % kBandW, dj = lane / kBandW;
    // the stack lies in one row of tiles: all its keys are in flight at once
    const uint32_t tile = (y0 >> 4) * v.tiles_x + (pi >> 4);
    unsigned long long z[STACK] = {};
    if (pi < W && tile_count[v.tile_base + tile]) {
        const unsigned long long *zp =
            zt + wave_tile(v, tile) + ((y0 & 15u) >> 1) * 32u + ((pi & 15u) >> 2) * 8u + dj * 4u + (pi & 3u);
#pragma unroll
        for (int k = 0; k < STACK; ++k) z[k] = zp[32 * k];
    }
#pragma unroll 1
    for (int k = 0; k < STACK; ++k) {
        const uint32_t y = y0 + kBandH * (uint32_t)k, pj = y + dj;
        if (y >= H) break;
        const unsigned long long zz = z[0];
#pragma unroll
        for (int n = 1; n < STACK; ++n) z[n - 1] = z[n];
        shade_band<kBandW, kBandH>(v, x0, y, (int)pi, (int)pj, pi < W && pj < H, __uint_as_float((uint32_t)(zz >> 32)),
                                   ~(uint32_t)zz, s_rgb, err);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
}

// ------------------------------------------------------------ host side
static inline uint32_t cdiv(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

static inline void mark(const LaunchPlan &L, int ev, hipStream_t s)
{
    if (L.prof && ((L.prof_mask >> (ev >> 1)) & 1u)) (void)hipEventRecord(L.prof[ev], s);
}

template <int TS>
static void launch_raster(const LaunchPlan &L, const RasterLaunch &R, hipStream_t s)
{
    if (R.wave) {
        hipLaunchKernelGGL(k_raster_wave, dim3(R.grid), dim3(64), 0, s, L.views, R.items, R.item_cap, L.wave_seg, L.queue, L.ctr,
                           L.pairs, L.skey, L.sbox, L.tile_count, L.tile_off, L.bins, L.zbuf, L.err);
        return;
    }
    if (R.lane_owned)
        hipLaunchKernelGGL((k_raster<TS, true>), dim3(R.grid), dim3(TS * TS), 0, s, L.views, R.items, L.queue,
                           L.ctr, L.pairs, L.skey, L.sbox, L.tile_count, L.tile_off, L.bins, R.partial, L.err);
    else if constexpr (TS != 16)
        hipLaunchKernelGGL((k_raster<TS, false>), dim3(R.grid), dim3(TS * TS), 0, s, L.views, R.items, L.queue,
                           L.ctr, L.pairs, L.skey, L.sbox, L.tile_count, L.tile_off, L.bins, R.partial, L.err);
}

template <int TS>
static void launch_resolve(const LaunchPlan &L, const RasterLaunch &R, hipStream_t s)
{
    if (R.wave) {
        auto *const k = R.stack == 4 ? k_resolve_wave<4> : R.stack == 2 ? k_resolve_wave<2> : k_resolve_wave<1>;
        hipLaunchKernelGGL(k, dim3(R.bands), dim3(kBandThreads), 0, s, L.views, R.lview, R.bpre, R.nl, L.tile_count,
                           L.zbuf, L.err);
        return;
    }
    hipLaunchKernelGGL(k_resolve<TS>, dim3(R.bands), dim3(kBandThreads), 0, s, L.views, R.lview, R.bpre,
                       R.nl, L.tile_count, L.tile_off, L.tile_item, R.partial, L.err);
}

hipError_t launch_scene(const MeshSource &m, uint32_t T, float *tpos, uint32_t *attr, float4 *cbox, float3 size, float grow,
                        SpreadSums *spread, hipStream_t s)
{
    hipLaunchKernelGGL(k_scene, dim3(cdiv(T, 256)), dim3(256), 0, s, m, T, tpos, attr, cbox, size, grow, spread);
    return hipGetLastError();
}

int raster_blocks_per_cu(int ts, bool lane_owned)
{
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (ts * 2 + (lane_owned ? 1 : 0)) {
    case 16: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster<8, false>, 64, 0); break;
    case 17: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster<8, true>, 64, 0); break;
    case 32: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster_wave, 64, 0); break;
    case 33: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster<16, true>, 256, 0); break;
    case 64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster<32, false>, 1024, 0); break;
    case 65: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_raster<32, true>, 1024, 0); break;
    default: break;
    }
    if (e != hipSuccess) (void)hipGetLastError();
    return (e == hipSuccess && n > 0) ? n : 1;
}

hipError_t launch_render(const LaunchPlan &L, hipStream_t s)
{
    if (L.direct) return launch_direct(L, s);
    const uint32_t nreset = L.nviews > L.ntiles ? L.nviews : L.ntiles;
    mark(L, 0, s);
    hipLaunchKernelGGL(k_reset, dim3(cdiv(nreset > 4 ? nreset : 4, 256)), dim3(256), 0, s, L.ctr,
                       L.nviews, L.tile_count, L.tile_cursor, L.ntiles, L.queue);
    mark(L, 1, s);
    mark(L, 2, s);
    hipLaunchKernelGGL(k_cull, dim3(L.cull_blocks, L.nviews), dim3(kCullBlock), 0, s, L.views, L.ctr, L.pairs);
    const size_t pre_bytes = 4u * (size_t)L.nviews;   // the per-view prefix in LDS
    hipLaunchKernelGGL(k_setup, dim3(L.setup_grid), dim3(kSetupBlock), pre_bytes, s, L.views, L.nviews, L.ctr,
                       L.pairs, L.skey, L.sbox, L.err);
    mark(L, 3, s);
    mark(L, 4, s);
    const bool large = L.max_tiles > kLdsTiles || L.coarse;
    auto *const k_count = large ? k_bin<false, true> : k_bin<false, false>;
    hipLaunchKernelGGL(k_count, dim3(L.bin_grid), dim3(kBinBlock), pre_bytes, s,
                       L.views, L.nviews, L.ctr, L.pairs, L.skey, L.sbox, L.tile_count, L.tile_off, L.tile_cursor, L.bins,
                       L.wave_seg, L.zbuf);
    mark(L, 5, s);
    mark(L, 6, s);
    uint32_t cap16 = 0;
    for (int k = 0; k < L.nraster; ++k)
        if (L.raster[k].wave) cap16 = L.raster[k].item_cap;
    if (L.max_tiles <= 64) {
        hipLaunchKernelGGL(k_bin_scan_small, dim3(cdiv(L.nviews, kSmallScanWaves)), dim3(64 * kSmallScanWaves), 0, s,
                           L.views, L.nviews, L.ctr, L.tile_count, L.tile_off, L.tile_item, L.queue, L.items[0],
                           L.items[1], L.items[2], L.wave_seg, cap16);
    } else {
        const uint32_t nt = L.max_tiles <= 256 ? 256 : 1024;
        hipLaunchKernelGGL(nt == 256 ? k_bin_scan<256> : k_bin_scan<1024>, dim3(L.nviews), dim3(nt), 0, s, L.views, L.ctr,
                           L.tile_count, L.tile_off, L.tile_item, L.queue, L.items[0], L.items[1], L.items[2],
                           L.wave_seg, cap16);
    }
    mark(L, 7, s);
    mark(L, 8, s);
    auto *const k_scatter = large ? k_bin<true, true> : k_bin<true, false>;
    hipLaunchKernelGGL(k_scatter, dim3(L.bin_grid), dim3(kBinBlock), pre_bytes, s,
                       L.views, L.nviews, L.ctr, L.pairs, L.skey, L.sbox, L.tile_count, L.tile_off, L.tile_cursor, L.bins,
                       L.wave_seg, L.zbuf);
    mark(L, 9, s);
    for (int k = 0; k < L.nraster; ++k) {
        const RasterLaunch &R = L.raster[k];
        if (!R.blocks) continue;
        const int ph = R.ts == 8 ? 5 : R.ts == 16 ? 6 : 7;
        mark(L, 2 * ph, s);
        switch (R.ts) {
        case 8: launch_raster<8>(L, R, s); break;
        case 16: launch_raster<16>(L, R, s); break;
        case 32: launch_raster<32>(L, R, s); break;
        default: return hipErrorInvalidValue;
        }
        mark(L, 2 * ph + 1, s);
    }
    mark(L, 2 * kPhaseResolve, s);
    for (int k = 0; k < L.nraster; ++k) {
        const RasterLaunch &R = L.raster[k];
        if (!R.blocks) continue;
        switch (R.ts) {
        case 8: launch_resolve<8>(L, R, s); break;
        case 16: launch_resolve<16>(L, R, s); break;
        case 32: launch_resolve<32>(L, R, s); break;
        default: return hipErrorInvalidValue;
        }
    }
    mark(L, 2 * kPhaseResolve + 1, s);
    return hipGetLastError();
}

// ------------------------------------------------------------ self-check
__global__ __launch_bounds__(256) void k_check_recip(uint32_t lo, uint32_t hi, unsigned long long *count)
{
    const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
    uint32_t bad = 0;
    for (unsigned long long b = lo + (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; b < hi; b += stride) {
        const float x = __uint_as_float((uint32_t)b);
        bad += __float_as_uint(recip_rn(x)) != __float_as_uint(1.0f / x) ? 1u : 0u;
    }
    const uint32_t tot = wave_sum_u32(bad);
    if (lane_id() == 0 && tot) atomicAdd(count, (unsigned long long)tot);
}

hipError_t launch_check_recip(uint32_t lo, uint32_t hi, unsigned long long *count, hipStream_t s)
{
    if (!count || lo >= hi || hi > 0x7F800000u) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_check_recip, dim3(2048), dim3(256), 0, s, lo, hi, count);
    return hipGetLastError();
}

}  // namespace habmi

// Host runtime: validation, workspace arena, launch planning and staging.
#include "runtime.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <unordered_map>

namespace habmi {

static constexpr float kDefaultBinFactor = 2.0f;
static constexpr uint32_t kDefaultTile = 16;
// Pixels + triangles / 4 up to which the direct path draws a launch, a half of
// a split batch, and a launch of fine triangles of at least a pixel; or the pixels a
// triangle times kDirectDense (kDirectWide with a view of more tiles than are binned at
// once), if that is more.
static constexpr uint64_t kDirectSize = 1150 * 1024, kDirectHalf = 740 * 1024, kDirectFine = 640 * 1024;
static constexpr uint64_t kDirectDense = 100 * 1024, kDirectWide = 190 * 1024;
// ... and the visits, spread and depth (choose_tiles) up to which it does.
static constexpr double kVisits = 30000.0, kSpread = 0.2, kDepth = 16.0;
// Triangles a tile up to which the binning takes large boxes a wave at a time (k_bin has both sides).
static constexpr uint32_t kCoarseTiles = 250;
// Triangles from which the largest scene of a launch counts as fine, and its clusters, where they spread, as many.
static constexpr uint32_t kFine = 10000, kSpreadMost = 7000;
// Resolve waves that a launch keeps when a wave shades two or four bands one
// after another (its search and start paid once): two rounds of the 8192 that
// are resident.  1024 depth frames of 64 x 64 resolve in 32 us with one band a
// wave and 22 with four; 32 textured 256 x 256 views, 33 k bands, in 40 with
// one, 42 with two and 47 with four, which leaves one round of long waves.
static constexpr uint64_t kStackWaves = 16384;
static constexpr uint64_t kIndexLimit = 1ull << 31; // per launch: survivors, bins, tiles

static inline uint32_t cdiv(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// Stable sort that allocates nothing for short ranges (insertion sort; the
// allocation-free render entry plans at most 256 views); longer ranges use
// std::stable_sort.
template <class It, class Cmp>
static void stable_sort_views(It b, It e, Cmp less)
{
    if (e - b > 256) {
        std::stable_sort(b, e, less);
        return;
    }
    for (It i = b + (e > b ? 1 : 0); i < e; ++i) {
        auto x = *i;
        It j = i;
        for (; j > b && less(x, *(j - 1)); --j) *j = *(j - 1);
        *j = x;
    }
}
static inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// ---------------------------------------------------------------- allocation
namespace {
std::mutex g_alloc_mu;
int64_t g_fail_after = -1;                      // allocations left before one fails (-1: never)
std::unordered_map<void *, size_t> g_live;      // pointer -> bytes

// After g_fail_after more successes every allocation fails, until reset.
bool inject_failure()
{
    if (g_fail_after < 0) return false;
    if (g_fail_after == 0) return true;
    --g_fail_after;
    return false;
}
}  // namespace

bool dev_alloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> g(g_alloc_mu);
    *p = nullptr;
    if (inject_failure()) return false;
    if (hipMalloc(p, std::max<size_t>(bytes, 1)) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return false;
    }
    g_live[*p] = bytes;
    return true;
}

void dev_free(void *p)
{
    if (!p) return;
    std::lock_guard<std::mutex> g(g_alloc_mu);
    g_live.erase(p);
    (void)hipFree(p);
}

bool pinned_alloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> g(g_alloc_mu);
    *p = nullptr;
    if (inject_failure()) return false;
    if (hipHostMalloc(p, std::max<size_t>(bytes, 1), hipHostMallocDefault) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return false;
    }
    g_live[*p] = bytes;
    return true;
}

void pinned_free(void *p)
{
    if (!p) return;
    std::lock_guard<std::mutex> g(g_alloc_mu);
    g_live.erase(p);
    (void)hipHostFree(p);
}

void alloc_fail_after(int64_t n)
{
    std::lock_guard<std::mutex> g(g_alloc_mu);
    g_fail_after = n;
}

void alloc_live(uint64_t *count, uint64_t *bytes)
{
    std::lock_guard<std::mutex> g(g_alloc_mu);
    uint64_t b = 0;
    for (const auto &e : g_live) b += e.second;
    *count = g_live.size();
    *bytes = b;
}

// ---------------------------------------------------------------- workspace
Workspace::~Workspace()
{
    if (has_done) (void)hipEventSynchronize(done);
    for (auto &s : slots) {
        if (s.pending) (void)hipEventSynchronize(s.ev);
        if (s.host) pinned_free(s.host);
        if (s.ev) (void)hipEventDestroy(s.ev);
    }
    if (arena && !external) dev_free(arena);
    if (done) (void)hipEventDestroy(done);
}

hab_status Workspace::ensure(size_t bytes)
{
    if (!done) HAB_HIP(hipEventCreateWithFlags(&done, hipEventDisableTiming));
    if (bytes <= cap) return HAB_OK;
    if (external) return HAB_ERR_CAPACITY;
    if (has_done) HAB_HIP(hipEventSynchronize(done));
    const size_t old = cap;
    if (arena) {
        dev_free(arena);
        arena = nullptr;
        cap = 0;
    }
    size_t want = std::max(bytes, old + old / 2);
    if (!dev_alloc(&arena, want)) {
        if (!dev_alloc(&arena, bytes)) return HAB_ERR_OUT_OF_MEMORY;
        want = bytes;
    }
    cap = want;
    return HAB_OK;
}

hab_status Workspace::staging(size_t bytes, void **host, int *slot)
{
    Slot &s = slots[next];
    *slot = next;
    next = (next + 1) % kSlots;
    if (!s.ev) HAB_HIP(hipEventCreateWithFlags(&s.ev, hipEventDisableTiming));
    if (s.pending) {
        HAB_HIP(hipEventSynchronize(s.ev));
        s.pending = false;
    }
    if (s.cap < bytes) {
        if (s.host) pinned_free(s.host);
        s.host = nullptr;
        s.cap = 0;
        size_t want = std::max(bytes, (size_t)64 << 10);
        if (!pinned_alloc(&s.host, want)) return HAB_ERR_OUT_OF_MEMORY;
        s.cap = want;
    }
    *host = s.host;
    return HAB_OK;
}

hab_status Workspace::reserve_staging(size_t bytes)
{
    for (int k = 0; k < kSlots; ++k) {
        Slot &s = slots[k];
        if (!s.ev) HAB_HIP(hipEventCreateWithFlags(&s.ev, hipEventDisableTiming));
        if (s.cap >= bytes) continue;
        if (s.pending) {
            HAB_HIP(hipEventSynchronize(s.ev));
            s.pending = false;
        }
        if (s.host) pinned_free(s.host);
        s.host = nullptr;
        s.cap = 0;
        if (!pinned_alloc(&s.host, bytes)) return HAB_ERR_OUT_OF_MEMORY;
        s.cap = bytes;
    }
    return HAB_OK;
}

hab_status Workspace::staging_reserved(size_t bytes, void **host, int *slot)
{
    Slot &s = slots[next];
    if (!s.ev || !s.host || s.cap < bytes) return HAB_ERR_CAPACITY;
    *slot = next;
    next = (next + 1) % kSlots;
    if (s.pending) {
        HAB_HIP(hipEventSynchronize(s.ev));
        s.pending = false;
    }
    *host = s.host;
    return HAB_OK;
}

void Workspace::reserve_planning(uint32_t n, size_t desc_bytes)
{
    desc.reserve(desc_bytes);
    dv.reserve(n);
    tpre.reserve(n);
    for (int c = 0; c < 3; ++c) {
        lview[c].reserve(n);
        lpre[c].reserve(n);
    }
}

// ---------------------------------------------------------------- validation
static double focal_of(uint32_t W, double hfov_deg)
{
    return (double)W / (2.0 * std::tan(hfov_deg * 3.14159265358979323846 / 360.0));
}

hab_status validate_sensor(const hab_sensor *s)
{
    if (!s) return HAB_ERR_INVALID_ARG;
    if (s->width == 0 || s->height == 0 || s->width > HAB_MAX_DIM || s->height > HAB_MAX_DIM)
        return HAB_ERR_INVALID_ARG;
    if (!(s->hfov_deg > 0.0f && s->hfov_deg < 180.0f)) return HAB_ERR_INVALID_ARG;
    if (!(s->near_m > 0.0f) || !std::isfinite(s->near_m)) return HAB_ERR_INVALID_ARG;
    if (s->outputs == 0 ||
        (s->outputs & ~(uint32_t)(HAB_OUT_RGB | HAB_OUT_DEPTH | HAB_OUT_TRI | HAB_OUT_SEMANTIC)))
        return HAB_ERR_INVALID_ARG;
    if (s->f != (float)focal_of(s->width, s->hfov_deg)) return HAB_ERR_INVALID_ARG;
    if (!(s->depth_noise_sigma >= 0.0f) || !std::isfinite(s->depth_noise_sigma)) return HAB_ERR_INVALID_ARG;
    return HAB_OK;
}

// Static fixed-point domain check: with D the largest distance from the
// camera to a corner of the scene's bounding box, every vertex at w >= near
// projects to at most D f 256 / near + max(W, H) 128 in 1/256 px; requiring
// that below 2^28 keeps |X|, |Y| < 2^29 with a factor-two margin for fp32
// rounding.  The rotation must be orthonormal to 1e-4.
hab_status validate_pose(const Scene *sc, const hab_sensor *s, const hab_pose *p)
{
    for (int k = 0; k < 3; ++k)
        if (!std::isfinite(p->position[k])) return HAB_ERR_INVALID_ARG;
    for (int k = 0; k < 9; ++k)
        if (!std::isfinite(p->rotation[k])) return HAB_ERR_INVALID_ARG;
    const float *R = p->rotation;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            double d = 0.0;
            for (int k = 0; k < 3; ++k) d += (double)R[3 * k + a] * (double)R[3 * k + b];
            if (std::fabs(d - (a == b ? 1.0 : 0.0)) > 1e-4) return HAB_ERR_INVALID_ARG;
        }
    double D2 = 0.0;
    for (int c = 0; c < 8; ++c) {
        double d2 = 0.0;
        for (int a = 0; a < 3; ++a) {
            double x = ((c >> a) & 1) ? sc->hi[a] : sc->lo[a];
            double d = x - (double)p->position[a];
            d2 += d * d;
        }
        D2 = std::max(D2, d2);
    }
    double reach = std::sqrt(D2) * (double)s->f * 256.0 / (double)s->near_m +
                   (double)std::max(s->width, s->height) * 128.0;
    if (!(reach < 268435456.0)) return HAB_ERR_RANGE;
    return HAB_OK;
}

hab_status to_view_req(const hab_view &hv, ViewReq &out)
{
    if (!hv.scene || !hv.sensor) return HAB_ERR_INVALID_ARG;
    hab_status st = validate_sensor(hv.sensor);
    if (st != HAB_OK) return st;
    const Scene *sc = hv.scene;
    st = validate_pose(sc, hv.sensor, &hv.pose);
    if (st != HAB_OK) return st;
    out.scene = sc;
    out.sensor = *hv.sensor;
    out.pose = hv.pose;
    out.rgb = (hv.sensor->outputs & HAB_OUT_RGB) ? hv.out_rgb : nullptr;
    out.depth = (hv.sensor->outputs & HAB_OUT_DEPTH) ? hv.out_depth : nullptr;
    out.tri = hv.out_tri;
    out.sem = (hv.sensor->outputs & HAB_OUT_SEMANTIC) ? hv.out_semantic : nullptr;
    out.noise_seed = hv.noise_seed;
    if (out.sem && !sc->inst) return HAB_ERR_INVALID_ARG;
    return HAB_OK;
}

// ---------------------------------------------------------------- autotune table
uint32_t class_key(const Scene *sc, const hab_sensor *s)
{
    uint32_t tlog = 0;
    while ((1u << tlog) < std::max<uint32_t>(sc->T, 1)) ++tlog;
    uint32_t wlog = 0;
    while ((1u << wlog) < std::max(s->width, s->height)) ++wlog;
    return (tlog << 9) | (wlog << 4) | (s->outputs & 15u);
}

uint32_t choose_tile(hab_context *ctx, const Scene *sc, const hab_sensor *s, const PlanOpts &o,
                     float *bin_factor)
{
    *bin_factor = o.bin_factor > 0.0f ? o.bin_factor : kDefaultBinFactor;
    if (o.tile_size) return o.tile_size;
    if (ctx) {
        const uint32_t key = class_key(sc, s);
        std::lock_guard<std::mutex> g(ctx->tune_mu);
        for (const Tuned &t : ctx->tuned)
            if (t.key == key) {
                if (o.bin_factor <= 0.0f) *bin_factor = t.bin_factor;
                return t.ts;
            }
    }
    return kDefaultTile;
}

// ---------------------------------------------------------------- planning
static inline uint32_t ts_log2(uint32_t ts) { return ts == 8 ? 3u : ts == 16 ? 4u : 5u; }

// How the direct path would draw a launch.
struct DirectTiles {
    uint32_t edge = 16, shares = 1;   // tile edge, blocks that share a tile's clusters
    double visits = 0.0;              // (cluster, tile) pairs it sets up, an estimate
    double depth = 0.0;               // clusters that a wave draws one after another where the whole scene
                                      //   falls on few tiles (0: it does not)
    double spread = 0.0;              // of the launch's triangles (Scene::spread)
    double density = 0.0;             // pixels a triangle
    double ragged = 1.0;              // the tiles' pixels, of the images'
};

// The part of the image that the box around a scene takes, if all of it lies in
// front of the camera (else 1).
static double covered(const ViewReq &r)
{
    const Scene &sc = *r.scene;
    const float *p = r.pose.position, *R = r.pose.rotation;
    if (p[0] >= sc.lo[0] && p[0] <= sc.hi[0] && p[1] >= sc.lo[1] && p[1] <= sc.hi[1] && p[2] >= sc.lo[2] && p[2] <= sc.hi[2])
        return 1.0;
    double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    for (int c = 0; c < 8; ++c) {
        double d[3];
        for (int a = 0; a < 3; ++a) d[a] = (double)((c >> a) & 1 ? sc.hi[a] : sc.lo[a]) - p[a];
        const double w = -(R[2] * d[0] + R[5] * d[1] + R[8] * d[2]);
        if (!(w > r.sensor.near_m)) return 1.0;
        const double x = r.sensor.f * (R[0] * d[0] + R[3] * d[1] + R[6] * d[2]) / w;
        const double y = r.sensor.f * (R[1] * d[0] + R[4] * d[1] + R[7] * d[2]) / w;
        x0 = std::min(x0, x), x1 = std::max(x1, x);
        y0 = std::min(y0, y), y1 = std::max(y1, y);
    }
    const double W = r.sensor.width, H = r.sensor.height;
    const double w = std::min(x1, W / 2) - std::max(x0, -W / 2), h = std::min(y1, H / 2) - std::max(y0, -H / 2);
    return std::max(w, 0.0) * std::max(h, 0.0) / (W * H);
}

// Of a view's clusters about a quarter is in sight, each about as large as an
// equal part of four times the image, and it meets every tile that it touches;
// but clusters that spread over the scene (whose 64 triangles are not neighbours)
// are in sight, and in every tile.
//
// The edge follows the largest scene (finer triangles, larger tiles: fewer
// clusters meet several).  It grows where there are many tiles, but of triangles
// of many pixels 64-pixel tiles hold too much (a frame of 512 x 512 over 20k
// triangles: 73 us with 32-pixel tiles, 176 with 64; twelve of 256 x 256 over 60k
// 189 and 122; five of 512 x 512 over 2k 89 and 149), and where clusters spread
// (one of 128 x 128 over 9.7k shuffled triangles: 70 and 52, 101 with 16-pixel
// tiles, but with half of them in order 62 and 64; four of 128 x 128 over 60k shuffled
// triangles: 113 and 63).  The shares give each wave of a block one or two
// clusters to draw, up to a round or two of resident blocks.  (One 256 x 256 view
// of 200k triangles: 64-pixel tiles with 4 / 16 / 64 shares take 105 / 57 / 66 us,
// 32-pixel tiles with 16 take 56.)
static DirectTiles choose_tiles(const ViewReq *v, uint32_t n)
{
    DirectTiles t;
    uint32_t max_t = 0;
    double px = 0.0, tri = 0.0;
    for (uint32_t k = 0; k < n; ++k) {
        max_t = std::max(max_t, v[k].scene->T);
        px += (double)v[k].sensor.width * v[k].sensor.height;
        tri += v[k].scene->T;
        t.spread += (double)v[k].scene->T * v[k].scene->spread;
    }
    t.spread /= std::max(tri, 1.0);
    t.density = px / std::max(tri, 1.0);
    const bool fine = max_t >= kFine;
    double tiles = 0.0, per_tile = 0.0;   // clusters that meet a tile, over the views
    auto count = [&]() {
        tiles = per_tile = t.visits = 0.0;
        double vt = 0.0, vp = 0.0, vv = 0.0;   // of the view before, often the same
        for (uint32_t k = 0; k < n; ++k) {
            const Scene &sc = *v[k].scene;
            const uint32_t W = v[k].sensor.width, H = v[k].sensor.height;
            if (!k || v[k - 1].scene != v[k].scene || v[k - 1].sensor.width != W || v[k - 1].sensor.height != H) {
                const double ncl = cdiv(sc.T, kCluster), seen = std::max(1.0, 0.27 * ncl);
                const double across = 1.0 + std::sqrt(4.0 * W * H / seen) / t.edge;
                vt = (double)cdiv(W, t.edge) * cdiv(H, t.edge);
                vp = std::min(seen * across * across / vt, seen);
                vv = vt * (vp * (1.0 - sc.spread) + ncl * sc.spread);
            }
            tiles += vt;
            per_tile += vp;
            t.visits += vv;
        }
    };
    auto most_tiles = [&](uint32_t edge) {
        const double by_density = 100.0 + 150.0 * t.density;
        return fine ? by_density : edge < 32 ? 1024.0 : std::max(1024.0, by_density);
    };
    const bool mixed = t.spread > kSpread && (fine || (t.spread > 4.0 * kSpread && max_t >= kSpreadMost && t.density < 8.0));
    t.edge = max_t >= 128000 || mixed ? 64u : fine ? 32u : 16u;
    for (count(); t.edge < 64 && (tiles > most_tiles(t.edge) || (t.edge < 32 && t.visits > kVisits)); count())
        t.edge *= 2;
    t.ragged = tiles * t.edge * t.edge / std::max(px, 1.0);
    const double waves = t.edge == 64 ? 8 : 4;
    const double want = std::min(1.5 * per_tile / n / waves, 256.0);
    const double most = (max_t >= 500000 ? 2048.0 : 1024.0) / std::max(tiles, 1.0);
    t.shares = (uint32_t)std::max(1.0, std::min(want, most));
    for (uint32_t k = 0; k < n; ++k) {
        const double part = covered(v[k]);
        if (part >= 1.0) continue;
        // (a cluster of triangles of half a pixel and more takes four times as long as one whose triangles mostly
        // cover none, and the lists of a large image take longer too; shares of a tile that touch only a few pixels
        // also wait for each other)
        const uint32_t W = v[k].sensor.width, H = v[k].sensor.height, T = v[k].scene->T;
        const double few = std::max(1.0, part * cdiv(W, t.edge) * cdiv(H, t.edge)), seen = part * W * H;
        const double each = (1.0 + std::min(3.4, 6.8 * seen / std::max(T, 1u))) / (1.0 + (double)W * H / 1048576.0);
        t.depth = std::max(t.depth, each * cdiv(T, kCluster) / (few * t.shares * waves) + (seen < 256.0 ? t.shares / 16.0 : 0.0));
    }
    return t;
}

// Does the direct path draw this launch?  It serves launches that ask for
// nothing the tile lists alone provide (a tiling, a list capacity, the
// lane-owned z-test, work counters), while they are small: the tile lists
// take eight dependent kernels whatever the size, the direct path four, but it
// sets up a triangle once per tile its cluster meets.  Measured (us a launch,
// tile lists against direct, by pixels + triangles / 4 in K): one 256 x 256 view
// of 200k triangles 92 / 61 (113), of 1M 87 / 51 (308), two of 1M 93 / 74 (616),
// twelve of 256 x 256 over 60k 119 / 122 (943), 16 of 128 x 128 over 200k 110 / 92
// (1044), four of 1M 119 / 133 (1232), three 512 x 384 views of 1M 122 / 156
// (1308), eight 128 x 96 of 1M 121 / 125 (2049).  The two halves of a split batch
// overlap, so theirs is the lower limit (back to back and with a wait, over 2k
// triangles, by the size of a half: 1025 views of 24 x 20 210 / 200 and 280 / 243
// (490), 1500 247 / 244 and 330 / 300 (718), 2048 295 / 304 and 399 / 370 (980)).
//
// The lists gain on fine triangles of a pixel and more (eight of 256 x 256 over 20k
// (565) 108 / 120, twelve (847) 114 / 136, eight over 60k (632) 106 / 110, three of 512 x
// 512 over 60k (813) 123 / 127) and lose again where a triangle has so many that a wave
// to a tile is slow: four of 512 x 512 over 20k (1044; 13 pixels a triangle) 150 / 144,
// five (1305) 161 / 164, eight (2088) 197 / 204, five over 2k (1282; 131) 179 / 95, 16
// (4104) 235 / 186, 48 of 256 x 256 over 2k (3096; 33) 182 / 152, 20 over 5k (1305; 13)
// 142 / 142.  Larger images are binned in windows: one of 1200 x 1000 over 100k (1196;
// 12) 263 / 157, one of 1600 x 1200 over 60k (1890; 32) 419 / 167.
// Images that fill little of their 64-pixel tiles share them among fewer blocks: over
// 200k triangles 12 of 128 x 128 (790) 102 / 77, of 129 x 129 102 / 102, 16 (1065)
// 105 / 91 and 105 / 140; 14 of 200 x 150 (1094) 111 / 141.
//
// Nor where its work is out of proportion to that size.  A visit takes about a
// nanosecond, and the lists about 30 us more than the direct path without any,
// and more again where a triangle has many pixels.  With each scene's triangles
// shuffled: one 512 x 512 view of 1M 114 / 805 (966k visits), one 256 x 256 view
// of 200k 84 / 117 (49k), eight of 128 x 128 over 60k 94 / 91 (29k), one 203 x 117
// of 200k 79 / 75 (20k); three 512 x 512 of a 2k-triangle room, 131 pixels a
// triangle, 190 / 83 (24k).  Spread clusters of several pixels a triangle also
// leave whole tiles to a wave: one 256 x 256 view of 20k shuffled triangles 89 / 117,
// 24 over 7.5k triangles, half of them shuffled, 167 / 222.
// A scene that falls on few tiles leaves the other tiles' blocks without work: within
// two pixels of a 256 x 256 view 1M triangles 58 / 108 (a depth of 31), 60k 53 / 100
// (45), within a fortieth of a 128 x 128 view 200k 61 / 33 (8), of four 512 x 512
// views 2k 80 / 56 (16), 5k 86 / 75 (10), 20k 88 / 141 (39).
static bool direct_launch(const ViewReq *v, uint32_t n, const PlanOpts &o, DirectTiles *t)
{
    if (o.tile_lists || o.tile_size || o.bin_factor > 0.0f || o.tile_cap || o.lane_owned_z || o.count_work) return false;
    uint64_t size = 0, px = 0, tri = 0;
    uint32_t max_t = 0, most = 0;
    for (uint32_t k = 0; k < n; ++k) {
        most = std::max(most, cdiv(v[k].sensor.width, kDefaultTile) * cdiv(v[k].sensor.height, kDefaultTile));
        const uint64_t view = (uint64_t)v[k].sensor.width * v[k].sensor.height;
        size += view + v[k].scene->T / 4;
        px += view;
        tri += v[k].scene->T;
        max_t = std::max(max_t, v[k].scene->T);
    }
    const double density = (double)px / std::max<uint64_t>(tri, 1);
    double limit = o.half ? kDirectHalf : kDirectSize;
    if (max_t >= kFine && density >= 1.0) limit = std::min(limit, (double)kDirectFine);
    if (!o.half) limit = std::max(limit, (most > kLdsTiles ? kDirectWide : kDirectDense) * density);
    if ((double)size > limit) return false;
    *t = choose_tiles(v, n);
    if (max_t >= kFine && t->edge == 64 && size * (1.0 + 0.35 * std::min(t->ragged - 1.0, 1.2)) > limit) return false;
    if (max_t >= kSpreadMost && max_t < kFine && t->spread > kSpread && t->edge == 64 && t->visits > 5000.0 * std::sqrt(t->density))
        return false;
    if (max_t >= kFine && t->spread > kSpread) return t->density < 1.0 && t->visits <= kVisits;
    return t->visits <= kVisits + 8000.0 * std::sqrt(std::min(t->density, 64.0)) && t->depth <= kDepth;
}

hab_status build_plan(hab_context *ctx, Workspace &ws, const ViewReq *v, uint32_t n,
                      const PlanOpts &o, Plan &plan, std::vector<uint8_t> &desc)
{
    if (n == 0 || n > kMaxViews) return HAB_ERR_INVALID_ARG;
    plan.n = n;
    plan.order.resize(n);
    std::iota(plan.order.begin(), plan.order.end(), 0u);
    stable_sort_views(plan.order.begin(), plan.order.end(),
                      [&](uint32_t a, uint32_t b) { return v[a].scene < v[b].scene; });

    // the workspace's buffers: no allocation once they have grown to n views
    std::vector<DView> &dv = ws.dv;
    dv.resize(n);
    std::vector<uint32_t> *lview = ws.lview, *lpre = ws.lpre;
    for (int c = 0; c < 3; ++c) {
        lview[c].clear();
        lpre[c].clear();
    }
    DirectTiles dt;
    const bool direct = direct_launch(v, n, o, &dt);
    uint64_t tile_total = 0, surv_total = 0, bin_total = 0, pair_total = 0;
    for (uint32_t k = 0; k < n; ++k) {
        const ViewReq &r = v[plan.order[k]];
        float bf;
        uint32_t ts = choose_tile(ctx, r.scene, &r.sensor, o, &bf);
        if (ts != 8 && ts != 16 && ts != 32) return HAB_ERR_INVALID_ARG;
        DView &d = dv[k];
        std::memset(&d, 0, sizeof d);
        for (int a = 0; a < 3; ++a) d.p[a] = r.pose.position[a];
        for (int a = 0; a < 9; ++a) d.R[a] = r.pose.rotation[a];
        d.fS = r.sensor.f * 256.0f;
        d.cxS = (float)r.sensor.width * 128.0f;
        d.cyS = (float)r.sensor.height * 128.0f;
        d.zn = r.sensor.near_m;
        d.W = r.sensor.width;
        d.H = r.sensor.height;
        d.T = r.scene->T;
        d.ts_log2 = ts_log2(ts);
        d.tpos = r.scene->tpos;
        d.attr = r.scene->attr;
        d.cbox = r.scene->cbox;
        d.rgb = r.rgb;
        d.depth = r.depth;
        d.tri = r.tri;
        d.inst = r.scene->inst;
        d.sem = r.sem;
        d.noise_sigma = r.sensor.depth_noise_sigma;
        d.noise_seed = r.noise_seed;
        d.tex = r.scene->tex;
        d.tex_w = r.scene->tw;
        d.tex_h = r.scene->th;
        d.tiles_x = cdiv(d.W, ts);
        d.tiles_y = cdiv(d.H, ts);
        d.tile_base = (uint32_t)tile_total;
        tile_total += (uint64_t)d.tiles_x * d.tiles_y;
        d.surv_base = (uint32_t)surv_total;
        surv_total += 2ull * d.T;
        uint64_t bc = (uint64_t)std::ceil((double)bf * (double)d.T);
        bc = std::max<uint64_t>(bc, 1024);
        bc = std::min<uint64_t>(bc, kIndexLimit / 4);
        d.bin_base = (uint32_t)bin_total;
        d.bin_cap = (uint32_t)bc;
        bin_total += bc;
        d.tile_cap = o.tile_cap ? o.tile_cap : 0xFFFFFFFFu;
        d.count_work = o.count_work ? 1u : 0u;
        d.pair_base = (uint32_t)pair_total;
        pair_total += cdiv(d.T, kCluster);
        // one resolve list for a direct launch, under the first view's tile size
        const int c = (int)(direct ? dv[0].ts_log2 : d.ts_log2) - 3;
        lview[c].push_back(k);
    }
    uint32_t stack[3] = {1, 1, 1};   // bands a resolve block shades
    // Raster blocks are dispatched roughly in block order: put the views of
    // the largest scenes (the longest tile lists) first so that their tiles
    // do not form the tail of the launch.
    for (int c = 0; c < 3; ++c) {
        stable_sort_views(lview[c].begin(), lview[c].end(),
                          [&](uint32_t a, uint32_t b) { return dv[a].T > dv[b].T; });
        uint64_t bands = 0;
        for (uint32_t k : lview[c]) bands += (uint64_t)cdiv(dv[k].W, 32u) * cdiv(dv[k].H, 2u);
        if (!direct && c == 1 && !o.lane_owned_z)
            stack[c] = bands >= 4 * kStackWaves ? 4u : bands >= 2 * kStackWaves ? 2u : 1u;
        // lpre: each view's first resolve block
        uint32_t pre = 0;
        for (uint32_t k : lview[c]) {
            lpre[c].push_back(pre);
            pre += cdiv(dv[k].W, 32u) * cdiv(dv[k].H, 2 * stack[c]);
        }
    }
    if (tile_total >= kIndexLimit || surv_total >= kIndexLimit || bin_total >= kIndexLimit ||
        pair_total >= kIndexLimit)
        return HAB_ERR_CAPACITY;

    const uint64_t npairs = pair_total;
    uint32_t max_t = 0;
    for (uint32_t k = 0; k < n; ++k) max_t = std::max(max_t, dv[k].T);

    // descriptor block
    uint32_t nclass[3] = {0, 0, 0};
    for (uint32_t k = 0; k < n; ++k) ++nclass[dv[k].ts_log2 - 3];
    size_t off = 0;
    plan.off_views = off;
    off = align256(off + sizeof(DView) * n);
    for (int c = 0; c < 3; ++c) {
        plan.off_lview[c] = off;
        off = align256(off + 4 * (size_t)nclass[c]);
        plan.off_lpre[c] = off;
        off = align256(off + 4 * (size_t)nclass[c]);
    }
    plan.off_ctl = off;          // control slot (the stepper's device-pose pointer)
    off = align256(off + 16);
    plan.desc_bytes = off;
    // scratch
    plan.off_ctr = off;
    off = align256(off + sizeof(DViewCounters) * n);
    plan.off_tcount = off;
    off = align256(off + 4 * tile_total);
    plan.off_toff = off;
    off = align256(off + 4 * tile_total);
    plan.off_tcur = off;
    off = align256(off + 4 * tile_total);
    plan.off_skey = off;
    off = align256(off + 4 * surv_total);
    plan.off_sbox = off;
    off = align256(off + 8 * surv_total);
    plan.off_bins = off;
    off = align256(off + 4 * bin_total);
    plan.off_pairs = off;
    off = align256(off + 4 * std::max<uint64_t>(npairs, 1));
    plan.off_titem = off;
    off = align256(off + 4 * tile_total);
    plan.off_queue = off;
    off = align256(off + sizeof(DQueue));
    // raster work items: a tile holds at most one item per kSegPerTile*TS^2
    // list entries (plus one), so a view needs at most tiles + bin_cap / S
    uint64_t item_cap[3] = {0, 0, 0};
    for (uint32_t k = 0; k < n; ++k) {
        const uint64_t S = (uint64_t)kSegPerTile << (2 * dv[k].ts_log2);
        item_cap[dv[k].ts_log2 - 3] += (uint64_t)dv[k].tiles_x * dv[k].tiles_y + (dv[k].bin_cap + S - 1) / S;
    }
    // a wave per 16-pixel tile: smaller work items, but one set of z-keys per
    // tile whatever its items; both fit the space the block form takes
    const bool wave16 = !o.lane_owned_z;
    uint64_t wave_tiles = 0, wave_items = 0, wave_tri = 0;
    uint32_t wave_seg = 0, wave_most = 0;
    for (uint32_t k = 0; k < n && wave16; ++k) {
        if (dv[k].ts_log2 != 4) continue;
        wave_tiles += (uint64_t)dv[k].tiles_x * dv[k].tiles_y;
        wave_tri += dv[k].T;
        wave_most = std::max(wave_most, dv[k].T);
    }
    if (wave16) wave_seg = wave_tiles < kWaveManyTiles ? kWaveSeg : kWaveSegLarge;
    // (a list of more than kMaxSegments items would overflow)
    for (int k = 1; k >= 0; --k)
        if (wave_seg && wave_tiles < kWaveManyTiles && wave_tri <= kWaveTriangles[k] && 2ull * wave_most < (uint64_t)kWaveSegSmall[k] * (kMaxSegments - 1))
            wave_seg = kWaveSegSmall[k];
    wave_tiles = 0;
    for (int c = 0; c < 3; ++c) {
        plan.off_items[c] = off;
        if (c == 1 && wave16) {
            for (uint32_t k = 0; k < n; ++k) {
                DView &d = dv[k];
                if (d.ts_log2 != 4) continue;
                d.zoff_lo = (uint32_t)(wave_tiles * 256);
                d.zoff_hi = (uint32_t)((wave_tiles * 256) >> 32);
                wave_tiles += (uint64_t)d.tiles_x * d.tiles_y;
                wave_items += (uint64_t)d.tiles_x * d.tiles_y + (d.bin_cap + wave_seg - 1) / wave_seg;
            }
            plan.off_zbuf = align256(off + 8 * wave_items);
        }
        off = align256(off + 8 * item_cap[c]);
        plan.off_partial[c] = off;
        off = align256(off + 8 * item_cap[c] * (64ull << (2 * c)));
        if (c == 1 && wave16) {
            off = std::max(off, align256((size_t)(plan.off_zbuf + 8 * 256 * wave_tiles)));
            item_cap[1] = wave_items;
        }
    }
    plan.arena_bytes = off;

    LaunchPlan &L = plan.L;
    L = LaunchPlan{};
    L.nviews = n;
    L.direct = direct;
    L.wave_seg = wave_seg;
    std::vector<uint32_t> &tpre = ws.tpre;
    const int c0 = (int)dv[0].ts_log2 - 3;
    if (direct) {
        // its own layout of the same arena, whose size stays the tile lists'
        // (they take more: 24 B a triangle and 4 KiB a view against 4 B, and
        // at least as many z-keys), so a launch fits a given scratch or does
        // not whichever path draws it
        uint64_t znum = 0;
        for (uint32_t k = 0; k < n; ++k) {
            DView &d = dv[k];
            d.zoff_lo = (uint32_t)znum;
            d.zoff_hi = (uint32_t)(znum >> 32);
            znum += ((uint64_t)d.W * d.H + 1) & ~1ull;
        }
        L.tile_edge = dt.edge;
        L.shares = dt.shares;
        tpre.clear();
        uint64_t pre = 0;
        for (uint32_t k : lview[c0]) {
            tpre.push_back((uint32_t)pre);
            pre += (uint64_t)cdiv(dv[k].W, L.tile_edge) * cdiv(dv[k].H, L.tile_edge) * L.shares;
        }
        if (pre >= kIndexLimit) return HAB_ERR_CAPACITY;
        L.tile_grid = (uint32_t)pre;
        L.znum = znum;
        size_t x = align256(sizeof(DView) * n);
        plan.off_lview[c0] = x;
        x = align256(x + 4 * (size_t)n);
        plan.off_lpre[c0] = x;
        x = align256(x + 4 * (size_t)n);
        plan.off_tpre = x;
        x = align256(x + 4 * (size_t)n);
        plan.off_ctl = x;
        x = align256(x + 16);
        plan.desc_bytes = x;
        plan.off_ctr = x;
        x = align256(x + sizeof(DViewCounters) * n);
        plan.off_recs = x;
        x = align256(x + sizeof(ClusterRec) * kBuckets * std::max<uint64_t>(npairs, 1));
        plan.off_zbuf = x;
        x = align256(x + 8 * znum);
        plan.arena_bytes = std::max(plan.arena_bytes, x);
    }
    desc.resize(plan.desc_bytes);
    std::memcpy(desc.data() + plan.off_views, dv.data(), sizeof(DView) * n);
    for (int c = 0; c < 3; ++c) {
        if (!lview[c].empty()) {
            std::memcpy(desc.data() + plan.off_lview[c], lview[c].data(), 4 * lview[c].size());
            std::memcpy(desc.data() + plan.off_lpre[c], lpre[c].data(), 4 * lpre[c].size());
        }
    }
    if (direct) std::memcpy(desc.data() + plan.off_tpre, tpre.data(), 4 * tpre.size());
    L.cull_blocks = std::max<uint32_t>(1, cdiv(cdiv(max_t, kCluster), 256));
    // one round of resident setup blocks (the waves take static shares of
    // the work, so a second partial round would only add a tail)
    const uint64_t setup_resident = (uint64_t)kSetupWavesPerSimd * 4 / (kSetupBlock / 64);
    L.setup_grid = (uint32_t)std::max<uint64_t>(
        1, std::min<uint64_t>((npairs + 15) / 16, setup_resident * (ctx ? ctx->cu_count : 256)));
    L.ntiles = (uint32_t)tile_total;
    uint64_t tri = 0;
    for (uint32_t k = 0; k < n; ++k) {
        L.max_tiles = std::max(L.max_tiles, dv[k].tiles_x * dv[k].tiles_y);
        tri += dv[k].T;
    }
    L.coarse = tile_total * kCoarseTiles >= tri;
    uint64_t ub = 0;
    for (uint32_t k = 0; k < n; ++k) ub += cdiv(dv[k].T, kCluster * kRun * kBinRuns);
    L.bin_grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(ub, 8ull * (ctx ? ctx->cu_count : 256)));
    L.nraster = 0;
    const uint32_t cus = ctx ? (uint32_t)ctx->cu_count : 256u;
    const int lo = o.lane_owned_z ? 1 : 0;
    const uint32_t kBlocksPerCu[3] = {ctx ? (uint32_t)ctx->raster_bpc[lo][0] : 1u,
                                      ctx ? (uint32_t)ctx->raster_bpc[lo][1] : 1u,
                                      ctx ? (uint32_t)ctx->raster_bpc[lo][2] : 1u};
    for (int c = 0; c < 3; ++c) {
        if (lview[c].empty()) continue;
        RasterLaunch &R = L.raster[L.nraster++];
        R.ts = c == 0 ? 8 : c == 1 ? 16 : 32;
        R.nl = (uint32_t)lview[c].size();
        const DView &last = dv[lview[c].back()];
        R.blocks = 0;
        for (uint32_t k : lview[c]) R.blocks += dv[k].tiles_x * dv[k].tiles_y;
        R.bands = lpre[c].back() + cdiv(last.W, 32u) * cdiv(last.H, 2 * stack[c]);
        R.stack = stack[c];
        R.item_cap = (uint32_t)item_cap[c];
        R.lane_owned = o.lane_owned_z;
        R.wave = c == 1 && wave16;
        // k_raster_wave may cut overflow tiles into more items than there is room for in the list
        R.grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(item_cap[c] * (R.wave ? 4 : 1), (uint64_t)cus * kBlocksPerCu[c]));
    }
    return HAB_OK;
}

void bind_plan(Plan &plan, void *arena, uint32_t *err)
{
    char *b = static_cast<char *>(arena);
    LaunchPlan &L = plan.L;
    L.views = reinterpret_cast<const DView *>(b + plan.off_views);
    L.ctr = reinterpret_cast<DViewCounters *>(b + plan.off_ctr);
    L.tile_count = reinterpret_cast<uint32_t *>(b + plan.off_tcount);
    L.tile_off = reinterpret_cast<uint32_t *>(b + plan.off_toff);
    L.tile_cursor = reinterpret_cast<uint32_t *>(b + plan.off_tcur);
    L.skey = reinterpret_cast<uint32_t *>(b + plan.off_skey);
    L.sbox = reinterpret_cast<uint2 *>(b + plan.off_sbox);
    L.bins = reinterpret_cast<uint32_t *>(b + plan.off_bins);
    L.tile_item = reinterpret_cast<uint32_t *>(b + plan.off_titem);
    L.queue = reinterpret_cast<DQueue *>(b + plan.off_queue);
    L.pairs = reinterpret_cast<uint32_t *>(b + plan.off_pairs);
    L.recs = reinterpret_cast<ClusterRec *>(b + plan.off_recs);
    L.tpre = reinterpret_cast<const uint32_t *>(b + plan.off_tpre);
    L.zbuf = reinterpret_cast<unsigned long long *>(b + plan.off_zbuf);
    L.err = err;
    for (int c = 0; c < 3; ++c) L.items[c] = reinterpret_cast<uint2 *>(b + plan.off_items[c]);
    for (int k = 0; k < L.nraster; ++k) {
        RasterLaunch &R = L.raster[k];
        const int c = R.ts == 8 ? 0 : R.ts == 16 ? 1 : 2;
        R.lview = reinterpret_cast<const uint32_t *>(b + plan.off_lview[c]);
        R.bpre = reinterpret_cast<const uint32_t *>(b + plan.off_lpre[c]);
        R.items = reinterpret_cast<uint2 *>(b + plan.off_items[c]);
        R.partial = reinterpret_cast<uint2 *>(b + plan.off_partial[c]);
    }
}

Footprint footprint(const ViewReq *v, uint32_t n, const PlanOpts &o, hab_context *ctx)
{
    Footprint f;
    uint64_t bytes = 0, tiles = 0;
    for (uint32_t k = 0; k < n; ++k) {
        float bf;
        uint32_t ts = choose_tile(ctx, v[k].scene, &v[k].sensor, o, &bf);
        uint64_t nt = (uint64_t)cdiv(v[k].sensor.width, ts) * cdiv(v[k].sensor.height, ts);
        tiles += nt;
        uint64_t bc = std::max<uint64_t>((uint64_t)std::ceil((double)bf * v[k].scene->T), 1024);
        const uint64_t S = (uint64_t)kSegPerTile * ts * ts;
        const uint64_t items = nt + (bc + S - 1) / S;
        bytes += 2ull * v[k].scene->T * 12ull + bc * 4ull + nt * 16ull + sizeof(DView) + sizeof(DViewCounters) + 64 +
                 4ull * cdiv(v[k].scene->T, kCluster) +
                 items * 8ull * (1 + (uint64_t)ts * ts);
    }
    f.desc_bytes = n * (sizeof(DView) + 32) + 4096;
    // + the work queues and the padding of the plan's 24 aligned arrays; a
    // multiple of 256, so that regions packed one after another in a pool
    // keep the arena's alignment (64-bit atomics need theirs)
    f.arena_bytes = align256(bytes + f.desc_bytes + sizeof(DQueue) + 31 * 256);
    (void)tiles;
    return f;
}

// ---------------------------------------------------------------- launching
// The descriptor block (in ws.desc) on its way to the arena: into `desc`, which
// the direct path's first kernel takes as an argument, or through a pinned slot
// and a copy on stream s.
static hab_status stage(Workspace &ws, Plan &plan, void *arena, hipStream_t s, bool reserved, InlineDesc &desc)
{
    if (plan.L.direct && plan.desc_bytes <= kInlineDesc) {
        std::memcpy(desc.bytes, ws.desc.data(), plan.desc_bytes);
        plan.L.desc = &desc;
        plan.L.desc_bytes = (uint32_t)plan.desc_bytes;
        return HAB_OK;
    }
    void *host;
    int slot;
    const hab_status st = reserved ? ws.staging_reserved(plan.desc_bytes, &host, &slot)
                                   : ws.staging(plan.desc_bytes, &host, &slot);
    if (st != HAB_OK) return st;
    std::memcpy(host, ws.desc.data(), plan.desc_bytes);
    HAB_HIP(hipMemcpyAsync(arena, host, plan.desc_bytes, hipMemcpyHostToDevice, s));
    HAB_HIP(hipEventRecord(ws.slots[slot].ev, s));
    ws.slots[slot].pending = true;
    return HAB_OK;
}

hab_status render_views(hab_context *ctx, Workspace &ws, const ViewReq *v, uint32_t n,
                        const PlanOpts &opts, hipStream_t s, hab_view_stats *stats)
{
    PlanOpts o = opts;
    o.count_work = stats != nullptr;
    Plan plan;
    hab_status st = build_plan(ctx, ws, v, n, o, plan, ws.desc);
    if (st != HAB_OK) return st;
    st = ws.ensure(plan.arena_bytes);
    if (st != HAB_OK) return st;
    if (reinterpret_cast<uintptr_t>(ws.arena) % 256) return HAB_ERR_DEVICE;   // a misplaced region: 64-bit atomics would fault
    if (ws.has_done && ws.last_stream != s) HAB_HIP(hipStreamWaitEvent(s, ws.done, 0));
    InlineDesc desc;
    st = stage(ws, plan, ws.arena, s, false, desc);
    if (st != HAB_OK) return st;
    bind_plan(plan, ws.arena, ctx->err);
    hab_context::ProfSet *ps = nullptr;
    if (ctx->prof_on) {
        if (ctx->prof_used == ctx->prof_sets.size()) {
            hab_context::ProfSet fresh{};
            for (int e = 0; e < kProfEvents; ++e) HAB_HIP(hipEventCreate(&fresh.ev[e]));
            ctx->prof_sets.push_back(fresh);
        }
        ps = &ctx->prof_sets[ctx->prof_used++];
        ps->mask = (plan.L.direct ? 0x3u : 0x1Fu) | (1u << kPhaseResolve);
        for (int k = 0; k < plan.L.nraster; ++k)
            if (plan.L.raster[k].blocks)
                ps->mask |= 1u << (plan.L.raster[k].ts == 8 ? 5 : plan.L.raster[k].ts == 16 ? 6 : 7);
        ps->mask &= ctx->prof_phase_mask;
        plan.L.prof = ps->ev;
        plan.L.prof_mask = ps->mask;
    }
    HAB_HIP(launch_render(plan.L, s));
    HAB_HIP(hipEventRecord(ws.done, s));
    ws.has_done = true;
    ws.last_stream = s;
    if (stats) {
        std::vector<DViewCounters> c(n);
        HAB_HIP(hipMemcpyAsync(c.data(), plan.L.ctr, sizeof(DViewCounters) * n, hipMemcpyDeviceToHost, s));
        HAB_HIP(hipStreamSynchronize(s));
        for (uint32_t k = 0; k < n; ++k) {
            hab_view_stats &o2 = stats[plan.order[k]];
            o2.survivors = c[k].surv_count;
            o2.bbox_tests = c[k].bbox_tests;
            o2.covered = c[k].covered;
        }
    }
    return HAB_OK;
}

hab_status stage_and_launch(hab_context *ctx, Workspace &ws, Plan &plan, void *arena, hipStream_t s,
                            bool reserved)
{
    InlineDesc desc;
    const hab_status st = stage(ws, plan, arena, s, reserved, desc);
    if (st != HAB_OK) return st;
    bind_plan(plan, arena, ctx->err);
    HAB_HIP(launch_render(plan.L, s));
    return HAB_OK;
}

hab_status render_all(hab_context *ctx, Workspace &ws, const ViewReq *v, uint32_t n,
                      const PlanOpts &o, hipStream_t s, hab_view_stats *stats)
{
    uint32_t k = 0;
    while (k < n) {
        uint32_t e = k;
        uint64_t surv = 0, bins = 0;
        while (e < n && e - k < kMaxViews) {
            float bf;
            (void)choose_tile(ctx, v[e].scene, &v[e].sensor, o, &bf);
            const uint64_t s2 = 2ull * v[e].scene->T;
            const uint64_t b2 = std::max<uint64_t>((uint64_t)std::ceil((double)bf * v[e].scene->T), 1024);
            if (e > k && (surv + s2 >= kIndexLimit / 2 || bins + b2 >= kIndexLimit / 2)) break;
            surv += s2;
            bins += b2;
            ++e;
        }
        hab_status st = render_views(ctx, ws, v + k, e - k, o, s, stats ? stats + k : nullptr);
        if (st != HAB_OK) return st;
        k = e;
    }
    return HAB_OK;
}

hab_status ensure_aux(hab_context *ctx)
{
    if (!ctx->aux) HAB_HIP(hipStreamCreateWithFlags(&ctx->aux, hipStreamNonBlocking));
    if (!ctx->fork_ev) HAB_HIP(hipEventCreateWithFlags(&ctx->fork_ev, hipEventDisableTiming));
    if (!ctx->join_ev) HAB_HIP(hipEventCreateWithFlags(&ctx->join_ev, hipEventDisableTiming));
    return HAB_OK;
}

// Measured (us a launch; one sequence, two), back to back and with a wait after
// each, by pixels + triangles / 4 in millions: 256 views of 64 x 64 over 20k
// triangles (2.3) 141 / 174 and 180 / 247; 64 of 100 x 80 over 50k to 400k (3.4)
// 142 / 156 and 173 / 221; 32 of 256 x 256 over 100k to 1M (6) 198 / 205 and
// 227 / 278; 64 of 160 x 160 over 100k to 800k (7) 239 / 239 and 271 / 307; the
// same 48 of 256 x 256 (9) 279 / 270 and 309 / 341, 64 (12) 374 / 354 and 403 /
// 413, 128 (24) 601 / 580 and 634 / 586.
//
// With more views the chain of small kernels grows, and two sequences win by a
// few percent from about 3 million on, back to back; a caller that waits for each
// launch loses more by them until there is about three times as much to do.  The
// line serves launches that follow each other: over 200k triangles, 81 of 128 x
// 128 (5.3) 212 / 196 and 244 / 269; 100 of 100 x 80 (5.6) 206 / 191 and 238 /
// 268; 120 of 96 x 72 (6.6) 237 / 233 and 269 / 296; 128 of 64 x 64 (6.8) 212 /
// 199 and 246 / 272; but over 60k 128 of 64 x 64 (2.4) 135 / 139.
//
// Above 1024 views always two, right but for the smallest: over 20k triangles
// 1100 of 64 x 64 (9.7) 420 / 380 and 543 / 509, 2048 (18) 711 / 621 and 923 /
// 813, 2048 of 24 x 20 (11) 465 / 413 and 675 / 589; over 2k 2048 of 64 x 64
// (9.2) 394 / 343 and 604 / 549, 4096 of 64 x 64 (18) 710 / 606 and 1117 / 970;
// but 1100 of 64 x 64 (5) 236 / 242 and 359 / 390, 2048 of 24 x 20 (2) 248 / 316
// and 457 / 428, and 1025 of 24 x 20 (1) 119 / 190 and 210 / 243, which the direct
// path draws.
bool split_batch(const ViewReq *v, uint32_t n)
{
    constexpr uint64_t kSplitSize = 8192 * 1024, kSplitManySize = 3072 * 1024;
    constexpr uint32_t kSplitMany = 80, kSplitAlways = 1024;
    if (n < kSplitViews) return false;
    if (n > kSplitAlways) return true;
    uint64_t size = 0;
    for (uint32_t k = 0; k < n; ++k)
        size += (uint64_t)v[k].sensor.width * v[k].sensor.height + v[k].scene->T / 4;
    return size >= (n > kSplitMany ? kSplitManySize : kSplitSize);
}

hab_status render_split(hab_context *ctx, const ViewReq *v, uint32_t n, const PlanOpts &o, hipStream_t s,
                        hab_view_stats *stats)
{
    if (o.one_sequence || !split_batch(v, n)) return render_all(ctx, ctx->ws, v, n, o, s, stats);
    hab_status st = ensure_aux(ctx);
    if (st != HAB_OK) return st;
    // views 0, 2, 4, ... and 1, 3, 5, ...: halves of like composition
    PlanOpts oh = o;
    oh.half = true;
    std::vector<ViewReq> half[2];
    std::vector<hab_view_stats> hs[2];
    for (int h = 0; h < 2; ++h) {
        half[h].reserve((n + 1) / 2);
        if (stats) hs[h].resize((n + 1 - (uint32_t)h) / 2);
    }
    for (uint32_t k = 0; k < n; ++k) half[k & 1u].push_back(v[k]);
    HAB_HIP(hipEventRecord(ctx->fork_ev, s));
    HAB_HIP(hipStreamWaitEvent(ctx->aux, ctx->fork_ev, 0));
    st = render_all(ctx, ctx->ws, half[0].data(), (uint32_t)half[0].size(), oh, s,
                    stats ? hs[0].data() : nullptr);
    if (st == HAB_OK)
        st = render_all(ctx, ctx->ws2, half[1].data(), (uint32_t)half[1].size(), oh, ctx->aux,
                        stats ? hs[1].data() : nullptr);
    // the join is enqueued whatever happened, so that s is ordered after
    // everything the call put on the second stream
    HAB_HIP(hipEventRecord(ctx->join_ev, ctx->aux));
    HAB_HIP(hipStreamWaitEvent(s, ctx->join_ev, 0));
    if (st != HAB_OK) return st;
    if (stats)
        for (uint32_t k = 0; k < n; ++k) stats[k] = hs[k & 1u][k >> 1];
    return HAB_OK;
}

}  // namespace habmi

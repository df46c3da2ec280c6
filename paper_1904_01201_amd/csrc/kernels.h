// Launch interface between the host runtime and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dtypes.h"

namespace habmi {

constexpr uint32_t kMaxViews = 4096;   // views per launch sequence
constexpr uint32_t kSegPerTile = 4;    // a work item covers <= 4 * TS^2 list entries
// List entries of a work item of k_raster_wave, by the launch's 16-pixel tiles and
// triangles.  A wave takes about 7 us for 64 entries while it shares its SIMD with
// five others, more without, so the launch ends on waves with a whole item left;
// but each item of a tile with several merges 256 keys.  Items of 256 -> of 128:
// eight 512 x 384 views of 1M triangles rasterise in 108 -> 96 us, 32 and 64 views of
// 256 x 256 in 101 -> 90 and 170 -> 165, 256 mixed views (two launches of 57 k tiles)
// take 1112 -> 1123.  Items of 128 -> 64 -> 32, us a launch: one 512 x 512 view of 5k
// triangles 238 -> 227 -> 224, two of 20k (40k triangles) 152 -> 143 -> 143, 16 of 256 x
// 256 over 20k (320k) 147 -> 138 -> 138, eight over 60k (480k) 119 -> 108 -> 110, over
// 200k (1.6M) 114 -> 110 -> 120; but 16 of them (3.2M) 142 -> 147 -> 176.
constexpr uint32_t kWaveSeg = 128, kWaveSegLarge = 256, kWaveManyTiles = 32768;
constexpr uint32_t kWaveSegSmall[2] = {32, 64}, kWaveTriangles[2] = {300000, 2000000};   // up to
constexpr int kWaveWavesPerSimd = 6;    // its register budget
constexpr uint32_t kMaxSegments = 1u << 14;

// One raster + resolve launch pair: all views of a batch that use the same
// tile size.
struct RasterLaunch {
    int ts;                    // 8, 16 or 32
    const uint32_t *lview;     // [nl] view index (resolve: block -> view)
    const uint32_t *bpre;      // [nl] first resolve block of each view (32 x 2 * stack pixels each)
    uint32_t nl;
    uint32_t blocks;           // total tiles
    uint32_t bands;            // total resolve blocks (resolve grid)
    uint32_t stack;            // bands of 32 x 2 pixels a resolve block shades one after another
    uint32_t grid;             // persistent raster blocks
    bool wave;                 // 16-pixel tiles, a wave each (k_raster_wave)
    bool lane_owned;           // atomic-free lane-owned z-test (else balanced steps, z-keys in LDS)
    uint32_t item_cap;         // work items the scratch below can hold
    uint2 *items;              // [item_cap] (view, tile | segment << 18)
    uint2 *partial;            // [item_cap][TS*TS] per-pixel (1/w bits, key) of each item
};

// A descriptor block small enough (four views or so) to go to the device as an
// argument of the direct path's first kernel.
constexpr uint32_t kInlineDesc = 2048;
struct alignas(16) InlineDesc {
    uint8_t bytes[kInlineDesc];
};

// Device pointers and sizes of one launch sequence.
struct LaunchPlan {
    const DView *views;
    uint32_t nviews;
    uint32_t cull_blocks;      // cull blocks per view (256 clusters each, for the largest scene)
    uint32_t setup_grid;       // setup grid (waves stride over the visible cluster runs)
    uint32_t *pairs;           // visible clusters, one segment per view
    DViewCounters *ctr;
    uint32_t *skey;
    uint2 *sbox;
    uint32_t *tile_count;
    uint32_t *tile_off;
    uint32_t *tile_cursor;
    uint32_t ntiles;
    uint32_t *bins;
    uint32_t *tile_item;       // first work item of each tile
    DQueue *queue;
    uint2 *items[3];           // per tile size (null when unused)
    uint32_t *err;
    uint32_t bin_grid;
    uint32_t max_tiles;        // of a view
    bool coarse;               // triangles of many tiles (k_bin)
    uint32_t wave_seg;         // 16-pixel tiles go to k_raster_wave, this many entries an item, their
                               //   z-keys to zbuf (0: to k_raster)
    RasterLaunch raster[3];
    int nraster;
    // direct path (draw.hip): drawn without tile lists when `direct`
    bool direct;
    unsigned long long *zbuf;  // z-keys: of every view, [znum]; or of the 16-pixel tiles (wave16)
    uint64_t znum;
    ClusterRec *recs;          // visible clusters, kBuckets segments per view
    const uint32_t *tpre;      // [nl] first tile block of each view of the list
    uint32_t tile_edge;        // 16, 32 or 64
    uint32_t shares;           // blocks that share a tile's clusters (1: the block shades it)
    uint32_t tile_grid;        // tile blocks
    uint32_t desc_bytes;       // of the descriptor block, a multiple of 256
    const InlineDesc *desc;    // the descriptor block, if its first kernel writes it (else null: it was copied)
    hipEvent_t *prof;          // null, or kProfEvents events recorded around the kernels
    uint32_t prof_mask;        // phases whose start/stop events are recorded
};

constexpr int kPhaseResolve = 8;
constexpr int kProfPhases = 9;
constexpr int kProfEvents = 2 * kProfPhases;   // start/stop per phase

// Resident k_raster<ts, lane_owned> blocks per compute unit (sizes the
// persistent grid).
int raster_blocks_per_cu(int ts, bool lane_owned);

// Enqueue the whole sequence on stream s (launch_direct: a direct plan's).
hipError_t launch_render(const LaunchPlan &L, hipStream_t s);
hipError_t launch_direct(const LaunchPlan &L, hipStream_t s);

// A mesh as it was uploaded: positions [V][3], indices [T][3], colours [V][3]
// bytes or null, texture coordinates [V][2] or null (they win over colours).
struct MeshSource {
    const float *pos;
    const uint32_t *idx;
    const uint8_t *col;
    const float *uv;
};

// Sums on lines of their own (one for all: k_scene took 98 us for scenes of 460k triangles on average, 17 so).
struct SpreadSums {
    unsigned long long sum[32][16];
};

// Write a scene's triangles out on stream s: positions, attributes (the colours may
// overwrite the indices) and the bounding box of every kCluster consecutive ones.
// Adds to the sums, in units of 2^-24, the part of the box of edges `size` that each
// of these takes, every side grown by `grow`.
hipError_t launch_scene(const MeshSource &m, uint32_t T, float *tpos, uint32_t *attr, float4 *cbox, float3 size, float grow,
                        SpreadSums *spread, hipStream_t s);

// Compare recip_rn with the IEEE division 1/x for every float whose bits
// lie in [lo, hi) (lo < hi <= 0x7F800000), adding the number of differing
// results to *count (device memory, one 64-bit word), on stream s.
hipError_t launch_check_recip(uint32_t lo, uint32_t hi, unsigned long long *count, hipStream_t s);

}  // namespace habmi

// Internal layouts shared by the host side of the C ABI (sgn_api.cpp) and
// the HIP kernels (sgn_kernels.hip).  Not part of the public interface.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "sgn_rules.h"

namespace sgn {

constexpr int kMaxNbr = 16;
constexpr int kWaveSize = 64;
constexpr int kBlockThreads = 256;      // 4 wavefronts per workgroup
constexpr int kNumCounters = 16;        // work-queue heads (one per XCD + spares)
constexpr int kInitSurfels = 128;       // most surfels that a wavefront of the initialisation looks through

// Division of n < 2^24 by a divisor known on the host: m = ceil(2^(24 + l) / d)
// with 2^l >= d, so that (n m) >> (24 + l) is exact.  Two instructions and a
// shift; a plain 32-bit division is about thirty.
struct FastDiv {
    uint32_t m;
    int32_t l;
};
inline FastDiv fast_div(int d) {
    int l = 0;
    while ((1 << l) < d) ++l;
    return {(uint32_t)(((1ull << (24 + l)) + (uint64_t)d - 1) / (uint64_t)d), l};
}

// Per-keyframe descriptor in device memory (one per batch item).
struct KfDev {
    const void* kf_img;
    float* inv_depth;
    float* nx;
    float* ny;
    float* nz;
    uint32_t* flags;
    float* cost;
    uint32_t* nvalid;
    uint32_t* last_update;
    const uint8_t* is_new;        // may be null
    float* inv_depth_out;         // may be null
    int32_t* index_out;           // may be null
    int32_t width, height, kf_pitch, n_nbr;
    int32_t gw, gh, frame_base, item_base;      // frames: [frame_base, frame_base + n_nbr)
    int32_t groups_x, n_items;                  // anchor blocks per row; work items
    // first wavefront of the initialisation (init_run surfels each) and of
    // the render (64 blocks of 4 x 4 pixels each)
    int32_t init_wave, render_wave;
    FastDiv div_gw, div_bx;       // by gw; by the 4-pixel blocks of a row
    int32_t patch, nbr_pitch_b;                   // neighbour-image row pitch in bytes
    // what follows in one cache line, the entry in four (16 mixed disc
    // keyframes: 2.04 ms, 2.06 packed to 216 bytes)
    int32_t pad[10];
    float fx, fy, cx, cy;                        // intrinsics, rounded to float
    float kf_scale, img_scale;
    // disc surfels (Eq. 4): centres of the surfels, radius in pixels; null
    // and 0 for tiles
    const float* disc_ux;
    const float* disc_uy;
    float disc_r;
    int32_t disc_count;           // surfels of the keyframe (an item is a run of them)
};
static_assert(sizeof(KfDev) == 256 && offsetof(KfDev, fx) >= 192, "cache lines");

// Per-neighbour-frame constants of Eq. 6, in device memory or in a lone
// keyframe's kernel arguments.
struct FrameDev {
    float zrow[4];  // hm[6], hm[7], kt[2] rounded to float (the q_z row), pad
    const void* img;  // next to zrow: one scalar load per frame fetches both
    double hm[9];   // K R K^-1
    double kt[3];   // K t
};
// What FrameDev is formed from: the caller's pose and the keyframe's
// intrinsics (fx, fy, cx, cy).
struct FrameIn {
    const void* img;
    double K[4];
    double R[9];
    double t[3];
};
// K R K^-1 and K t (Eq. 6) in double, the q_z row rounded once to float.  A
// lone keyframe's frames are formed on the host and a batch's on the device:
// every operation is an IEEE one, and which product of a fused pair is
// rounded by itself is written out, so both give the same bits (an ulp here
// moves the last bits of a few warp constants, and with them the path of
// some weakly determined surfels).
__host__ __device__ inline void frame_constants(const FrameIn& in, FrameDev& F) {
#pragma clang fp contract(off)
    const double fx = in.K[0], fy = in.K[1], cx = in.K[2], cy = in.K[3];
    const double* R = in.R;
    // K R
    const double k[9] = {fma(fx, R[0], cx * R[6]), fma(fx, R[1], cx * R[7]), fma(fx, R[2], cx * R[8]),
                         fma(cy, R[6], fy * R[3]), fma(fy, R[4], cy * R[7]), fma(cy, R[8], fy * R[5]),
                         R[6],                     R[7],                     R[8]};
    for (int r = 0; r < 3; ++r) {
        // times K^-1 = [[1/fx, 0, -cx/fx], [0, 1/fy, -cy/fy], [0, 0, 1]]
        F.hm[3 * r + 0] = k[3 * r] / fx;
        F.hm[3 * r + 1] = k[3 * r + 1] / fy;
        F.hm[3 * r + 2] = k[3 * r + 2] - k[3 * r] * cx / fx - k[3 * r + 1] * cy / fy;
    }
    F.kt[0] = fma(fx, in.t[0], cx * in.t[2]);
    F.kt[1] = fma(cy, in.t[2], fy * in.t[1]);
    F.kt[2] = in.t[2];
    F.zrow[0] = (float)F.hm[6];
    F.zrow[1] = (float)F.hm[7];
    F.zrow[2] = (float)F.kt[2];
    F.zrow[3] = 0.f;
    F.img = in.img;
}

// Header of one batch: every per-call value of the kernels, in device memory
// for a batch, in the kernel arguments for a lone keyframe.
struct BatchHeader {
    KfDev* kfs;
    FrameDev* frames;
    int32_t n_kf, n_frames, total_items;
    int32_t init_waves, render_waves;   // of the batch
    int32_t init_run;                   // surfels per wavefront of the initialisation (a multiple of 64)
    int32_t iters;
    float huber_k;
    float kappa_fp64;
    int32_t depth_only;
    float beta_r;
    uint32_t stamp;
    int32_t n_queues;
    float lm_lambda;
    QueueDev queues[kNumCounters];
};

enum : uint32_t {
    F_DEGENERATE = 1u << 0,
    F_FEW_SAMPLES = 1u << 1,
    F_SOLVE_FAIL = 1u << 2,
    F_REJECTED = 1u << 3,
    F_FP64_SOLVE = 1u << 4,
    F_UNINIT = 1u << 5,
    F_GN_BITS = F_DEGENERATE | F_FEW_SAMPLES | F_SOLVE_FAIL | F_REJECTED | F_FP64_SOLVE,
};

// A lone keyframe's whole table, passed by value as the first kernel
// argument (kernels that need no frames take it up to kf): no upload, no
// staging slot.  hdr.kfs and hdr.frames are not used.  Kernel arguments hold
// 4 KB.
struct LoneKf {
    BatchHeader hdr;
    KfDev kf;
};
struct LoneBatch {
    LoneKf one;
    FrameDev frames[kMaxNbr];
};
static_assert(sizeof(LoneBatch) <= 3072, "kernel arguments of a lone keyframe");

// Kernel variants.
struct GnVariant {
    int dtype;      // 0 f32, 1 f16, 2 u8
    int patch;      // 4, 8 or 16
    int tiles_x, tiles_y;
    int lds;        // stage footprints in LDS
    int groups;     // surfel groups per work item (1, 2 or 4)
    int by_row;     // neighbour rows read by index (rows_by_index)
    int deep;       // frames whose taps are in flight at once (0: one sample at a time)
    int split;      // lanes per pixel column of the 4x4 layout (1, 2 or 4)
    int persistent; // a grid of fixed size pulling items from device queues
    int shared;     // a workgroup's wavefronts share their surfels' solves
    int damped;     // Levenberg-Marquardt (read by the split forms)
};
// Row pitch (bytes) up to which neighbour images are read through a
// structured buffer, the row as the index: the descriptor's stride field holds
// 14 bits.  Wider rows are read with raw byte offsets.
constexpr unsigned kMaxRowStride = 16384;

// Work-item geometry of the Gauss-Newton kernel.  Surfels are taken in
// aligned anchor blocks of 16 x 16 pixels (ab x ab tiles).  A work item is an
// ix x iy tile sub-block of one anchor block holding K groups of tx x ty
// tiles (one group fills a wavefront: four or eight 4 x 4 surfels, one 8 x 8
// or one 16 x 16 surfel), arranged gx x gy, as wide as the anchor block
// allows; ipb items tile an anchor block.
struct ItemGeo {
    int ab, gx, gy, ix, iy, ipb;
};
constexpr ItemGeo item_geo(int S, int TX, int TY, int K) {
    const int ab = 16 / S;
    const int gx = (S == 4) ? (K < 4 / TX ? K : 4 / TX) : (K >= 2 ? 2 : 1);
    const int gy = K / gx;
    const int ix = gx * TX, iy = gy * TY;
    return ItemGeo{ab, gx, gy, ix, iy, (ab / ix) * (ab / iy)};
}

// Arguments of the re-gridding kernels (Eq. 10).  Surfel arrays are device
// memory; best/win are scratch of one entry per destination tile.
struct RegridSurfels {
    float* inv_depth;
    float* nx;
    float* ny;
    float* nz;
    uint32_t* flags;
    float* cost;
    uint32_t* nvalid;
    uint32_t* last_update;
};
struct RegridArgs {
    RegridSurfels src, dst;
    double src_K[4], dst_K[4];   // fx, fy, cx, cy
    double R[9], t[3];           // X_dst = R X_src + t
    int32_t src_gw, src_shift, dst_gw, dst_gh, dst_shift;    // grids; log2 of the tile edges
    FastDiv div_src, div_dst;      // by src_gw and dst_gw
    unsigned long long* best;    // closest landing per destination tile (bits of 1/p'_z)
    int32_t* win;                // winning source index per destination tile
    uint8_t* is_new;
    int32_t* src_index;          // may be null
    int32_t dst_base;              // destination tiles of the table's earlier pairs (best, win offsets)
    int32_t src_count, dst_count;  // this pair's source surfels / destination tiles
    int32_t src_wave, dst_wave;    // this pair's first 64-lane wavefront over sources / tiles
};

// Launchers implemented in sgn_kernels.hip.  All return hipError_t of the
// launch.  `one` (host memory) or `hdr` (device memory) gives the table: hdr
// null means the lone keyframe of `one`, whose contents are copied into the
// launch.
//
// Table upload: n16 16-byte words from pinned host memory to the device
// table, the constants of n_frames frames formed from `in` (pinned host
// memory), and the work-queue counters cleared.
hipError_t launch_stage(const void* host, void* dev, int n16, const FrameIn* in, FrameDev* frames, int n_frames,
                        uint32_t* counters, hipStream_t s);
hipError_t launch_init(const LoneKf& one, const BatchHeader* hdr, int waves, hipStream_t s);
hipError_t launch_render(const LoneKf& one, const BatchHeader* hdr, int waves, hipStream_t s);
// The two events are recorded on the stream before and after the kernel.
hipError_t launch_gn(const GnVariant& v, const LoneBatch& one, const BatchHeader* hdr, uint32_t* counters,
                     int grid_blocks, hipStream_t s, hipEvent_t start, hipEvent_t stop);
// Device address of the static scratch array on `device` (which must be the
// current device), looked up on the first call for that device and kept.
hipError_t static_scratch_on(int device, void** out);
// Re-gridding of n_pairs keyframe pairs: a device table, or (table null) the
// one entry `one`.  A wavefront
// never spans two pairs: pair k's sources run over the
// wavefronts from src_wave on (surfel i at lane i % 64 of wavefront
// src_wave + i / 64), likewise its tiles from dst_wave; src_waves and
// dst_waves are the totals.
// The first launch also copies the table (table_bytes from pinned host memory;
// 0 for one pair) and clears the scratch of n_tiles destination tiles (best
// and win, both padded to 16 bytes); `uploaded` (or null) is recorded after it.
hipError_t launch_regrid(const RegridArgs& one, const void* host, RegridArgs* table, size_t table_bytes,
                         int n_pairs, int src_waves, int dst_waves, void* best, void* win, int n_tiles,
                         hipStream_t s, hipEvent_t uploaded);

// Disc surfels (Eq. 4).
constexpr float kDiscMaxRadius = 12.f;
// Disc surfels per wavefront of the Gauss-Newton kernel, by image type
// (0 f32, 1 f16, 2 u8): two (32 lanes each) where a pixel's LDS slot packs
// into one word, one for f32 images.
constexpr int disc_surfels_per_wave(int dtype) { return dtype == 0 ? 1 : 2; }
// Gauss-Newton over the disc surfels of a batch: work items of
// disc_surfels_per_wave(dtype) surfels of one keyframe (KfDev::n_items =
// ceil(disc_count / that), item_base their prefix).
// grid_blocks workgroups of four items of one wavefront or of one item of
// several (with one share per XCD in the header, workgroup b serves share
// b % kXcds)
hipError_t launch_disc_gn(int dtype, const DiscForm& form, const LoneBatch& one, const BatchHeader* hdr,
                          int total_items, int grid_blocks, bool by_row, float max_radius, int max_nbr, hipStream_t s,
                          hipEvent_t start, hipEvent_t stop);
// Depth-buffered render of the discs of several keyframes: one table entry
// per keyframe (device memory; null for one keyframe, `one`).
struct DiscRenderItem {
    const float* inv_depth;
    const float* nx;
    const float* ny;
    const float* nz;
    const uint32_t* flags;
    const float* ux;
    const float* uy;
    float* inv_depth_out;         // [width * height]
    int32_t* index_out;           // [width * height] or null
    int32_t count, width, height, surfel_base;
    float radius;
    int32_t tiles_x;              // render tiles per row (kRenderTile pixels square)
    double fx, fy, cx, cy;
    int32_t tile_base;            // render tiles of the table's earlier keyframes
    int32_t pad;
};
constexpr int kRenderTile = 16;
// Per usable surfel: centre, normal and the denominator of Eq. 3, in double.
struct DiscRaster {
    double cx, cy, n0, n1, n2, den;
};
// The render's scratch: raster records [surfels], tile counts [tiles] and
// after them the list's cursor, list starts [tiles], tile lists
// [kDiscMaxTilesPerSurfel * surfels].
constexpr int kDiscMaxTilesPerSurfel = 9;     // a box of <= 2 r + 1 <= 25 pixels meets <= 3 x 3 tiles
struct DiscRenderScratch {
    DiscRaster* rec;
    int32_t* count;
    int32_t* start;
    int32_t* list;
};
// px: pixels per lane of the raster (raster_pixels).
hipError_t launch_disc_render(const DiscRenderItem& one, const DiscRenderItem* table, int n_items, int total_surfels,
                              int total_tiles, bool bin_lds, int px, const DiscRenderScratch& w, hipStream_t s);
// The search for empty areas on the lattice (spacing/2 + i spacing, ...),
// placement of the qualifying candidates as surfels first .. and their
// neighbour initialisation from the index map.
struct DiscPlaceArgs {
    float* inv_depth;
    float* nx;
    float* ny;
    float* nz;
    uint32_t* flags;
    float* cost;
    uint32_t* nvalid;
    uint32_t* last_update;
    float* ux;
    float* uy;
    const int32_t* index_map;     // [width * height]
    int32_t first, room;          // existing surfels; free entries after them
    int32_t width, height, spacing, cand_x, cand_y;   // lattice of cand_x x cand_y candidates
    float radius, alpha, beta;
    float fx, fy, cx, cy;
    uint8_t* cand_flag;           // scratch [cand_x * cand_y]
    int32_t* counts;              // device [2]: placed, qualifying
    int32_t cand_base;            // candidates of the table's earlier keyframes
    int32_t init_base;            // new-surfel slots (min(room, candidates)) of earlier keyframes
};
// Placement for n_items keyframes: search (one wavefront per candidate),
// compaction (one workgroup per keyframe), initialisation (one wavefront per
// new-surfel slot; small: no window of theirs has more than two pixels per lane).
// table (device) may be null up to kDiscPlaceArgs keyframes.
constexpr int kDiscPlaceArgs = 16;
hipError_t launch_disc_place(const DiscPlaceArgs* items, const DiscPlaceArgs* table, int n_items,
                             int total_cands, int total_init, bool small, hipStream_t s);
// Eq. 10 for disc surfels: each usable source surfel moves to p' = R p + t,
// n' = R n, and is re-centred at K_dst pi(p'); those landing in the
// destination image are written in source order.
struct DiscTransferArgs {
    const float* inv_depth;
    const float* nx;
    const float* ny;
    const float* nz;
    const uint32_t* flags;
    const uint32_t* last_update;
    const float* ux;
    const float* uy;
    int32_t count, dst_w, dst_h, capacity;
    double sK[4], dK[4];          // fx, fy, cx, cy of source and destination
    double R[9], t[3];            // X_dst = R X_src + t
    RegridSurfels dst;
    float* dux;
    float* duy;
    int32_t* src_index;           // may be null
    int32_t* counts;              // device [2]: written, landed
};
// One workgroup per keyframe pair; table (device) may be null up to
// kDiscXferArgs pairs.
constexpr int kDiscXferArgs = 11;
hipError_t launch_disc_transfer(const DiscTransferArgs* pairs, const DiscTransferArgs* table, int n_pairs,
                                hipStream_t s);
hipError_t launch_quantize(const float* src, int src_pitch, void* dst, int dst_pitch,
                           int width, int height, int dtype, float scale, hipStream_t s);
bool gn_variant_supported(const GnVariant& v);

}  // namespace sgn

// Rules of the host side that need neither the device nor the runtime (plain
// C++, so that tests compile them by themselves).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sgn {

constexpr int kXcds = 8;

// One past the last byte, from an image's first, that the taps of a sample can
// touch when rows are read by index: corners reach x0 = width - 2 and the
// second row is the last.  Float taps are the pair itself; halves and bytes
// come as eight bytes from the aligned dword below the pair, which at the
// row's end is up to four bytes more than the row's last dword.
inline size_t tap_reach(int width, int height, size_t pitch_b, int elem_bytes) {
    const size_t col = (size_t)(width - 2) * elem_bytes;
    return (size_t)(height - 1) * pitch_b + (elem_bytes == 4 ? col : col & ~size_t(3)) + 8;
}
// One past the image's last dword (the size that loads by byte offset are
// checked against).
constexpr size_t image_end(int width, int height, size_t pitch_b, int elem_bytes) {
    return (size_t)(height - 1) * pitch_b + (((size_t)width * elem_bytes + 3) & ~size_t(3));
}

// Whether an image's rows may be read by index.  Those loads check the row
// only, so where taps reach past the image the bytes there have to be mapped:
// they are in the page of the image's last byte, or the next image starts
// there (next: its address, or 0), or the memory's owner says so
// (mapped_end(address of the last byte): one past the last mapped byte).
// Otherwise the rows are read by byte offset, which the hardware checks
// against the image's size.
template <class MappedEnd>
bool rows_by_index_safe(uintptr_t data, int width, int height, size_t pitch_b, int elem_bytes, uintptr_t next,
                        MappedEnd&& mapped_end) {
    constexpr uintptr_t kPage = 4096;              // the smallest page
    const uintptr_t end = data + image_end(width, height, pitch_b, elem_bytes);
    const uintptr_t reach = data + tap_reach(width, height, pitch_b, elem_bytes);
    if (reach <= end || end % kPage != 0 || next == end) return true;
    return reach <= mapped_end(end - 1);
}

// Tiles to either side of its own that a new surfel's initialisation looks at.
inline int init_reach(float beta_r, int patch) {
    const float br = beta_r > 0.f ? beta_r : (float)patch;
    return (int)std::min((br + 0.5f * (float)(patch - 1)) / (float)patch, 1e6f);
}

// Work queue (or run) q covers the global item range [begin, end).
struct QueueDev {
    int32_t begin, end;
};

// Cuts the items of the table's keyframes (in share_order) into nq runs of
// equal work, one per XCD: a run reads one part of the images through one
// L2, and no XCD waits for another.  An item's work is its neighbour frames
// plus what does not depend on them (about `fixed` frames' worth).  Whole
// keyframes per XCD keep the same locality but leave XCDs idle where few or
// unequal keyframes do not divide by eight: the Gauss-Newton of 16 mixed
// disc keyframes took 2.95 ms so, the heaviest share holding 1.5 times the
// mean, and 1.82-1.97 ms cut.  (Ordered by neighbour count alone, so that each
// XCD has items of one length, the 64-keyframe tile batch took 8 % longer:
// an error of the work estimate then adds up over a whole XCD.)
template <class Kf>
void cut_shares(int nq, const Kf* kfs, int n, double fixed, QueueDev* queues) {
    double total = 0.0;
    for (int i = 0; i < n; ++i) total += (double)kfs[i].n_items * (kfs[i].n_nbr + fixed);
    int k = 0, end = 0;
    double before = 0.0;                       // work of the keyframes before k
    for (int q = 0; q < nq; ++q) {
        queues[q].begin = end;
        const double want = total * (q + 1) / nq;
        while (k < n && before + (double)kfs[k].n_items * (kfs[k].n_nbr + fixed) <= want) {
            before += (double)kfs[k].n_items * (kfs[k].n_nbr + fixed);
            ++k;
        }
        const int last = n > 0 ? kfs[n - 1].item_base + kfs[n - 1].n_items : 0;
        int at = k < n ? kfs[k].item_base + (int)((want - before) / (kfs[k].n_nbr + fixed)) : last;
        if (q == nq - 1) at = last;
        end = std::min(last, std::max(end, at));
        queues[q].end = end;
    }
}

// Workgroups of a one-wavefront-per-item grid: workgroup b serves share
// b % kXcds, so with shares the grid covers the largest one kXcds times.
inline int item_blocks(int nq, const QueueDev* queues, int items, int wpb) {
    if (nq != kXcds) return std::max(1, (items + wpb - 1) / wpb);
    int widest = 1;
    for (int q = 0; q < kXcds; ++q) widest = std::max(widest, (queues[q].end - queues[q].begin + wpb - 1) / wpb);
    return kXcds * widest;
}

// How the disc kernel runs: wavefronts per item (1, 4, 8 or 16) and frames
// whose taps are in flight at once (4 with several wavefronts, else 0, 2 or
// 4), and whether a workgroup's wavefronts share their surfels' solves.
// Results do not depend on it.
struct DiscForm {
    int waves, deep, shared;
};

// The disc kernel's form for a batch of w work items per SIMD whose discs take
// `slots` pixel slots each (32 pixels; f32 64), as several wavefronts deal the
// slots out: without enough slots they only wait for each other.  Times: 15
// iterations, 6 neighbours, radius 10 (ten slots, f32 five), f16 with two
// discs per item unless f32 is said, with one.
//   one slot   one wavefront, four frames in flight: radius 2.5 at w = 1 58 us
//              against 63 with four wavefronts, at 1.5 60 against 106.
//   w <= 0.25  sixteen wavefronts per item, one workgroup per CU: 79 us at
//              187 items against 97 with eight and 316 with one.  (Two slots
//              or four: as with four wavefronts, within 1 us.)
//   w <= 0.45  eight: 107 us at 424 items (sixteen 152, four 131).
//   w <= 1     four, all resident: 142 us at 755 items (eight 201, one with
//              four frames in flight 271); two slots at w = 1 69 against 81,
//              four 79 against 125; f32 96 against 149 at 848.
//   w <= 1.7, four slots and more, not f32
//              four in two rounds: 266 us against 290 at 1,716 items; four
//              slots at w = 1.5 129 against 132, but two 109 against 84; f32
//              170 against 158 at 1,510.
//   w <= 2.2, f32 4
//              one, four frames in flight (four wavefronts per SIMD): 320 us
//              at 2,267 items (one sample at a time 363); f32 198 at 3,020
//              (shared 203).
//   beyond     one, the workgroup's solves shared, two frames in flight at six
//              per SIMD.  Whole calls: 360 us at 3,020 items (four frames
//              unshared 375), 465 against 511 at 4,530, 548 / 597 at 6,040,
//              982 / 1,088 at 12,080; f32 296 / 328 at 6,040, 512 / 607 at
//              12,080, 1,810 / 2,001 at 48,320.
// The damped variant's cost sums run over the slots in turn: one wavefront,
// its solves its own.  Four frames in flight to w = 4 (703 us against 718 with
// two and 737 with one sample at a time at w = 3.5), two to 5 (828 / 833, four
// 1,065, at 4.5), one sample to 6 (all resident; 1,047, two 1,177, at 5.5),
// four again to 8 (two full rounds: 648 us at 6,800 items against 753),
// beyond that one sample (f32 two frames: 1,062 against 1,137 at 14).
inline DiscForm disc_form(double w, double slots, bool f32, bool damped) {
    if (!damped) {
        const bool deal = slots > 1.0;
        if (deal && w <= 0.25) return {16, 4, 0};
        if (deal && w <= 0.45) return {8, 4, 0};
        if (deal && w <= (f32 || slots < 4.0 ? 1.0 : 1.7)) return {4, 4, 0};
        if (w <= (f32 ? 4.0 : 2.2)) return {1, 4, 0};
        return {1, 2, 1};
    }
    if (w <= 4.0) return {1, 4, 0};
    if (w <= 5.0) return {1, 2, 0};
    if (w <= 6.0) return {1, 0, 0};
    if (w <= 8.0) return {1, 4, 0};
    return {1, f32 ? 2 : 0, 0};
}

// Damped four-pixels-per-lane batches of w > 3 items per SIMD: one frame's taps
// in flight, five wavefronts per SIMD, or one sample at a time, seven (whole
// calls, one frame / one sample, us).  A keyframe has `pixels` pixels, `frames`
// neighbours and `bytes` of images.
//   w <= 5     one frame, all resident: 291 / 303 (320x240 f16, six neighbours, w
//              = 3.2); small keyframes of many neighbours to 4.1 only: 704 / 676
//              f16, 642 / 615 f32 (320x240, twelve, w = 4.7).
//   w <= 7     one sample, all resident at seven only, for 16 x 16 surfels (270 /
//              251 f16, 261 / 237 f32, 640x480, w = 5.9) and small keyframes (421
//              / 390 f16, 399 / 354 f32, 320x240); else to w = 6.2 where L2 holds
//              much of the images: 315 / 303 u8, but 551 / 622 f16 with twelve
//              neighbours (8 MB), 293 / 379 f32 (640x480, w = 5.9); 388 / 428 f16
//              (480x360, nine, w = 6.7).
//   w <= 9     one frame: one sample's second round is nearly empty: 562 / 578 and,
//              twelve neighbours, 1,172 / 1,266 (320x240 f16, w = 8.2), 397 / 413
//              (640x480); 16 x 16 ones 436 / 454 f32 (320x240, twelve, w = 8.8).
//   beyond     one frame to w = 24, and further where taps come from far (4x4
//              surfels 2,541 / 3,178 f16 of 24 MB, 1,346 / 1,770 f32 of 26 MB, w =
//              28); one sample for small images: 4x4 surfels of few neighbours
//              988 / 936 f16, 912 / 873 f32 (320x240, six, w = 16; twelve equal,
//              400x304, nine, 899 / 925), 16 x 16 ones 847 / 793 f16 (320x240), 438 /
//              415 u8 (480x360), but 795 / 826 f32 of 4.9 MB (400x304).
inline bool damped_one_frame(double w, int patch, double pixels, double bytes, double frames, bool far_taps) {
    const bool tiny = pixels < 100e3;
    if (w <= (patch == 4 && tiny && frames >= 8.0 ? 4.1 : 5.0)) return true;
    if (w <= 7.0 && (patch == 16 || tiny)) return false;
    if (w <= 6.2 && bytes < 4.5e6) return false;
    if (w <= 9.0) return true;
    const bool near = patch == 16 ? tiny || (pixels < 250e3 && bytes < 2.4e6)
                                  : pixels < 150e3 && bytes < 2.2e6 && frames < 8.0;
    return !near && (w <= 24.0 || far_taps);
}

// Whether the disc render bins each keyframe in one workgroup's LDS: its tile
// counts have to fit, and the largest keyframe's surfels, which one CU then
// works through, must not take longer than the launches that are saved.  Few
// keyframes leave the other CUs idle; many share the device either way, and
// spare the atomics in memory.  Whole renders, LDS / memory: 1 keyframe of
// 1,564 discs 17 / 23 us, 2,304 24 / 25, 3,072 25 / 29 (640x480), 3,108 28 /
// 26 (1920x1080), 4,641 29 / 26, 15,252 108 / 40; 8 keyframes of 4,641
// 64 / 63, of 10,549 124 / 105; 12 of 4,641 79 / 80; 16 of 3,600 96 / 94, of
// 4,641 94 / 98, of 6,279 108 / 125, of 8,040 208 / 186; 64 of 4,641 276 / 306.
constexpr int kBinTiles = 15360;
constexpr int kBinSurfels = 6400;
inline bool bin_in_lds(int keyframes, int64_t most_tiles, int64_t most_surfels) {
    return most_tiles <= kBinTiles && most_surfels <= (keyframes >= 12 ? kBinSurfels : 3072);
}

// Pixels per lane of the disc raster's wavefronts, for render tiles of 16 x 16
// whose lists hold `mean` surfels by their discs' boxes.  Four, a wavefront per
// tile, unless there are so few tiles that each SIMD has one wavefront or two
// and each of those a long list to walk: then one, four wavefronts per tile.
// Whole renders, one pixel per lane / four: 640x480 (1,200 tiles) 1,536 discs
// of radius 12 (8 per list) 18.5 / 21.1 us, 12,288 (64) 67 / 80, 24,576 (128)
// 114 / 133; two such keyframes (2,400) 25.4 / 26.1, 87 / 96, 152 / 157;
// 1280x720 (3,600) 31.8 / 31.2, 105 / 102, 192 / 182.  With shorter lists both
// are within about 2 us of each other either way.
inline int raster_pixels(int64_t tiles, double mean, int cus) {
    return mean >= 8.0 && tiles <= 5 * (int64_t)cus ? 1 : 4;
}
// Render tiles that a disc's box meets, on average over where its centre lies.
inline double mean_tiles(double radius, int tile) {
    const double m = 1.0 + 2.0 * radius / tile;
    return m * m;
}

}  // namespace sgn

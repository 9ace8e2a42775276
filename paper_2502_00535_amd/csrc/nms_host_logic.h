// Index arithmetic, sort keys and workspace layout of the NMS library: plain functions with no
// device-only construct in them, shared by the kernels and the launch code and compilable by a
// host compiler alone (the host tests sweep them without a GPU).
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include "nms_pair.h"  // NMS_HD

// ---- rank keys ----------------------------------------------------------------------------
// Unique ascending 64-bit key of (score, index): a better score sorts first, equal scores by
// lower index; -0.0 ties with +0.0.  Valid for every float but NaN (negative scores, denormals
// and both infinities order as the numbers they are).
NMS_HD unsigned long long nms_rank_key(float score, unsigned idx)
{
    unsigned u;
    memcpy(&u, &score, sizeof u);
    if (u == 0x80000000u) u = 0u;
    const unsigned asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending in the score
    return ((unsigned long long)(~asc) << 32) | idx;
}

// ---- work units of the map step -------------------------------------------------------------
// One unit = one column tile tc (64 outranking boxes) against a "super-row" of kSuper
// consecutive victim tile rows, i.e. up to kSuper tiles of the ranked lower triangle.
// Super-row sr has min(kSuper*(sr+1), T) units (tc = 0 .. last tile row of the super-row), so
// the units before super-row sr number kSuper * sr*(sr+1)/2.

// Number of units for T tile rows.
NMS_HD int nms_triangle_units(int T, int super)
{
    const int SR = (T + super - 1) / super;
    return SR == 0 ? 0 : super * (SR - 1) * SR / 2 + T;
}

// Linear unit index g -> (sr, tc): the largest sr with kSuper*sr*(sr+1)/2 <= g, by a float
// square root and a correction in exact integer arithmetic.
template <int kSuper>
NMS_HD void nms_triangle_unit(int g, int &sr, int &tc)
{
    int r = (int)((sqrtf(1.0f + (8.0f / kSuper) * (float)g) - 1.0f) * 0.5f);
    while ((long long)kSuper * r * (r + 1) / 2 > g) --r;
    while ((long long)kSuper * (r + 1) * (r + 2) / 2 <= g) ++r;
    sr = r;
    tc = g - kSuper * r * (r + 1) / 2;
}

// ---- workspace of the whole-path calls --------------------------------------------------------
NMS_HD size_t nms_align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Byte offsets of the parts of the workspace (every part 256-byte aligned), for frames of at most
// n_max boxes, n_pad = n_max rounded up to a multiple of 64.  `end` is the size.
struct NmsRunLayout {
    size_t order;    // int32 [frames][n_max]          rank -> input index
    size_t sorted5;  // float [frames][5 * n_pad]      box table: rows (x1,y1,x2,y2), then areas
    size_t ysc;      // float4 [frames][n_pad]         boxes with y * 2^-14, rank order
    size_t ytile;    // uint32 [frames][n_pad / 64]    1 = every box of the tile may use the y-scaled form
    size_t tsc;      // float [frames][n_pad]          per box, 2^-14 x the float32 its intersections are compared with
    size_t keys;     // uint64 [frames][n_pad]         chunk-sorted keys, only when n_max > sort_chunk
    size_t stage;    // uint64 [frames][n_pad / 64][32] eliminated-victim masks of the two-launch route, only when n_max > sort_chunk
    size_t end;
};

NMS_HD NmsRunLayout nms_run_layout(int n_max, int n_pad, int frames, int sort_chunk)
{
    NmsRunLayout l;
    size_t p = 0;
    l.order = p;
    p += nms_align256((size_t)frames * (size_t)n_max * sizeof(int32_t));
    l.sorted5 = p;
    p += nms_align256((size_t)frames * 5 * (size_t)n_pad * sizeof(float));
    l.ysc = p;
    p += nms_align256((size_t)frames * (size_t)n_pad * 4 * sizeof(float));
    l.ytile = p;
    p += nms_align256((size_t)frames * (size_t)(n_pad / 64) * sizeof(uint32_t));
    l.tsc = p;
    p += nms_align256((size_t)frames * (size_t)n_pad * sizeof(float));
    l.keys = p;
    if (n_max > sort_chunk) p += nms_align256((size_t)frames * (size_t)n_pad * sizeof(unsigned long long));
    l.stage = p;
    if (n_max > sort_chunk) p += nms_align256((size_t)frames * (size_t)(n_pad / 64) * 32 * sizeof(unsigned long long));
    l.end = p;
    return l;
}

// ---- rank step ----------------------------------------------------------------------------------
// Ranks by counting (n compares per box over the whole chip) instead of a sort of one workgroup per
// frame, whose time hardly depends on the number of frames.  Measured, the rank step alone, counted
// against sorted, us: 1 x 4096 4.8 / 16.2, 4 x 4096 8.3 / 16.4, 8 x 4096 12.2 / 16.5, 10 x 4096 16.8 / 16.6; 8 x 3000 9.6 / 14.0,
// 14 x 3000 13.2 / 14.1; 16 x 2048 7.9 / 10.5, 24 x 2048 10.4 / 10.5; 32 x 1000 5.6 / 8.1, 64 x 1000 9.0 / 8.2; 64 x 500
// 4.5 / 6.8, 120 x 500 6.8 / 6.8; 128 x 256 3.7 / 6.2; 512 x 64 3.0 / 6.6: the line is a number of boxes.
NMS_HD bool nms_use_count_rank(int n_max, int frames, int sort_chunk)
{
    return n_max <= sort_chunk && (long long)frames * n_max <= 32768;
}

// Elements per workgroup there.  Every workgroup stages its whole frame, so sixteen only pay while that
// puts one workgroup, or two of longer frames, on a compute unit that sixty-four would leave idle.  16 against 64
// elements, us: 1 x 4096 4.8 / 7.8, 2 x 4096 6.5 / 8.0, 3 x 4096 8.7 / 8.1; 3 x 2500 5.1 / 5.9, 4 x 2500 6.7 / 6.0; 6 x 1300 4.2 / 4.4,
// 7 x 1300 5.3 / 4.4; 4 x 1000 3.3 / 3.7, 5 x 1000 3.9 / 3.8, 16 x 1000 6.2 / 4.1; 8 x 500 3.1 / 3.2, 10 x 500 3.4 / 3.2; 1 x 360 2.8 / 2.8,
// 17 x 360 3.3 / 3.0; 64 x 64 2.9 / 2.4.
NMS_HD int nms_count_rank_elements(int n_max, int frames)
{
    return n_max > 384 && (long long)frames * n_max <= (n_max > 1024 ? 8192 : 4096) ? 16 : 64;
}

// ---- greedy rule, small frames -----------------------------------------------------------------------
// Frames of at most this many boxes are settled by one workgroup in one launch (greedy_small_kernel) instead of rank, mask and
// sweep.  Whole call, us, one launch / three: 30 x 70 6.7 / 11.6 (IoU 7.0 / 14.1, with labels 9.6 / 16.5), 1 x 128 7.3 / 12.3, 200 x 128 7.9 / 12.5,
// 50 x 160 8.8 / 12.2, 400 x 70 7.6 / 15.0; with a fourth tile 20 x 200 11.4 / 12.3, 100 x 256 12.8 / 13.1, 8000 x 250 263 / 243.
constexpr int kGreedySmallBoxes = 192;

// ---- greedy rule with labels ----------------------------------------------------------------------
// Large batches under the greedy rule with labels (greedy_classes_kernel; a batch there holds at least
// 131,072 boxes).  The figures: IoU, whole call, scenes where much / little is eliminated, in us.
//
// The largest bin of labels that one wavefront settles, in a frame of n_f boxes; a frame with a larger
// one is walked by the whole workgroup.  A bin is a chain that grows with the square of its rows, the walk
// shares the frame out: the line is a share of the frame.  Class by class against walked: 128 x 3000 in bins
// of 1000 502 / 1045 against 207 / 527, of 600 221 / 300 against 280 / 545; 263 x 500 in bins of 250 51 / 90 against
// 46 / 72, of 167 40 / 56 against 51 / 72; 300 x 1024 in bins of 512 128 / 244 against 72 / 183, of 341 90 / 138
// against 88 / 184.  Frames of three tiles or fewer are walked whatever their labels (2048 x 64, 20 labels 51 / 51
// against 25 / 24; 683 x 192 28 / 28 against 32 / 27).
NMS_HD int nms_class_bin_limit(int n_f)
{
    if (n_f <= 192) return 0;
    if (n_f <= 1024) return 7 * n_f / 16;
    return n_f / 4 > 448 ? n_f / 4 : 448;
}

// Wavefronts per workgroup: enough to walk a frame quickly, few enough that the wavefronts without a bin
// do not hold the places of other frames' when there are more frames than fit at once.  4 / 8 / 16 wavefronts, one
// label: 512 x 640 52, 44, 68; 2048 x 64 26, 30, 47; three labels: 300 x 1024 89 / 139, 90 / 138, 93 / 138; 1024 x 500
// 57 / 83, 71 / 98, 75 / 105; twenty: 128 x 1024 40 / 38, 34 / 32, 31 / 30.
NMS_HD int nms_class_waves(int n_max, int frames)
{
    if (n_max > 1024) return 16;
    return frames <= 768 ? 8 : 4;
}

// ---- which kernels a whole-path call runs ------------------------------------------------------
// All routes return the same keep vector (the paper's rule, section "Algorithm Correctness");
// they differ in what they launch.  Values of nms_route() and nms_route_at() in the C ABI.
constexpr int kNmsRouteDirect = 0;     // one launch, full n x n pair set with the score test inside (no rank step)
constexpr int kNmsRouteAllPairs = 1;   // rank, then every pair of the ranked triangle
constexpr int kNmsRouteTwoLaunch = 2;  // rank, every victim against the best 2048 ranks, then the live victims only
constexpr int kNmsRouteEarlyExit = 3;  // rank, then stages that drop a victim once it has an eliminator
constexpr int kNmsRouteSmallFrames = 4;  // frames of at most 1024 boxes, or a few of up to 4096: two such stages in one launch, no sort
constexpr int kNmsRoutePlaceFrames = 5;  // boxes in order of place, one launch
constexpr int kNmsRoutePlaceTable = 6;   // the same for frames beyond sort_chunk boxes: a table launch and a scan launch

// Frames small enough that launch latency, not arithmetic, decides: one launch of the
// direct form instead of rank + map.  (Twice the pairs and two more compares per pair:
// about 2.5x the VALU work of the ranked triangle.)
// The crossover in GPU time sits near 2^25 pair slots per batch and moves with the frame size,
// because the rank step it saves does (15 us at 1024 boxes, 23 us at 4096): measured 24 to 32
// frames of 1024 boxes, 8 to 12 of 2048, 3 to 4 of 4096.
NMS_HD bool nms_use_direct_form(int n_max, int frames)
{
    const long long slots = (long long)frames * n_max * n_max;
    const long long limit = n_max > 2048 ? (3ll << 24) : (n_max > 512 && n_max <= 1024 ? (3ll << 23) : (1ll << 25));
    return n_max <= 4096 && slots <= limit;
}

// Frames beyond sort_chunk boxes, a few of them (2^27 to 2^31 pair slots: one frame of 16,384
// boxes, four of them, eight of 8192): two launches with the decided victims dropped in between.
// Measured on dense crowd scenes, whole call: 1 x 16,384 38 us (all pairs 50), 4 x 16,384 82 us
// (all pairs 143, the early-exit kernels 98), 1 x 32,400 94 us (137 / 108); from 2^31 slots on
// the early-exit kernels are quicker (16 x 16,384: 200 us against 262).  Thresholds with a division-free form
// take the boxes in order of place instead (1 x 16,384 20 us, 16 x 16,384 42): the rule, like the early-exit
// rule below, is that of the others.
NMS_HD bool nms_use_two_launches(int n_max, int frames, int sort_chunk)
{
    const long long slots = (long long)frames * n_max * n_max;
    return n_max > sort_chunk && slots >= (1ll << 27) && slots < (1ll << 31);
}

// Large batches of frames of a thousand boxes or more: the route that stops testing a victim
// once it has an eliminator returns the same keep vector 1.3 to 3.3 times sooner on clustered
// detections (what a detector emits) and 0.7 to 1.0 times as fast when almost nothing is
// eliminated (measured on 32 to 1024 frames of 1024 to 4096 boxes).  Frames of 512 boxes or
// fewer never gain: their stages are mostly barriers.  From 2^28 pair slots on (64 x 2048: 40 us
// against 43 for all pairs; 64 x 1536, below: 38 against 33).  Frames beyond sort_chunk boxes take
// it from 2^31 pair slots on (below that the two launches are quicker).  (nms_route_for asks
// nms_use_small_frames first, which takes the batches of frames of up to 1024 boxes and small
// batches of longer ones.)
NMS_HD bool nms_use_early_exit(int n_max, int frames, int sort_chunk)
{
    const long long slots = (long long)frames * n_max * n_max;
    return n_max > sort_chunk ? slots >= (1ll << 31) : (n_max > 1024 && slots >= (1ll << 28));
}

// Workgroups that share a frame in the small-frames kernels (each builds the tables of the whole
// frame and takes every parts-th tile of victims; a share is at most 16 tiles, and more workgroups
// than tiles would only build tables).  Frames of up to 1024 boxes: doubled while that leaves at most
// one workgroup per compute unit (256), and once more -- two workgroups fit a compute unit -- as
// long as a share keeps four tiles of victims (measured: 256 x 1024 31.6 -> 28.4 us, 256 x 768
// 36.3 -> 26.5; with two-tile shares, 64 x 1024 12.4 -> 13.9).  Longer frames: one workgroup per
// compute unit (their tables fill its LDS), as many as that allows.
NMS_HD int nms_small_frames_parts(int frames, int n_max)
{
    const int tiles = (n_max + 63) / 64;
    const int most = tiles < 64 ? tiles : 64;  // a workgroup without a tile of victims would only build tables
    int parts = (tiles + 15) / 16;
    if (n_max <= 512) {  // workgroups of 512 threads, up to four on a compute unit
        parts = 1;
        while (parts * 2 <= tiles && (long long)frames * parts * 2 <= 512) parts *= 2;
        return parts;
    }
    if (n_max > 1024) {
        const int fit = 256 / (frames < 256 ? frames : 256);
        return fit > most ? most : (fit < parts ? parts : fit);
    }
    while (parts * 2 <= most && (long long)frames * parts * 2 <= 256) parts *= 2;
    while (parts * 2 <= most && (long long)frames * parts * 2 <= 512 && tiles / (parts * 2) >= 4) parts *= 2;
    return parts;
}

// Frames of 513 to 1024 boxes, ten or more of them (longer and shorter frames: inside): one launch without a sort, in which a
// workgroup of 1024 threads tests every victim of its frame against the two best-ranked of every
// sixteen input elements and the victims still alive against the whole frame (clustered detections,
// whole call: 64 x 1024 11.8 us, all pairs 20.8; 256 x 1024 28.4, early exit 34.5, all pairs 43.2;
// 2048 x 1024 155, early exit 197; 128 x 640 17.6, all pairs 20.3).  Its workgroups are 1024 threads
// and its tables 1024 rows whatever the frame size, so short frames gain nothing (256 x 512: 19.3
// against 20.4; 192 x 576: 26.0 against 21.7), and between 256 and 512 frames the workgroups beyond
// one per compute unit share a compute unit with another (300 x 768: 40.8 against 37.7; 300 x 1024:
// 45.0 against 47.9).  In tiles of 64 boxes per frame:
NMS_HD bool nms_use_small_frames(int n_max, int frames)
{
    const int tiles = (n_max + 63) / 64;
    if (n_max > 1024) {
        // Frames of 1025 to 4096 boxes (two or four elements per thread), a few of them.  Below 2^25 pair slots the
        // direct form is quicker (4 x 2048: 9.5 us against 10.6; the tables cost 4 us before the first pair test).
        // Above that the kernel wins while a workgroup's share stays at four tiles of victims (five beyond 2048
        // boxes) with one workgroup per compute unit: 8 x 2048 11 us against 17 (direct), 32 x 2048 25 against 30
        // (all pairs), 4 x 4096 15 against 29, 16 x 4096 33 against 40 (early exit), 40 x 1536 24.5 against 26.4;
        // 44 x 1536 31.5 against 28.5, 56 x 1100 30.8 against 25.0, 29 x 3000 47.8 against 48.1.
        if (n_max > 4096 || frames > 256 || (long long)frames * n_max * n_max < (1ll << 25)) return false;
        const int parts = nms_small_frames_parts(frames, n_max);
        return (tiles + parts - 1) / parts <= (n_max > 2048 ? 5 : 4);
    }
    // frames of 449 to 512 boxes (workgroups of 512 threads), many of them: 256 x 512 16.3 us against 20.1 for all pairs,
    // 2048 x 512 72 against 97; 128 x 512 13.2 against 14.4 (direct); shorter frames or fewer gain nothing (512 x 384: 25.0
    // against 23.9; 64 x 512: 8.9 against 8.6)
    if (n_max <= 512) return tiles == 8 && frames >= 128;
    // against the direct form, where that would be taken (10 to 32 frames: 12 x 1024 7.1 us against 8.5, 24 x 1024 8.2
    // against 15.4, 32 x 768 8.5 against 9.4; 8 x 1024 7.0 against 6.3, 16 x 768 7.2 against 6.2, 32 x 576 8.8 against 8.0)
    if (nms_use_direct_form(n_max, frames)) return tiles >= 10 && (long long)frames * n_max * n_max > (5ll << 21);
    if (frames <= 128) return tiles >= 9;
    if (frames <= 256) return tiles >= 11;
    if (frames < 512) return tiles >= 15;
    return tiles >= 11;
}

// ---- boxes in order of place (spatial_frames_kernel) -----------------------------------------------
// Frames of up to 4096 boxes, for thresholds with a division-free form, whatever nms_route_for names for the
// rest.  Its tables cost some 7 us whatever the batch; the line is where it passes the direct form and the
// sort-free kernels on clustered detections (much eliminated) and on sparse anchors (little eliminated).  Whole
// call, us, place / before: 28 x 1000 7.4 / 8.0 and 10.2 / 12.8, 31 x 900 (before) 8.2 and 12.7, 44 x 640 7.0 / 10.2 and 9.9 / 16.0, 16 x 1024
// 7.5 / 7.0, 16 x 600 6.8 / 5.9; 8 x 1025 7.5 / 7.4 and 9.1 / 7.4, 9 x 1025 7.5 / 8.7 and 9.0 / 8.6, 6 x 1350 7.4 / 7.3 and 8.7 / 7.3, 7 x 1350
// 7.5 / 9.6 and 8.7 / 9.6, 5 x 1600 7.7 / 8.2 and 9.3 / 8.2, 5 x 1650 7.7 / 10.6 and 8.9 / 10.6, 4 x 2048 8.1 / 9.5 and 9.1 / 9.6; 2 x 2049
// 9.2 / 6.8 and 10.3 / 6.8, 2 x 2240 9.2 / 9.3 and 9.9 / 9.3, 2 x 2300 9.3 / 10.9 and 10.2 / 11.0, 3 x 2176 9.4 / 9.6 and 10.2 / 9.6, 4 x 2049 9.4 / 10.8 and
// 10.2 / 10.7; 1 x 4096 10.2 / 8.9, 2 x 4096 11.0 / 14.5.  Shorter frames gain on clustered detections only
// (1000 x 300 14 / 34, but anchors 35 / 34) until there are many of some 500 boxes (512 x 512 11.3 / 18.7 and 32 / 41).
NMS_HD bool nms_use_spatial_frames(int n_max, int frames, int sort_chunk)
{
    const long long total = (long long)frames * n_max;
    if (n_max > sort_chunk) return false;
    if (n_max > 2048) return frames >= (n_max >= 2300 ? 2 : 4);
    if (n_max > 1024) return total >= (n_max >= 1640 ? 8000 : 9000);
    if (n_max > 512) return total >= 28000;
    return n_max > 448 && frames >= 512;
}

// Workgroups that share a frame: one per compute unit, each with a tile of victims.
NMS_HD int nms_spatial_frames_parts(int n_max, int frames)
{
    const int tiles = (n_max + 63) / 64;
    const int fit = 256 / (frames < 256 ? frames : 256);
    return fit < tiles ? fit : tiles;
}

// log2 of the wavefronts (of W) that share 64 victims in its first stage.
NMS_HD int nms_spatial_frames_split(int n_max, int parts, int W)
{
    const int tiles = ((n_max + 63) / 64 + parts - 1) / parts;
    return tiles * 4 <= W ? 2 : (tiles * 2 <= W ? 1 : 0);
}

// The same for the paper's rule with IoU, labels, a strict compare or ignored ties, against rank and map step.  Whole call, us, place / before,
// sparse anchors, then clustered.  IoU without labels: 1 x 600 9.3 / 11.6, 7.3 / 14.4; 8 x 500 9.7 / 10.5, 7.4 / 13.5; 60 x 1000 19.6 / 23.9, 9.3 / 28.9; 80 x 1000 24.4 / 25.8,
// 10.3 / 32; 100 x 520 19.4 / 20.9, 9.1 / 23.4; 95 x 800 27 / 24.8, 10.8 / 30; 97 x 1024 31.9 / 28.2, 12 / 35; 130 x 520 28.5 / 22.3, 10.7 / 27: what is left of a frame that little is
// eliminated from is one compute unit's work, of two frames of three beyond 85 frames.  Longer frames keep it although such batches lose: 100 x 1500 45 / 49, 16 / 60;
// 20 x 4096 28 / 71; 200 x 1025 49 / 50, 16.5 / 61, but 150 x 1100 53 / 44, 18 / 54 and 300 x 1100 100 / 82, 30 / 110.  20 labels: 1 x 64 7.3 / 8.8, 7.0 / 11.8; 46 x 256 8.2 / 11.5, 8.2 / 13.6;
// 97 x 1024 30.8 / 33.9, 27 / 38; 100 x 2000 60 / 95, 46 / 102; one label 46 x 256 8.6 / 12.3, 7.0 / 16.5, 20 x 4096 60 / 94, 21 / 106; labels beyond 255, which are looked up in memory where
// boxes hit, 60 x 1000 22 / 28, 20 x 4096 36 / 88.  Strict compare: 8 x 500 8.0 / 8.7, 97 x 1024 19.8 / 26.7.  Longer frames: 5 x 7000 crowd 19 / 60.
NMS_HD bool nms_use_spatial_variant(int n_max, int frames, bool iou, bool labelled)
{
    const long long total = (long long)frames * n_max;
    if (n_max > 1024) return true;
    if (n_max > 512) return total <= (!iou || labelled ? 100000 : (frames <= 85 ? 87040 : 70000)) && (!iou || labelled || frames <= 128);
    if (n_max > 256) return total <= 6000;
    return labelled && total <= 12000;
}

// The greedy rule under IoU in order of place (place_relation_kernel, place_resolve_kernel) against rank, mask and sweep; from walk_boxes boxes in
// frames of up to sort_chunk on the walk and the class kernel take them.  Whole call, us, place / rank, mask and sweep, clustered, then sparse anchors:
// 1 x 4096 27.3 / 36.0, 26.9 / 35.6; 4 x 4096 35 / 50, 32 / 48; 31 x 4096 91 / 134, 86 / 121; 20 x 3000 55 / 71, with 20 labels 49 / 74; 1 x 2049
// 22.5 / 23.5; clustered 1 x 8000 61 / 89, 6 x 8000 90 / 142, 60 x 8000 334 / 725.  Shorter frames gain nothing, and at a lower threshold lose: 2 x 2048 at
// 0.3 34 / 23, 3 x 1500 26 / 22.  Where thousands of candidates crowd around few objects: one object 1 x 4096 54 / 39, 31 x 4096 78 / 192, 1 x 8000 133 / 96; four
// 83 / 38, 198 / 192, 147 / 96; sixteen 41 / 38, 172 / 190, 184 / 96.  A chain of 4096 eliminators in place order 270 / 187, in random order 939 / 187.
// (Under the default measure a box has ten times the eliminators: 24 x 3000 anchors 133 / 60.)  Against the walk the line has not been drawn anew.
NMS_HD bool nms_use_place_greedy(int n_max, int frames, int sort_chunk, long long walk_boxes)
{
    const long long total = (long long)frames * n_max;
    if (n_max <= 2048 || n_max > 2 * sort_chunk) return false;
    return n_max > sort_chunk || total < walk_boxes;
}

// A frame's block of the relation, in 64-bit words; its place is the mask's, n_pad / 64 * n_pad words.  A row's first kRelationWords masks
// lie side by side, the others in a column each; behind them the ranked rows of the walk (box, input index, score, label).
constexpr int kRelationWords = 4;
constexpr int kRelationMasks = 16;
struct NmsRelationBlock {
    size_t more, ranked, end;
};
NMS_HD NmsRelationBlock nms_relation_block(int n_pad)
{
    NmsRelationBlock b;
    b.more = (size_t)kRelationWords * n_pad;
    b.ranked = (size_t)kRelationMasks * n_pad;
    b.end = b.ranked + (size_t)n_pad * (16 + 3 * 4) / 8;
    return b;
}

// Places per workgroup of place_sort_kernel: a multiple of 64, at most 1024; a workgroup per compute unit where the batch allows.  Twice and four times
// the share (half and a quarter of the workgroups, whole call, us, share / twice / four times): 1 x 16,384 20.4 / 20.5 / 21.2; 2 x 16,384 24.2 / 24.4 / 25.1; 16 x 5000
// 20.9 / 21.0 / 21.3; 8 x 5000 18.6 / 18.6 / 18.8; 1 x 4200 and 64 x 8192 alike; only 1 x 30,000 takes 44.1 / 41.6 / 42.0 (every workgroup reads the whole frame again).
NMS_HD int nms_place_share(int n_max, int frames)
{
    const int parts = 256 / (frames < 256 ? frames : 256);
    const int share = ((n_max + parts - 1) / parts + 63) / 64 * 64;
    return share < 1024 ? share : 1024;
}

// The route of the automatic whole-path call for a batch shape (1 <= n_max, 1 <= frames) where the threshold takes the literal division.  Its
// lines were drawn with division-free thresholds, before those took the boxes in order of place from some batch size on.  With the
// literal form, whole call, us, this route / all pairs, at 2^-41 (every overlap eliminates), then at 2^22 (nothing does): 64 x 1024 clustered 13 / 32, 48 / 31;
// 8 x 2048 8.5 / 25, 26 / 25; 16 x 4096 34 / 91, 184 / 91; 64 x 2048 46 / 86, 118 / 85; 256 x 4096 anchors 111 / 1079, 1218 / 1075; 1 x 16384 crowd 51 / 87, 117 / 87;
// 16 x 16384 264 / 1109, 1250 / 1103; at 0 10 / 31 to 94 / 1076.
NMS_HD int nms_route_for(int n_max, int frames, int sort_chunk)
{
    if (nms_use_small_frames(n_max, frames)) return kNmsRouteSmallFrames;
    if (nms_use_direct_form(n_max, frames)) return kNmsRouteDirect;
    if (nms_use_early_exit(n_max, frames, sort_chunk)) return kNmsRouteEarlyExit;
    if (nms_use_two_launches(n_max, frames, sort_chunk)) return kNmsRouteTwoLaunch;
    return kNmsRouteAllPairs;
}

// The same at a threshold: division_free as in NmsThetaConst::fast.
NMS_HD int nms_route_with(int n_max, int frames, int sort_chunk, bool division_free)
{
    if (division_free && nms_use_spatial_frames(n_max, frames, sort_chunk)) return kNmsRoutePlaceFrames;
    if (division_free && n_max > sort_chunk) return kNmsRoutePlaceTable;
    return nms_route_for(n_max, frames, sort_chunk);
}

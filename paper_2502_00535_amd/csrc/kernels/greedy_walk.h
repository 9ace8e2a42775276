// Part of nms_kernels.hip (included there, inside its anonymous namespace): classic greedy rule without a mask: one workgroup walks a frame in rank order (also with the variants).
#pragma once

// ----------------------------------------------------------------------------- greedy rule without a mask

// The classic sequential rule walked tile by tile in rank order, one workgroup (16
// wavefronts) per frame, no mask in memory.  Under this rule a box that is eliminated
// neither eliminates others nor needs any further test, so only the SURVIVORS are ever used
// as outranking boxes: about 600 of 4096 on frames like configuration 4, i.e. a seventh of
// the pair grid.  A frame is one compute unit's work, so the route pays from a few dozen
// frames on.
//
// The rows that are left (at first all of them) are numbered in rank order and cut into tiles
// of 64; wavefront w owns the tiles w, w + 16, w + 32, w + 48 and keeps their boxes in
// registers, lane = row, with one wave-uniform 64-bit word per tile for the rows that are out.
// Round t settles tile t, whose rows its owner has put into LDS:
//   - all wavefronts, a share each: the survivors of tile t-1 ("list t-1", in LDS) against the
//     tile, and for each row of the tile the better-ranked rows of the tile itself that
//     eliminate it (one 64-bit word per row); barrier;
//   - the owner combines the shares and finds the tile's survivors as the fixed point of
//     "alive, and not eliminated by a surviving better-ranked row of the tile", writes them
//     to LDS as list t and marks them in keep_out; meanwhile every wavefront applies list t-1
//     to all its other tiles; barrier.
//
// Most rows that die do so early (on configuration 4 more than half of the rows are out after
// the first two tiles), and a tile costs the same with one row alive as with 64.  So the walk
// runs in stages of 2, 4, 8, ... tiles; after a stage the rows still alive are compacted (their
// rank numbers through LDS, their boxes gathered again from the table) into fewer tiles and
// the walk starts over on them.  The last stage begins once 16 tiles or fewer are left.
// (With W wavefronts: greedy_classes_kernel walks frames of up to 1024 boxes with 4 or 8.)
constexpr int kFusedWaves = 16;

// The greedy calls take the walk from frames * n_max boxes on, rank + mask + sweep below.  The line was drawn against
// a sweep of twice the present one's time and knows neither measure nor scene.  Walk against mask, whole call, us, much /
// little eliminated: 32 x 4096 75 / 140 against 114 / 109, 64 x 2100 50 / 90 against 66 / 63, 128 x 1024 34 / 60 against 39 / 36, 128 x 3000
// 54 / 113 against 177 / 166; IoU 32 x 4096 132 / 541 against 140 / 124, 64 x 2100 55 / 240 against 82 / 70, 128 x 1024 42 / 103 against
// 50 / 40, 256 x 4096 141 / 562 against 687 / 600: on detections that cluster the walk is ahead of the mask from the line on.
// Below the line frames of 2049 to 4096 boxes under IoU go in order of place (nms_use_place_greedy), at 31 x 4096 91 / 86; the walk has not been
// timed against that, and one frame more costs 129 / 524.  Where thousands of candidates crowd around one object it is the walk that is ahead, 29 against 78.
constexpr long long kGreedyFusedBoxes = 32ll * 4096;

struct FusedCandidate {  // a survivor as an outranking box (fields a variant does not use are never read)
    float x1, y1, x2, y2, area, T, score;
    int label;
};

enum { kExTiesIgnore = 2, kExClasses = 4 };                       // flags of the variants (AUX)
enum { kExBoundary = 0, kExDivideGe = 1, kExDivideGt = 2 };      // how a variant decides the threshold (MODE)

// What the walk needs beyond the box table when it runs a variant of the rule (EX): see
// map_tile_ex_kernel below for the arithmetic.
struct FusedVariant {
    const float *ranked_score;    // [frames][n_pad], rank order (AUX)
    const int32_t *ranked_label;  // [frames][n_pad], rank order (AUX with labels)
    double boundary;              // rounding boundary of the division next to theta (MODE == kExBoundary)
    float offset;                 // 1 or 0
    int flags;
};

// The float32 that a candidate carries in FusedCandidate::T when the threshold has a boundary form.
// The default measure and the outranking-area variants: the value that decides (nms_pair.h).
// Intersection over union: the value below which a pair is a certain miss whatever the victim -- the
// float32 at or below boundary * area * (1 - 2^-21), by the argument at map_tile_ex_kernel's c_T1;
// where that is not positive (a candidate without area) nothing is a certain miss.  A variant's value
// that is not positive becomes -infinity: every intersection, none included, reaches it.
template <bool EX, bool IOU>
__device__ __forceinline__ float fused_threshold(float area, double boundary)
{
    if (!IOU) {
        const float t = nms_pair_threshold(area, boundary);
        return !EX || t > 0.0f ? t : -INFINITY;
    }
    const double t = boundary * (double)area * (1.0 - 0x1p-21);
    float t1 = (float)t;
    if ((double)t1 > t) t1 = __uint_as_float(__float_as_uint(t1) - 1u);  // next float32 down (t > 0)
    return t1 > 0.0f ? t1 : -INFINITY;
}

// First test of a pair, decisive but for AUX in boundary form, where scores and labels are still to be
// looked at and a hit under IoU only means "maybe".  One floor is enough there: a negative width
// times a floored height reaches no positive T, and T = -infinity passes everything on.  The union of
// IoU is no smaller than either box, so the victim's own T (v_T) bounds the intersection too: with the
// candidate's alone every box that contains the candidate is a "maybe".
template <bool EX, bool IOU, int MODE, bool AUX>
__device__ __forceinline__ bool fused_first(const float4 v, float v_area, float v_T, float v_score, int v_label,
                                            const FusedCandidate &c, float theta, const FusedVariant &o)
{
    if (!EX) {
        if (MODE == kExBoundary) return nms_eliminates_fast(v.x, v.y, v.z, v.w, c.x1, c.y1, c.x2, c.y2, c.T);
        return nms_eliminates_exact(v.x, v.y, v.z, v.w, c.x1, c.y1, c.x2, c.y2, c.area, theta);
    }
    float iw = (fminf(v.z, c.x2) - fmaxf(v.x, c.x1)) + o.offset;
    if (MODE != kExBoundary || (IOU && !AUX)) iw = fmaxf(0.0f, iw);
    const float ih = fmaxf(0.0f, (fminf(v.w, c.y2) - fmaxf(v.y, c.y1)) + o.offset);
    const float inter = iw * ih;
    const float denom = IOU ? (v_area + c.area) - inter : c.area;
    if (MODE == kExBoundary && IOU && !AUX) return (double)inter >= o.boundary * (double)denom;
    if (MODE == kExBoundary) return inter >= (IOU ? fmaxf(c.T, v_T) : c.T);
    bool hit = MODE == kExDivideGe ? !(inter / denom < theta) : inter / denom > theta;
    if (AUX) {
        hit = hit && ((o.flags & kExTiesIgnore) == 0 || c.score > v_score);
        hit = hit && ((o.flags & kExClasses) == 0 || c.label == v_label);
    }
    return hit;
}

// Is there anything to decide after fused_first?
template <bool EX, bool IOU, int MODE, bool AUX>
constexpr bool kFusedSecond = EX && MODE == kExBoundary && AUX;

// What is left to decide for the lanes of `word` (not 0) that fused_first let through.
template <bool IOU, bool AUX>
__device__ __forceinline__ unsigned long long fused_second(unsigned long long word, const float4 v, float v_area, float v_score,
                                                           int v_label, const FusedCandidate &c, const FusedVariant &o)
{
    if (AUX) {
        if (o.flags & kExTiesIgnore) word &= __ballot(c.score > v_score);
        if (o.flags & kExClasses) word &= __ballot(c.label == v_label);
    }
    if (IOU && word != 0) {
        const float iw = fmaxf(0.0f, (fminf(v.z, c.x2) - fmaxf(v.x, c.x1)) + o.offset);
        const float ih = fmaxf(0.0f, (fminf(v.w, c.y2) - fmaxf(v.y, c.y1)) + o.offset);
        const float inter = iw * ih;
        const float denom = (v_area + c.area) - inter;
        word &= __ballot((double)inter >= o.boundary * (double)denom);
    }
    return word;
}

// Does candidate c eliminate the victim?  The lane mask over the lanes of `open` (the others do not
// matter).  !EX: the default measure (MODE kExBoundary = the division-free form of nms_pair.h, else the
// literal division).  EX: the variants.  With scores or labels to look at, what follows the first test sits
// behind a wave-uniform branch (40 frames of 4096 boxes of one label, which are walked, IoU, the whole call: 191 -> 172 us
// where much is eliminated, 833 -> 578 where little is).  IoU alone takes the float64 compare for every pair: the branch gains 1 % where
// few pairs hit (64 x 2100) and costs 5 to 9 % where many do (300 x 600: 52 -> 57 us).
template <bool EX, bool IOU, int MODE, bool AUX>
__device__ __forceinline__ unsigned long long fused_word(unsigned long long open, const float4 v, float v_area, float v_T,
                                                         float v_score, int v_label, const FusedCandidate &c, float theta, const FusedVariant &o)
{
    unsigned long long word = __ballot(fused_first<EX, IOU, MODE, AUX>(v, v_area, v_T, v_score, v_label, c, theta, o)) & open;
    if (kFusedSecond<EX, IOU, MODE, AUX> && word != 0) {
        asm volatile("" ::: "memory");  // keeps this a branch
        word = fused_second<IOU, AUX>(word, v, v_area, v_score, v_label, c, o);
    }
    return word;
}

// Bitwise OR over each row of 16 lanes, in the row's last lane.
__device__ __forceinline__ unsigned row_or16(unsigned x)
{
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);  // row_shr:1
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);  // row_shr:2
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);  // row_shr:4
    x |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);  // row_shr:8
    return x;
}

constexpr int kWalkChunk = 4;  // survivors fetched from LDS at a time
constexpr int kWalkLists = 2;  // lists kept in LDS: the one being written and the one being applied

// W: wavefronts of the workgroup; N: the longest frame, of W, 2 W or 4 W tiles.
template <int W, int N>
struct WalkShared {
    float4 box[kWalkLists + 1][kTile];      // list t in buffer t % kWalkLists
    float aux[kWalkLists + 1][kTile];
    float area[kWalkLists + 1][kTile];
    float score[kWalkLists + 1][kTile];
    int label[kWalkLists + 1][kTile];
    int count[kWalkLists];
    unsigned long long part[W];             // rows of the tile being settled that a wavefront's share of the list before eliminates
    unsigned long long hitters[kTile];      // per row of that tile: the better-ranked rows of the tile that eliminate it
    int alive[N / kTile];                   // compaction: rows alive per tile
    int ids[N / kTile > W ? N : 1];         // compaction: rank numbers of the rows left
};

// One frame, by all wavefronts of the workgroup.
template <bool EX, bool IOU, int MODE, bool AUX, int W, int N>
__device__ __forceinline__ void walk_frame(WalkShared<W, N> &sh, const float *__restrict__ sorted_f, const int32_t *__restrict__ order_f,
                                           const float *__restrict__ score_f, const int32_t *__restrict__ label_f, int n_f, int n_max,
                                           int n_pad, const NmsThetaConst th, const FusedVariant opt, uint8_t *__restrict__ keep_f)
{
    constexpr int kOwned = N / kTile / W;
    static_assert(kOwned == 1 || kOwned == 2 || kOwned == 4, "apply() dispatches on up to four slots");
    constexpr bool kUseT = MODE == kExBoundary && (!IOU || AUX);  // the list carries T, else the area
    constexpr bool kUseArea = kUseT && IOU;              // ... and the area as well
    constexpr bool kSecond = kFusedSecond<EX, IOU, MODE, AUX>;
    constexpr int kTileBuf = kWalkLists;                 // one more buffer of the same layout: the rows of the tile being settled
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const float4 *box4 = reinterpret_cast<const float4 *>(sorted_f);
    const float *area = sorted_f + 4 * (size_t)n_pad;

    for (int i = (int)threadIdx.x; i < n_max; i += W * 64) keep_f[i] = 0;  // survivors are marked as they are found

    // The owned tiles that are not settled yet, the next one to settle in slot 0 (after a tile is
    // settled the others move down one slot).
    float4 vb[kOwned];
    FusedCandidate self[kOwned];     // the same rows in their role as outranking boxes
    int rank_of[kOwned];             // rank number of the lane's row
    unsigned long long out[kOwned];  // wave-uniform; bit r: row r is eliminated or does not exist
    int left = 0;                         // owned tiles not settled yet
    int tn = 0;                           // number of the tile in slot 0 (the others follow in steps of W)
    int n_cur = n_f;                      // rows in the current numbering

    // (re)load the owned tiles of the current numbering; `compacted`: rank numbers come from sh.ids
    auto load_tiles = [&](bool compacted) __attribute__((always_inline)) {
        left = 0;
        tn = wave;
#pragma unroll
        for (int i = 0; i < kOwned; ++i) {
            const int first = (wave + W * i) * kTile;
            const bool has = first < n_cur;
            left += has ? 1 : 0;
            const int q = first + lane;
            const bool real = q < n_cur;
            const int r = real ? (compacted ? sh.ids[q] : q) : 0;  // rows that do not exist read row 0 and are marked out
            rank_of[i] = r;
            vb[i] = box4[r];
            FusedCandidate me;
            me.x1 = vb[i].x, me.y1 = vb[i].y, me.x2 = vb[i].z, me.y2 = vb[i].w;
            me.area = EX ? ((vb[i].z - vb[i].x) + opt.offset) * ((vb[i].w - vb[i].y) + opt.offset) : area[r];
            me.T = kUseT ? fused_threshold<EX, IOU>(me.area, EX ? opt.boundary : th.m) : 0.0f;
            me.score = AUX ? score_f[r] : 0.0f;
            me.label = (AUX && (opt.flags & kExClasses)) ? label_f[r] : 0;
            self[i] = me;
            out[i] = !has ? ~0ull : (first + kTile <= n_cur ? 0ull : ~0ull << (n_cur - first));
        }
    };
    load_tiles(false);
    __syncthreads();  // the zero fill is complete before any survivor's byte is written

    // Entry k of buffer `buf` (a list's survivor, or a row of the tile being settled).  With a
    // wave-uniform k every lane gets the same entry (a broadcast read); with k = lane, its own.
    auto entry = [&](int buf, int k) __attribute__((always_inline)) {
        FusedCandidate c;
        const float4 b = sh.box[buf][k];
        c.x1 = b.x, c.y1 = b.y, c.x2 = b.z, c.y2 = b.w;
        c.T = kUseT ? sh.aux[buf][k] : 0.0f;
        c.area = kUseArea ? sh.area[buf][k] : (kUseT ? 0.0f : sh.aux[buf][k]);
        c.score = AUX ? sh.score[buf][k] : 0.0f;
        c.label = AUX ? sh.label[buf][k] : 0;
        return c;
    };
    // What fused_first needs of it, and under IoU the label: where a second test follows, its other fields are only fetched or made there.
    auto first_entry = [&](int buf, int k) __attribute__((always_inline)) {
        if (!kSecond) return entry(buf, k);
        FusedCandidate c;
        const float4 b = sh.box[buf][k];
        c.x1 = b.x, c.y1 = b.y, c.x2 = b.z, c.y2 = b.w;
        c.T = sh.aux[buf][k];
        c.area = c.score = 0.0f;
        c.label = IOU ? sh.label[buf][k] : 0;
        return c;
    };
    // The list in buffer `buf` against the tiles in slots 0 .. S-1.  Survivors are fetched four
    // at a time into two sets of registers in turn, the next four while the current four are
    // tested; a full chunk has no branch inside.
    auto apply_slots = [&](auto slots, int buf) __attribute__((always_inline)) {
        constexpr int S = decltype(slots)::value;
        const int count = __builtin_amdgcn_readfirstlane(sh.count[buf]);
        if (count == 0) return;
        auto fetch = [&](FusedCandidate (&c)[kWalkChunk], int k0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kWalkChunk; ++u) c[u] = first_entry(buf, k0 + u < count ? k0 + u : count - 1);
        };
        // survivor c (entry k) against the S tiles
        auto test_one = [&](const FusedCandidate &c, int k) __attribute__((always_inline)) {
            unsigned long long word[S];
            unsigned long long any = 0;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                word[i] = __ballot(fused_first<EX, IOU, MODE, AUX>(vb[i], self[i].area, self[i].T, self[i].score, self[i].label, c, th.theta, opt));
                if (kSecond) {
                    word[i] &= ~out[i];
                    any |= word[i];
                } else {
                    out[i] |= word[i];
                }
            }
            if (kSecond && any != 0) {
                asm volatile("" ::: "memory");  // keeps this a branch
                FusedCandidate full = c;
                if (IOU) {  // no second round trip to LDS: where much is eliminated, most survivors come this way
                    full.area = ((c.x2 - c.x1) + opt.offset) * ((c.y2 - c.y1) + opt.offset);
                    if (opt.flags & kExTiesIgnore) full.score = sh.score[buf][k];
                } else {
                    full = entry(buf, k);
                }
#pragma unroll
                for (int i = 0; i < S; ++i)
                    if (word[i] != 0)
                        out[i] |= fused_second<IOU, AUX>(word[i], vb[i], self[i].area, self[i].score, self[i].label, full, opt);
            }
        };
        auto test = [&](const FusedCandidate (&c)[kWalkChunk], int k0) __attribute__((always_inline)) {
            if (k0 + kWalkChunk <= count) {
#pragma unroll
                for (int u = 0; u < kWalkChunk; ++u) test_one(c[u], k0 + u);
            } else {
#pragma unroll
                for (int u = 0; u < kWalkChunk - 1; ++u)
                    if (k0 + u < count) test_one(c[u], k0 + u);  // wave-uniform
            }
        };
        FusedCandidate even[kWalkChunk], odd[kWalkChunk];
        fetch(even, 0);
        for (int k0 = 0; k0 < count; k0 += 2 * kWalkChunk) {
            if (k0 + kWalkChunk < count) fetch(odd, k0 + kWalkChunk);
            test(even, k0);
            if (k0 + kWalkChunk >= count) break;
            if (k0 + 2 * kWalkChunk < count) fetch(even, k0 + 2 * kWalkChunk);
            test(odd, k0 + kWalkChunk);
        }
    };
    auto apply = [&](int slots, int buf) __attribute__((always_inline)) {  // the same for a number of slots known at run time
        if (slots == 1) apply_slots(std::integral_constant<int, 1>(), buf);
        if constexpr (kOwned >= 2) {
            if (slots == 2) apply_slots(std::integral_constant<int, 2>(), buf);
        }
        if constexpr (kOwned == 4) {
            if (slots == 3) apply_slots(std::integral_constant<int, 3>(), buf);
            else if (slots >= 4) apply_slots(std::integral_constant<int, 4>(), buf);
        }
    };

    // the rows of slot 0 into LDS for the round that settles them
    auto post_tile = [&]() __attribute__((always_inline)) {
        sh.box[kTileBuf][lane] = vb[0];
        sh.aux[kTileBuf][lane] = kUseT ? self[0].T : self[0].area;
        if (kUseArea) sh.area[kTileBuf][lane] = self[0].area;
        if (AUX) sh.score[kTileBuf][lane] = self[0].score;
        if (AUX) sh.label[kTileBuf][lane] = self[0].label;
    };

    int g = 0;          // rounds so far over all stages: round g writes list g, into buffer g % kWalkLists
    for (int stage_tiles = 2;; stage_tiles *= 2) {
        const int tiles_cur = (n_cur + kTile - 1) / kTile;
        const int rounds = (tiles_cur <= W || stage_tiles >= tiles_cur) ? tiles_cur : stage_tiles;
        if (wave == 0) post_tile();  // tile 0 of this numbering
        lds_barrier();
        for (int t = 0; t < rounds; ++t, ++g) {
            const int pending = (g - 1) & (kWalkLists - 1);  // buffer of the list before (there is none in the very first round)
            // All wavefronts, a share each, on the tile being settled (its rows are in LDS, lane =
            // row): the survivors of the list before against it, and for each of its rows the
            // better-ranked rows of the tile itself that eliminate it.
            {
                const FusedCandidate row = entry(kTileBuf, lane);
                const float4 row_box = make_float4(row.x1, row.y1, row.x2, row.y2);
                const int count = g > 0 ? __builtin_amdgcn_readfirstlane(sh.count[pending]) : 0;
                unsigned long long part = 0;
                for (int k = wave; k < count; k += W)
                    part |= fused_word<EX, IOU, MODE, AUX>(~part, row_box, row.area, row.T, row.score, row.label, entry(pending, k),
                                                           th.theta, opt);
                if (lane == 0) sh.part[wave] = part;
#pragma unroll 1
                for (int j0 = 0; j0 < kTile / W; j0 += 4) {
                    FusedCandidate victim[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) victim[j] = entry(kTileBuf, wave + W * (j0 + j));
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int r = wave + W * (j0 + j);
                        const unsigned long long hitters = fused_word<EX, IOU, MODE, AUX>(
                            (1ull << r) - 1ull, make_float4(victim[j].x1, victim[j].y1, victim[j].x2, victim[j].y2), victim[j].area,
                            victim[j].T, victim[j].score, victim[j].label, row, th.theta, opt);
                        if (lane == 0) sh.hitters[r] = hitters;
                    }
                }
            }
            lds_barrier();
            if (wave == (t & (W - 1))) {
                // Settle tile t (slot 0).  A row survives iff it is alive and no surviving
                // better-ranked row of the tile eliminates it; iterated from "every alive row
                // survives" this settles one more row per pass at least, in practice a few passes.
                __builtin_amdgcn_s_setprio(3);
                const unsigned long long share = sh.part[lane & (W - 1)];
                const unsigned dead_lo = row_or16((unsigned)share), dead_hi = row_or16((unsigned)(share >> 32));
                const unsigned long long dead =
                    out[0] | ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)dead_hi, 15) << 32) |
                    (unsigned)__builtin_amdgcn_readlane((int)dead_lo, 15);
                const unsigned long long hitters = sh.hitters[lane];
                const bool alive = ((~dead >> lane) & 1ull) != 0;
                unsigned long long kept = ~dead;
                for (int pass = 0; pass < kTile; ++pass) {
                    const unsigned long long next = __ballot(alive && (hitters & kept) == 0);
                    if (next == kept) break;
                    kept = next;
                }
                const float4 v = vb[0];
                const FusedCandidate mine = self[0];
                const bool is_kept = (kept >> lane) & 1ull;
                const int into = g & (kWalkLists - 1);
                if (is_kept) {  // survivor number k of the tile is entry k of the list
                    const int k = __builtin_popcountll(kept & ((1ull << lane) - 1ull));
                    sh.box[into][k] = v;
                    sh.aux[into][k] = kUseT ? mine.T : mine.area;
                    if (kUseArea) sh.area[into][k] = mine.area;
                    if (AUX) sh.score[into][k] = mine.score;
                    if (AUX) sh.label[into][k] = mine.label;
                }
                if (lane == 0) sh.count[into] = __builtin_popcountll(kept);
                __builtin_amdgcn_s_setprio(0);
                if (is_kept) keep_f[order_f[rank_of[0]]] = 1;
#pragma unroll
                for (int i = 0; i + 1 < kOwned; ++i) {
                    vb[i] = vb[i + 1];
                    self[i] = self[i + 1];
                    rank_of[i] = rank_of[i + 1];
                    out[i] = out[i + 1];
                }
                --left;
                tn += W;
            } else if (t + 1 < rounds && wave == ((t + 1) & (W - 1))) {
                post_tile();  // the next round's tile
            }
            if (g > 0) apply(left, pending);  // the list before against the tiles that are left
            lds_barrier();
        }
        if (rounds == tiles_cur) break;  // every tile is settled
        if constexpr (kOwned > 1) {

            // End of a stage: the rows still alive move together (the list just written has not been
            // applied yet; it holds boxes, not row numbers, and is applied in the next stage's first
            // round like any other).  Tile `rounds + j` of the old numbering reports its count in
            // sh.alive[j]; a prefix sum gives every tile its place in sh.ids.
            const int tiles_left = tiles_cur - rounds;
#pragma unroll
            for (int i = 0; i < kOwned; ++i) {
                if (i < left && lane == 0) sh.alive[tn - rounds + W * i] = __builtin_popcountll(~out[i]);
            }
            lds_barrier();
            const unsigned mine_alive = lane < tiles_left ? (unsigned)sh.alive[lane] : 0u;
            const unsigned incl = wave_inclusive_sum(mine_alive);
            const int total = __builtin_amdgcn_readlane((int)incl, 63);
#pragma unroll
            for (int i = 0; i < kOwned; ++i) {
                if (i < left) {  // wave-uniform
                    const int base = __builtin_amdgcn_readlane((int)(incl - mine_alive), tn - rounds + W * i);
                    const unsigned long long alive = ~out[i];
                    if ((alive >> lane) & 1ull) sh.ids[base + __builtin_popcountll(alive & ((1ull << lane) - 1ull))] = rank_of[i];
                }
            }
            lds_barrier();
            n_cur = total;
            load_tiles(true);
        }
    }
}

template <bool EX, bool IOU, int MODE, bool AUX>
__global__ void __launch_bounds__(kFusedWaves * 64)
greedy_fused_kernel(const float *__restrict__ sorted5, const int32_t *__restrict__ order,
                    const int32_t *__restrict__ counts, int n_max, int n_pad, NmsThetaConst th, FusedVariant opt,
                    uint8_t *__restrict__ keep_out)
{
    __shared__ WalkShared<kFusedWaves, NMS_SORT_CHUNK> sh;
    const int f = blockIdx.x;
    walk_frame<EX, IOU, MODE, AUX>(sh, sorted5 + (size_t)f * 5 * n_pad, order + (size_t)f * n_max,
                                   AUX ? opt.ranked_score + (size_t)f * n_pad : nullptr,
                                   AUX ? opt.ranked_label + (size_t)f * n_pad : nullptr,
                                   frame_count(counts, f, n_max), n_max, n_pad, th, opt, keep_out + (size_t)f * n_max);
}

// Part of nms_kernels.hip (included there, inside its anonymous namespace): the paper's rule on frames of up to 4096 boxes, boxes in order of place, one launch.
#pragma once

// ----------------------------------------------------------------------------- frames in order of place

// Two boxes that do not touch decide nothing, and of the pairs of a picture few touch: 159 of 4096 boxes
// touch a given one on regressed anchors, 103 on clustered detections.  Algorithm 1 asks of a pair only which
// box is ranked first, one compare of the rank keys, so nothing has to be sorted by score.  Here the boxes are
// put in order of PLACE, and the pairs that are far apart are left out.  A workgroup per frame (or several,
// which build the same tables and share the victims), everything in LDS:
//
//   cells     a grid over the centres, in four classes of box size (a large box among small ones would stretch
//             the hull of its tile); boxes are counted per cell, and a prefix sum over the cells, a Hilbert curve
//             per class, gives every cell its rows of the table;
//   tiles     64 rows: their hull (the smallest box around them), smallest threshold T and best rank;
//   stage 1   lane = victim, against the best-ranked box of each of the nine cells around it, in its own size
//             class and in the next smaller one (a box is eliminated by what it covers).  This settles seven
//             victims of eight: 504 of 4096 are left on anchors, of which 362 survive;
//   stage 2   the victims left, four neighbours at a time, lane = outranking box, against the tiles that can
//             eliminate one of them (five to six of the 64): min, max, rounded subtraction, addition and
//             multiplication are all monotone, so the victim's float32 intersection with a tile's hull is no
//             smaller than with any box of the tile, and where it stays below the tile's smallest T no pair
//             test of the tile can succeed.
//
// The pair test itself is that of the other routes, and a pair is left out only when it is certain to fail or its
// victim has an eliminator: the same keep vector, bit for bit.  For thresholds with a division-free form (T > 0).
// The order of boxes inside a cell and the boxes of stage 1 are whatever the atomics make them; no result
// depends on them.
//
// What bounds it: on large batches VALU issue (by counters 74 k of 97 k cycles at 256 x 4096 anchors; the LDS is indexed in 34 k, 8 k of
// them bank conflicts; 17 k are the tables, 20 k stage 1, 55 k stage 2); on small ones the chain of seven barriers (256 x 1024: 18 k cycles).
// Measured, whole call, us, against the kernels that took these batches before (rank order, early exit):
// 256 x 4096 anchors 45.5 / 145, clustered 33.0 / 99; 48 ragged frames of 1777 boxes 10.0 / 29.3; 64 x 1024 8.5 / 11.7;
// 512 x 1024 anchors 45 / 133.
constexpr int kPlaceWaves = 16;  // most wavefronts of a workgroup

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_keep(float x)  // x of another lane; the lane's own where there is none
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, ROWS, 0xf, false));
}
// Minimum over each row of sixteen lanes, in the row's last lane.
__device__ __forceinline__ float row_min(float x)
{
    x = fminf(x, dpp_keep<0x111, 0xf>(x));  // row_shr:1, 2, 4, 8
    x = fminf(x, dpp_keep<0x112, 0xf>(x));
    x = fminf(x, dpp_keep<0x114, 0xf>(x));
    x = fminf(x, dpp_keep<0x118, 0xf>(x));
    return x;
}

// The same over the wavefront, wave-uniform.
__device__ __forceinline__ float wave_min(float x)
{
    x = row_min(x);
    x = fminf(x, dpp_keep<0x142, 0xa>(x));  // row_bcast:15 into rows 1, 3
    x = fminf(x, dpp_keep<0x143, 0xc>(x));  // row_bcast:31 into rows 2, 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// The grid over a frame's box centres (doubled centres: x1 + x2): AXIS x AXIS cells in four classes of box size.
struct PlaceGrid {
    float x0, y0, sx, sy;  // column = (x1 + x2 - x0) * sx
};
// A range that is empty or not finite maps to column 0.
__device__ __forceinline__ float place_scale(float lo, float hi, float cells)
{
    const float range = hi - lo;
    return range > 0x1p-100f && range < 0x1p100f ? cells * __builtin_amdgcn_rcpf(range) : 0.0f;
}
// Row and column of a box's centre.  Any coordinates give a legal cell: clamped before the conversion, masked after.
template <int AXIS>
__device__ __forceinline__ unsigned place_spot(const float4 b, const PlaceGrid &g)
{
    const float cx = fminf(fmaxf((b.x + b.z - g.x0) * g.sx, 0.0f), (float)(AXIS - 1));
    const float cy = fminf(fmaxf((b.y + b.w - g.y0) * g.sy, 0.0f), (float)(AXIS - 1));
    unsigned c = (unsigned)(int)cy * AXIS + (unsigned)(int)cx;
    asm volatile("" : "+v"(c));
    return c & (unsigned)(AXIS * AXIS - 1);
}
// Cell number: size class (area below 2, 8, 32 cells of a 16 x 16 grid, or more), row, column.
template <int AXIS>
__device__ __forceinline__ unsigned place_cell(const float4 b, const PlaceGrid &g)
{
    const float t = ((b.z - b.x) * g.sx) * ((b.w - b.y) * g.sy) * (256.0f / (AXIS * AXIS));  // (g is for doubled coordinates: t = area in cells / 4)
    const unsigned cls = t < 0.5f ? 0u : (t < 2.0f ? 1u : (t < 8.0f ? 2u : 3u));
    return cls * (unsigned)(AXIS * AXIS) + place_spot<AXIS>(b, g);
}
// The cells of a class in the order of Hilbert's curve (D. Hilbert, Mathematische Annalen 38, 1891): neighbours on the curve are neighbours in
// the picture.  From his construction: the curve of twice the side is four copies of the one before, the first mirrored
// in the diagonal, the next two as they are, the last mirrored in the other diagonal.
template <int AXIS>
struct HilbertCells {
    uint16_t at[AXIS * AXIS];
    constexpr HilbertCells() : at()
    {
        for (unsigned side = 1; side < (unsigned)AXIS; side *= 2) {
            const unsigned cells = side * side;
            for (unsigned i = 0; i < cells; ++i) {
                const unsigned x = at[i] % AXIS, y = at[i] / AXIS;
                at[i] = (uint16_t)(x * AXIS + y);
                at[cells + i] = (uint16_t)((y + side) * AXIS + x);
                at[2 * cells + i] = (uint16_t)((y + side) * AXIS + (x + side));
                at[3 * cells + i] = (uint16_t)((side - 1 - x) * AXIS + (2 * side - 1 - y));
            }
        }
    }
};
template <int AXIS>
__device__ constexpr HilbertCells<AXIS> hilbert_cells = HilbertCells<AXIS>();
// The cell that comes i-th: class by class, every second class backwards.
template <int AXIS>
__device__ __forceinline__ unsigned curve_cell(unsigned i)
{
    constexpr unsigned kClass = AXIS * AXIS;
    const unsigned cls = i / kClass, d = i % kClass;
    return cls * kClass + hilbert_cells<AXIS>.at[(cls & 1u) ? kClass - 1u - d : d];
}

constexpr int kPlaceGroup = 4;  // victims of a wavefront in the second stage
constexpr int kPlaceBins = 16;  // of labels

// The variant of the pair test and of the rule.
struct PlaceTest {
    double boundary;         // rounding boundary next to the threshold (map_tile_ex_kernel)
    float offset;            // pixel offset (IoU; the outranking-area forms are for 1)
    int ties_ignore;
    const int32_t *classes;  // null: no labels
};

// The tables of a frame.  P rows, AXIS cells per axis and size class.
template <int P, int AXIS>
struct PlaceShared {
    static constexpr int kCells = 4 * AXIS * AXIS;
    float4 box[P];
    float T[P];
    unsigned upper[P];                // upper half of the rank key
    unsigned meta[P];                 // input index, cell << 16, bits 4 to 7 of the label << 28
    union {
        uint8_t keep[P];              // parts == 1: by input index
        uint16_t row[P];              // parts > 1: row of an input element
    };
    float4 hull[kTile];               // per tile
    uint2 tile[kTile];                // smallest T, best (smallest) upper half of the tile
    unsigned bins[kTile];             // labels: the bins that the tile holds
    union {
        __align__(16) unsigned start[kCells];  // boxes per cell, then their first rows
        uint16_t list[P > 2 * kCells ? P : 2 * kCells];  // after that: rows still alive after the first stage
    };
    unsigned best[kCells + 2 * AXIS + 2];  // from a line and one on: a well-ranked box of the cell: 20 bits of the rank key, 12 bits of the row; ~0: no box
    unsigned wave_sum[kPlaceWaves];
    unsigned long long dead[kPlaceWaves];  // first stage, few victims: per 64 of them
    unsigned listed, next, wide;
};

// W: wavefronts; E: boxes per thread (frames of at most 64 W E).  Grid: frames x parts workgroups; a workgroup builds the tables
// of the whole frame and takes the victims of every parts-th 64 boxes.  split_log2: wavefronts per
// 64 victims in stage 1; when above 0 the workgroup has at most W / 2 such tiles.  (Integer divisions by the number of
// workgroups or tiles cost a chain this short 1.0 us: what they would say is in the grid and in split_log2.)
//
// IOU: intersection over union; the first test can only err towards "maybe", and what passes is decided in float64 behind a
// branch, as in map_tile_ex_kernel.  A box without area (T = 0) may eliminate what it does not touch: its tile reaches everything.
// LABELS: sixteen bins of labels take the place of the size classes, each with a grid of half the lines: tiles hold a label or
// two, and a victim meets the tiles of its bin only.  The bin and the four bits kept in meta tell labels from 0 to 255
// apart; a frame with others (wide) looks them up where boxes hit.
template <int W, int E, int AXIS, bool IOU, bool LABELS>
__global__ void __launch_bounds__(W * 64)
spatial_frames_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ counts,
                      int n_max, int split_log2, PlaceTest test, uint8_t *__restrict__ keep_out)
{
    constexpr int kThreads = W * 64;
    constexpr int P = E * kThreads;
    constexpr int kPer = 4 * AXIS * AXIS / kThreads;  // cells per thread in the prefix sum
    constexpr int A = LABELS ? AXIS / 2 : AXIS;       // cells per axis
    constexpr int kLines = LABELS ? 3 : 6;            // of cells tried in stage 1
    constexpr unsigned kSame = (unsigned)(kPlaceBins - 1) * (unsigned)(A * A) << 16 | 0xf0000000u;  // of meta: the label
    static_assert(kPer >= 1 && kPer * kThreads == 4 * AXIS * AXIS && E <= 4 && P <= 4096, "cells per thread, sixteen lanes per tile, rows in 12 bits");
    __shared__ PlaceShared<P, AXIS> sh;
    const int f = blockIdx.x;
    const int part = blockIdx.y, parts = gridDim.y;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    const float4 *box_f = reinterpret_cast<const float4 *>(boxes) + (size_t)f * n_max;
    const float *score_f = scores + (size_t)f * n_max;
    const int32_t *label_f = LABELS ? test.classes + (size_t)f * n_max : nullptr;
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const float off = IOU ? test.offset : 1.0f;
    if (part == 0)
        for (int i = n_f + tid; i < n_max; i += kThreads) keep_f[i] = 0;
    if (n_f == 0) return;

    const float4 sample = box_f[(unsigned)(lane * n_f) / 64u];
    float4 b[E];
    unsigned upper[E];
    int label[E];
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const int e = q * kThreads + tid;
        b[q] = box_f[e < n_f ? e : 0];
        upper[q] = (unsigned)(nms_rank_key(score_f[e < n_f ? e : 0], 0u) >> 32);
        label[q] = LABELS ? label_f[e < n_f ? e : 0] : 0;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        sh.start[i * kThreads + tid] = 0u;
        sh.best[i * kThreads + tid] = ~0u;
    }
    if (tid < 2 * AXIS + 2) sh.best[4 * AXIS * AXIS + tid] = ~0u;
    if (parts == 1) {
#pragma unroll
        for (int q = 0; q < E; ++q) sh.keep[q * kThreads + tid] = 0;
    }
    if (tid < kPlaceWaves) sh.dead[tid] = 0ull;
    if (LABELS && tid < kTile) sh.bins[tid] = 0u;
    if (tid == 0) {
        sh.listed = 0u;
        sh.next = 0u;
        sh.wide = 0u;
    }
    unsigned mine[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) mine[i] = curve_cell<A>((unsigned)(kPer * tid + i));
    lds_barrier();

    // ---- the grid, over the centres of 64 boxes spread over the input (what lies outside goes to the border cells)
    PlaceGrid grid;
    {
        const float cx = sample.x + sample.z, cy = sample.y + sample.w;
        grid.x0 = wave_min(cx), grid.y0 = wave_min(cy);
        const float hx = wave_min(-cx), hy = wave_min(-cy);
        grid.sx = place_scale(grid.x0, -hx, (float)A);
        grid.sy = place_scale(grid.y0, -hy, (float)A);
    }

    // ---- boxes per cell, the first row of every cell along the curve, the table
    unsigned cell[E], within[E];
#pragma unroll
    for (int q = 0; q < E; ++q) {
        cell[q] = LABELS ? nms_place_bin(label[q]) * (unsigned)(A * A) + place_spot<A>(b[q], grid) : place_cell<A>(b[q], grid);
        within[q] = 0;
        if (q * kThreads + tid < n_f) {
            within[q] = atomicAdd(&sh.start[cell[q]], 1u);
            if (LABELS && (unsigned)label[q] > 255u) sh.wide = 1u;
        }
    }
    lds_barrier();
    {
        unsigned in_cell[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            in_cell[i] = sh.start[mine[i]];
            sum += in_cell[i];
        }
        const unsigned incl = wave_inclusive_sum(sum);
        if (lane == 63) sh.wave_sum[wave] = incl;
        lds_barrier();
        const unsigned sums = row16_inclusive_sum(sh.wave_sum[lane & (W - 1)]);
        unsigned at = (wave == 0 ? 0u : (unsigned)__builtin_amdgcn_readlane((int)sums, wave - 1)) + incl - sum;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            sh.start[mine[i]] = at;
            at += in_cell[i];
        }
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const int e = q * kThreads + tid;
        if (e < n_f) {
            const unsigned row = sh.start[cell[q]] + within[q];
            sh.box[row] = b[q];
            sh.T[row] = nms_place_threshold<IOU>(((b[q].z - b[q].x) + off) * ((b[q].w - b[q].y) + off), test.boundary);
            sh.upper[row] = upper[q];
            sh.meta[row] = (unsigned)e | (cell[q] << 16) | (LABELS ? (unsigned)(label[q] & 0xf0) << 24 : 0u);
            atomicMin(&sh.best[A + 1 + cell[q]], (upper[q] & ~4095u) | row);
            if (LABELS) atomicOr(&sh.bins[row / kTile], 1u << nms_place_bin(label[q]));
            if (parts > 1) sh.row[e] = (uint16_t)row;
        }
    }
    const int tiles = (n_f + kTile - 1) / kTile;
    if (tid < tiles * kTile - n_f) {  // rows behind the last box: eliminate nothing
        sh.box[n_f + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
        sh.T[n_f + tid] = INFINITY;
        sh.upper[n_f + tid] = ~0u;
        sh.meta[n_f + tid] = 0u;
    }
    lds_barrier();
    const bool wide = LABELS && sh.wide != 0u;

    // ---- per tile: hull, smallest T, best rank; sixteen lanes share a tile
    {
        const int t = tid / 16;
        if (t < tiles) {  // (whole rows of sixteen lanes)
            float4 h = make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
            float least = INFINITY;
            unsigned best = ~0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = t * kTile + i * 16 + (lane & 15);
                const float4 v = sh.box[row];
                const unsigned u = sh.upper[row];
                nms_place_hull_add<IOU>(h, least, v, sh.T[row], row < n_f);
                best = u < best ? u : best;
            }
            h.x = row_min(h.x), h.y = row_min(h.y), h.z = row_min(h.z), h.w = row_min(h.w);
            least = row_min(least);
            best = row16_min(best);
            if ((lane & 15) == 15) {
                sh.hull[t] = make_float4(h.x, h.y, -h.z, -h.w);
                sh.tile[t] = make_uint2(__float_as_uint(least), best);
            }
        }
    }
    auto inter_with = [&](const float4 v, const float4 c) __attribute__((always_inline)) { return nms_place_inter(v, c, off); };
    auto area_of = [&](const float4 v) __attribute__((always_inline)) { return ((v.z - v.x) + off) * ((v.w - v.y) + off); };

    // A lane's victim against the boxes named in the cells of a line around it: `below` classes smaller, dy lines on (at the border of the
    // grid the cells of a neighbouring line: any box will do).  Scores equal in the upper 20 bits are left to the scan.
    struct LaneVictim {
        float4 box;
        float T, area;
        unsigned key, meta;
        int label;
    };
    auto lane_victim = [&](int row) __attribute__((always_inline)) {
        LaneVictim v;
        v.box = sh.box[row];
        v.key = sh.upper[row] & ~4095u;
        v.meta = sh.meta[row];
        v.T = IOU ? sh.T[row] : 0.0f;
        v.area = IOU ? area_of(v.box) : 0.0f;
        v.label = wide ? label_f[v.meta & 0xffffu] : 0;
        return v;
    };
    auto try_line = [&](const LaneVictim &v, bool &alive, int below, int dy) __attribute__((always_inline)) {
        const unsigned c = (v.meta >> 16) & 0xfffu;
        if (!alive || (below && c < (unsigned)(A * A))) return;
        const unsigned *at_line = sh.best + c + (A + 1 + A * dy - A * A * below);
        unsigned r[3];
        float4 cb[3];
        float cT[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) r[x] = at_line[x - 1];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            cb[x] = sh.box[r[x] & (P - 1)];  // (of an empty cell: whatever is there, it is ranked before nothing)
            cT[x] = sh.T[r[x] & (P - 1)];
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const float inter = inter_with(v.box, cb[x]);
            bool hit = inter >= (IOU ? fmaxf(cT[x], v.T) : cT[x]) && r[x] < v.key;
            if ((IOU || LABELS) && __ballot(hit) != 0) {
                asm volatile("" ::: "memory");  // keeps this a branch
                if (IOU) hit = hit && (double)inter >= test.boundary * (double)((v.area + area_of(cb[x])) - inter);
                if (LABELS) {
                    const unsigned cm = sh.meta[r[x] & (P - 1)];
                    hit = hit && ((cm ^ v.meta) & kSame) == 0;
                    if (wide && hit) hit = label_f[cm & 0xffffu] == v.label;
                }
            }
            alive = alive && !hit;
        }
    };
    auto try_lines = [&](const LaneVictim &v, bool &alive) __attribute__((always_inline)) {
#pragma unroll 1
        for (int below = 0; below < kLines / 3; ++below) {
#pragma unroll
            for (int y = 0; y < 3; ++y) try_line(v, alive, below, y == 2 ? -1 : y);
            if (__ballot(alive) == 0) break;
        }
    };
    // the lanes' rows go to a list of the workgroup
    auto append = [&](bool is, int row, uint16_t *list, unsigned *count) __attribute__((always_inline)) {
        const unsigned long long m = __ballot(is);
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(count, (unsigned)__builtin_popcountll(m));
        at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
        if (is) list[at + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = (uint16_t)row;
    };

    // ---- first stage: lane = victim
    // (one workgroup: 64 rows of the table; several: 64 neighbours of the input -- the order of rows inside a cell is each workgroup's own)
    const int split = 1 << split_log2;
    auto victim_row = [&](int t, bool &there) __attribute__((always_inline)) {
        const int e = t * kTile + lane;
        there = e < n_f;
        return parts == 1 ? (there ? e : n_f - 1) : (int)sh.row[there ? e : n_f - 1];
    };
#pragma unroll 1
    for (int t = part + parts * (wave >> split_log2); t < tiles; t += parts * W) {
        bool owned;
        const int row = victim_row(t, owned);
        const LaneVictim v = lane_victim(row);
        bool alive = owned;
        if (split_log2 == 0) {
            try_lines(v, alive);
        } else {
#pragma unroll 1
            for (int l = wave & (split - 1); l < kLines; l += split) {
                const int y = l >= 3 ? l - 3 : l;
                try_line(v, alive, l >= 3 ? 1 : 0, y == 2 ? -1 : y);
            }
            const unsigned long long gone = __ballot(owned && !alive);
            if (lane == 0 && gone != 0) atomicOr(&sh.dead[wave >> split_log2], gone);
            break;
        }
        append(alive, row, sh.list, &sh.listed);
        if (owned && !alive && parts > 1) keep_f[v.meta & 0xffffu] = 0;
    }
    lds_barrier();
    if (split_log2 > 0) {  // uniform; at most eight tiles of victims
        // what each tile's wavefronts found together; a wavefront's place in the list follows from all of it
        const int t_lane = lane & (kPlaceWaves - 1);
        const int in_tile = n_f - (part + t_lane * parts) * kTile;
        const unsigned long long there = in_tile >= kTile ? ~0ull : (in_tile > 0 ? (1ull << in_tile) - 1ull : 0ull);
        const unsigned sums = row16_inclusive_sum((unsigned)__builtin_popcountll(there & ~sh.dead[t_lane]));
        const int total = __builtin_amdgcn_readlane((int)sums, kPlaceWaves - 1);
        const int before = wave == 0 ? 0 : __builtin_amdgcn_readlane((int)sums, wave - 1);
        bool owned;
        const int row = victim_row(part + wave * parts, owned);
        if (owned) {
            const unsigned long long m = ~sh.dead[wave];
            if ((m >> lane) & 1ull)  // (what is not there lies behind the last lane that is)
                sh.list[before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = (uint16_t)row;
            else if (parts > 1)
                keep_f[sh.meta[row] & 0xffffu] = 0;
        }
        if (tid == 0) sh.listed = (unsigned)total;
    }
    if (split_log2 > 0) lds_barrier();

    // ---- second stage: the victims still alive, a group of neighbours at a time, lane = outranking box, the tiles that reach a victim
    const float4 th_hull = sh.hull[lane < tiles ? lane : 0];
    const uint2 th_tile = sh.tile[lane < tiles ? lane : 0];
    const unsigned th_bins = LABELS ? sh.bins[lane < tiles ? lane : 0] : 0u;
    const float tile_T = __uint_as_float(th_tile.x);
    constexpr int G = kPlaceGroup;
    float4 g_box[G];
    float g_T[G], g_area[G];
    unsigned g_upper[G], g_meta[G];
    int g_label[G];
    static_assert(G == 4, "a lane per member further down");
    {
        const int listed = (int)sh.listed;
        const int group = listed >= W * G ? G : (listed + W - 1) / W;  // (no wavefront idle while another has several)
#pragma unroll 1
        for (int i0 = wave * group; i0 < listed;) {  // the first group is the wavefront's own, the others are handed out through a counter
            int next = 0;
            if (lane == 0) next = W * group + (int)atomicAdd(&sh.next, (unsigned)group);
            const int members = listed - i0 < group ? listed - i0 : group;
            unsigned dead = 0;
            unsigned long long reach[G];  // tiles that reach victim u; none once it is settled
            unsigned long long left = 0;
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const unsigned row = sh.list[u < members ? i0 + u : i0];
                g_box[u] = sh.box[row];
                g_upper[u] = sh.upper[row];
                g_meta[u] = sh.meta[row];
                g_T[u] = IOU ? sh.T[row] : 0.0f;
                g_area[u] = IOU ? area_of(g_box[u]) : 0.0f;
                g_label[u] = wide ? label_f[g_meta[u] & 0xffffu] : 0;
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                reach[u] = 0;
                if (u < members) {
                    bool near = nms_place_reaches<IOU>(g_box[u], g_T[u], g_upper[u], th_hull, tile_T, th_tile.y, off);
                    if (LABELS) near = near && ((th_bins >> ((g_meta[u] >> 16) / (unsigned)(A * A) & (kPlaceBins - 1))) & 1u) != 0;
                    reach[u] = __ballot(near) & nms_place_tile_lanes(0, tiles);
                }
                left |= reach[u];
            }
            while (left != 0) {
                const int t0 = __builtin_ctzll(left);
                left &= left - 1;
                const int t1 = left != 0 ? __builtin_ctzll(left) : t0;
                left &= left - 1;  // (0 stays 0)
                const int r0 = t0 * kTile + lane, r1 = t1 * kTile + lane;
                const float4 c0 = sh.box[r0], c1 = sh.box[r1];
                const float T0 = sh.T[r0], T1 = sh.T[r1];
                const unsigned u0 = sh.upper[r0], u1 = sh.upper[r1];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    if ((((reach[u] >> t0) | (reach[u] >> t1)) & 1ull) != 0) {  // wave-uniform
                        const float i0 = inter_with(g_box[u], c0), i1 = inter_with(g_box[u], c1);
                        unsigned long long near0 = __ballot(i0 >= (IOU ? fmaxf(T0, g_T[u]) : T0)) & __ballot(u0 <= g_upper[u]);
                        unsigned long long near1 = __ballot(i1 >= (IOU ? fmaxf(T1, g_T[u]) : T1)) & __ballot(u1 <= g_upper[u]);
                        if ((near0 | near1) != 0) {
                            asm volatile("" ::: "memory");  // keeps this a branch
                            if (IOU) {
                                near0 &= __ballot((double)i0 >= test.boundary * (double)((g_area[u] + area_of(c0)) - i0));
                                near1 &= __ballot((double)i1 >= test.boundary * (double)((g_area[u] + area_of(c1)) - i1));
                            }
                            if (LABELS) {
                                const unsigned m0 = sh.meta[r0], m1 = sh.meta[r1];
                                near0 &= __ballot(((m0 ^ g_meta[u]) & kSame) == 0);
                                near1 &= __ballot(((m1 ^ g_meta[u]) & kSame) == 0);
                                if (wide) {
                                    near0 &= __ballot(((near0 >> lane) & 1ull) != 0 && label_f[m0 & 0xffffu] == g_label[u]);
                                    near1 &= __ballot(((near1 >> lane) & 1ull) != 0 && label_f[m1 & 0xffffu] == g_label[u]);
                                }
                            }
                            const unsigned long long before0 = __ballot(u0 < g_upper[u]), before1 = __ballot(u1 < g_upper[u]);
                            unsigned long long out0 = near0 & before0, out1 = near1 & before1;
                            // equal scores: the lower index is ranked first (the victim itself is not)
                            if (!test.ties_ignore && (out0 | out1) == 0) {
                                out0 |= near0 & ~before0 & __ballot((sh.meta[r0] & 0xffffu) < (g_meta[u] & 0xffffu));
                                out1 |= near1 & ~before1 & __ballot((sh.meta[r1] & 0xffffu) < (g_meta[u] & 0xffffu));
                            }
                            if ((out0 | out1) != 0) {
                                dead |= 1u << u;
                                reach[u] = 0;
                                left &= reach[0] | reach[1] | reach[2] | reach[3];
                            }
                        }
                    }
                }
            }
            if (lane < members) {
                const unsigned meta = lane == 0 ? g_meta[0] : (lane == 1 ? g_meta[1] : (lane == 2 ? g_meta[2] : g_meta[3]));
                const bool alive = ((dead >> lane) & 1u) == 0;
                if (parts > 1) {
                    keep_f[meta & 0xffffu] = alive ? 1 : 0;
                } else if (alive) {
                    sh.keep[meta & 0xffffu] = 1;
                }
            }
            i0 = __builtin_amdgcn_readfirstlane(next);
        }
    }
    if (parts == 1) {
        lds_barrier();
#pragma unroll
        for (int q = 0; q < E; ++q) {
            const int e = q * kThreads + tid;
            if (e < n_f) keep_f[e] = sh.keep[e];
        }
    }
}

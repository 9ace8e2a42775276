// Part of nms_kernels.hip (included there, inside its anonymous namespace): boxes in order of place in memory (long frames, and what the greedy rule and IoU need): the table, the scan of the tiles that reach a victim.
#pragma once

// ----------------------------------------------------------------------------- order of place, in memory

// What spatial_frames_kernel does in the LDS of one workgroup, for frames that do not fit there: one launch puts the boxes
// of a frame in order of place, in tiles of 64 rows, with the tiles' hulls, another tests the victims of a tile per workgroup.
// The table is built by several workgroups per frame, each of which counts the cells of the whole frame: what bounds
// a single frame is that they all read it (64 MB through L2 at 1 x 16,384 boxes, 10 k of 32 k cycles, the prefix sum 3 k, finding
// the share's boxes 8 k), what bounds a batch the pair tests.  Whole call, us, against rank order in two launches or with early
// exit: 1 x 16,384 crowd 20.1 / 36.1 (table 14, scan 6), 1 x 4200 15.0 / 21.7, 1 x 32,768 49 / 104, 4 x 16,384 26 / 85,
// 16 x 16,384 42 / 206, 64 ragged frames of 8192 62 / 162, 128 x 5000 78 / 166.
struct PlaceTable {
    float4 *box;         // [frames][n_pad]
    float *T;            // [frames][n_pad]        smallest intersection that may eliminate (see nms_place_threshold)
    unsigned *upper;     // [frames][n_pad]        upper half of the rank key
    unsigned *index;     // [frames][n_max]        input index
    int32_t *label;      // [frames][n_pad]        class labels, where the call has them
    float4 *hull;        // [frames][n_pad / 64]
    uint2 *tile;         // [frames][n_pad / 64]   smallest T, best (smallest) upper half
};

constexpr int kSortWaves = 16;
constexpr int kSortThreads = kSortWaves * 64;
constexpr int kSortAxis = 32;
constexpr int kSortCells = 4 * kSortAxis * kSortAxis;
constexpr int kSortShare = 1024;  // most places of a workgroup

struct PlaceSortShared {
    __align__(16) unsigned start[kSortCells + 1];  // boxes per cell, then the first place of each cell; the last: of no cell
    float4 box[kSortShare];
    unsigned index[kSortShare];
    unsigned wave_sum[kSortWaves];
    unsigned part_sum[2][kSortWaves];  // boxes of the first / last cell of the share, per wavefront
    unsigned edge[4];                  // first cell of the share and its first place, last cell and its first place
};

// Several workgroups per frame: each counts the cells of the whole frame (the boxes stay in registers up to 16,384 of
// them) and writes the places [lo, lo + share) of the table, share a multiple of 64.  Cells, their first places and the order
// inside the two cells that a share may cut depend on the input alone (numbered by wavefront, chunk, register, lane), so the
// workgroups agree without exchanging anything.  E: boxes per thread and chunk of 1024 E; MULTI: several chunks, read again in
// each pass.
template <int E, bool MULTI, bool IOU>
__global__ void __launch_bounds__(kSortThreads)
place_sort_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ counts,
                  int n_max, int n_pad, int share, PlaceTest test, PlaceTable tab, uint8_t *__restrict__ keep_out)
{
    __shared__ PlaceSortShared sh;
    constexpr int kSpan = kSortThreads * E;
    const int f = blockIdx.x;
    const int part = blockIdx.y, parts = gridDim.y;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    const float4 *box_f = reinterpret_cast<const float4 *>(boxes) + (size_t)f * n_max;
    const float *score_f = scores + (size_t)f * n_max;
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    for (int i = n_f + part * kSortThreads + tid; i < n_max; i += parts * kSortThreads) keep_f[i] = 0;
    const int lo = part * share;
    if (lo >= n_f) return;
    const int hi = lo + share < n_f ? lo + share : n_f;
    const int chunks = MULTI ? (n_f + kSpan - 1) / kSpan : 1;

    const float4 sample = box_f[(unsigned)(((long long)lane * n_f) >> 6)];
    float4 b[E];
    auto element = [&](int base, int q) __attribute__((always_inline)) { return base + q * kSortThreads + tid; };
    auto fetch_boxes = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < E; ++q) {
            int e = element(base, q);
            asm volatile("" : "+v"(e));
            b[q] = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(box_f) + 16u * (unsigned)(e < n_f ? e : 0));
        }
    };
    fetch_boxes(0);
    constexpr int kPer = kSortCells / kSortThreads;
    unsigned mine[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        mine[i] = curve_cell<kSortAxis>((unsigned)(kPer * tid + i));
        sh.start[i * kSortThreads + tid] = 0u;
    }
    if (tid == 0) sh.start[kSortCells] = ~0u;
    lds_barrier();
    PlaceGrid grid;
    {
        const float cx = sample.x + sample.z, cy = sample.y + sample.w;
        grid.x0 = wave_min(cx), grid.y0 = wave_min(cy);
        const float hx = wave_min(-cx), hy = wave_min(-cy);
        grid.sx = place_scale(grid.x0, -hx, (float)kSortAxis);
        grid.sy = place_scale(grid.y0, -hy, (float)kSortAxis);
    }

    // ---- boxes per cell
    constexpr unsigned kNoCell = kSortCells;
    unsigned cell[E];
#pragma unroll 1
    for (int k = 0; k < chunks; ++k) {
        const int base = k * kSpan;
        if (MULTI && k > 0) fetch_boxes(base);
#pragma unroll
        for (int q = 0; q < E; ++q) {
            cell[q] = element(base, q) < n_f ? place_cell<kSortAxis>(b[q], grid) : kNoCell;
            if (cell[q] != kNoCell) atomicAdd(&sh.start[cell[q]], 1u);
            // what the cell was worked out from is not kept: registers are what is short here
            asm volatile("" : "+v"(b[q].x), "+v"(b[q].y), "+v"(b[q].z), "+v"(b[q].w), "+v"(cell[q]));
        }
    }
    lds_barrier();

    // ---- first place of every cell; the cells that hold the share's first and last place
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
        const unsigned sums = row16_inclusive_sum(sh.wave_sum[lane & (kSortWaves - 1)]);
        unsigned at = (wave == 0 ? 0u : (unsigned)__builtin_amdgcn_readlane((int)sums, wave - 1)) + incl - sum;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const unsigned end = at + in_cell[i];
            sh.start[mine[i]] = at;
            if (at <= (unsigned)lo && (unsigned)lo < end) {
                sh.edge[0] = mine[i];
                sh.edge[1] = at;
            }
            if (at <= (unsigned)(hi - 1) && (unsigned)(hi - 1) < end) {
                sh.edge[2] = mine[i];
                sh.edge[3] = at;
            }
            at = end;
        }
    }
    lds_barrier();
    const unsigned cell_a = sh.edge[0], place_a = sh.edge[1], cell_z = sh.edge[2], place_z = sh.edge[3];

    // ---- boxes of the two border cells per wavefront
    {
        unsigned in_a = 0, in_z = 0;
#pragma unroll 1
        for (int k = 0; k < chunks; ++k) {
            const int base = k * kSpan;
            if (MULTI) fetch_boxes(base);
#pragma unroll
            for (int q = 0; q < E; ++q) {
                if (MULTI) cell[q] = element(base, q) < n_f ? place_cell<kSortAxis>(b[q], grid) : kNoCell;
                in_a += (unsigned)__builtin_popcountll(__ballot(cell[q] == cell_a));
                in_z += (unsigned)__builtin_popcountll(__ballot(cell[q] == cell_z));
            }
        }
        if (lane == 0) {
            sh.part_sum[0][wave] = in_a;
            sh.part_sum[1][wave] = in_z;
        }
    }
    lds_barrier();

    // ---- the boxes of the share
    {
        const unsigned sums_a = row16_inclusive_sum(sh.part_sum[0][lane & (kSortWaves - 1)]);
        const unsigned sums_z = row16_inclusive_sum(sh.part_sum[1][lane & (kSortWaves - 1)]);
        unsigned at_a = place_a + (wave == 0 ? 0u : (unsigned)__builtin_amdgcn_readlane((int)sums_a, wave - 1));
        unsigned at_z = place_z + (wave == 0 ? 0u : (unsigned)__builtin_amdgcn_readlane((int)sums_z, wave - 1));
#pragma unroll 1
        for (int k = 0; k < chunks; ++k) {
            const int base = k * kSpan;
            if (MULTI) fetch_boxes(base);
            unsigned first[E];
#pragma unroll
            for (int q = 0; q < E; ++q) {
                if (MULTI) cell[q] = element(base, q) < n_f ? place_cell<kSortAxis>(b[q], grid) : kNoCell;
                first[q] = sh.start[cell[q]];
            }
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const bool is_a = cell[q] == cell_a, is_z = cell[q] == cell_z;
                const bool inside = first[q] >= (unsigned)lo && first[q] < (unsigned)hi;
                if (__ballot(is_a || is_z || inside) == 0) continue;
                asm volatile("" ::: "memory");  // keeps this a branch: few wavefronts hold a box of the share
                const unsigned long long in_a = __ballot(is_a), in_z = __ballot(is_z);
                unsigned place = ~0u;
                if (is_a)
                    place = at_a + __builtin_amdgcn_mbcnt_hi((unsigned)(in_a >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in_a, 0u));
                else if (is_z)
                    place = at_z + __builtin_amdgcn_mbcnt_hi((unsigned)(in_z >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in_z, 0u));
                else if (inside)  // a cell inside the share counts its boxes up from its first place; the counter is below hi until the last of them
                    place = atomicAdd(&sh.start[cell[q]], 1u);
                at_a += (unsigned)__builtin_popcountll(in_a);
                at_z += (unsigned)__builtin_popcountll(in_z);
                if (place >= (unsigned)lo && place < (unsigned)hi) {
                    sh.box[place - lo] = b[q];
                    sh.index[place - lo] = (unsigned)element(base, q);
                }
            }
        }
    }
    lds_barrier();

    // ---- written out, a row per thread; sixteen lanes share a tile for its hull
    const int i = tid;                                              // share <= kSortThreads
    const int rows = (hi - lo + kTile - 1) / kTile * kTile;         // with the last tile's empty rows
    if (i < rows) {  // whole wavefronts
        const bool there = i < hi - lo;
        // (coordinates that are not finite: a box counted under one cell and placed under another would leave a place unwritten)
        const unsigned written = there ? sh.index[i] : 0u;
        const unsigned e = written < (unsigned)n_f ? written : 0u;
        const float score = score_f[e];
        const float4 v = there ? sh.box[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float area = ((v.z - v.x) + test.offset) * ((v.w - v.y) + test.offset);
        const float T = there ? nms_place_threshold<IOU>(area, test.boundary) : INFINITY;
        const unsigned upper = there ? (unsigned)(nms_rank_key(score, e) >> 32) : ~0u;
        const size_t at = (size_t)f * n_pad + lo + i;
        tab.box[at] = v;
        tab.T[at] = T;
        tab.upper[at] = upper;
        if (there) tab.index[(size_t)f * n_max + lo + i] = e;
        if (test.classes != nullptr) tab.label[at] = test.classes[(size_t)f * n_max + e];
        float4 h = make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
        float T_hull = INFINITY;
        nms_place_hull_add<true>(h, T_hull, v, T, there);
        const float hx = wave_min(h.x), hy = wave_min(h.y), hz = wave_min(h.z), hw = wave_min(h.w);
        const float least = wave_min(T_hull);
        unsigned best = row16_min(upper);  // in every lane of the row
        {
            const unsigned b0 = (unsigned)__builtin_amdgcn_readlane((int)best, 0), b1 = (unsigned)__builtin_amdgcn_readlane((int)best, 16);
            const unsigned b2 = (unsigned)__builtin_amdgcn_readlane((int)best, 32), b3 = (unsigned)__builtin_amdgcn_readlane((int)best, 48);
            const unsigned lo2 = b0 < b1 ? b0 : b1, hi2 = b2 < b3 ? b2 : b3;
            best = lo2 < hi2 ? lo2 : hi2;
        }
        if (lane == 0) {
            const size_t t = (size_t)f * (n_pad / kTile) + (lo + i) / kTile;
            tab.hull[t] = make_float4(hx, hy, -hz, -hw);
            tab.tile[t] = make_uint2(__float_as_uint(least), best);
        }
    }
}

// Value of another lane, wave-uniform.
__device__ __forceinline__ float lane_value(float x, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); }

// Where the boxes of a frame lie (PlaceTable at frame f).
struct PlaceFrame {
    const float4 *__restrict__ box;
    const float *__restrict__ T;
    const unsigned *__restrict__ upper;
    const unsigned *__restrict__ index;
    const int32_t *__restrict__ label;
    const float4 *__restrict__ hull;
    const uint2 *__restrict__ tile;
    int n, tiles;
};
__device__ __forceinline__ PlaceFrame place_frame(const PlaceTable &tab, int f, int n_f, int n_max, int n_pad)
{
    PlaceFrame p;
    p.box = tab.box + (size_t)f * n_pad;
    p.T = tab.T + (size_t)f * n_pad;
    p.upper = tab.upper + (size_t)f * n_pad;
    p.index = tab.index + (size_t)f * n_max;
    p.label = tab.label + (size_t)f * n_pad;
    p.hull = tab.hull + (size_t)f * (n_pad / kTile);
    p.tile = tab.tile + (size_t)f * (n_pad / kTile);
    p.n = n_f;
    p.tiles = (n_f + kTile - 1) / kTile;
    return p;
}

// A victim, wave-uniform.
struct PlaceVictim {
    float4 box;
    unsigned upper, index;
    float T, area;  // IOU
    int label, row;
};

// Lane mask of the boxes of a tile (rows r = 64 t + lane; c, T, u: the lane's) that are ranked before the victim and eliminate it.
template <bool IOU>
__device__ __forceinline__ unsigned long long place_eliminators(const PlaceFrame &p, const PlaceTest &test, const PlaceVictim &v, int r,
                                                                const float4 c, float T, unsigned u)
{
    const float inter = nms_place_inter(v.box, c, test.offset);
    unsigned long long near = __ballot(inter >= (IOU ? fmaxf(T, v.T) : T)) & __ballot(u <= v.upper);
    if (near == 0) return 0;
    asm volatile("" ::: "memory");  // keeps this a branch
    if (IOU) {
        const float area = ((c.z - c.x) + test.offset) * ((c.w - c.y) + test.offset);
        near &= __ballot((double)inter >= test.boundary * (double)((v.area + area) - inter));
    }
    if (test.classes != nullptr && near != 0) near &= __ballot(p.label[r] == v.label);
    const unsigned long long before = __ballot(u < v.upper);
    const unsigned long long tied = near & ~before & ~__ballot(r == v.row);
    near &= before;
    if (tied != 0 && !test.ties_ignore)  // equal scores: the lower index is ranked first
        near |= tied & __ballot(p.index[r < p.n ? r : 0] < v.index);
    return near;
}

// What a group of victims is tested against: the tiles that reach one of them, 256 tiles at a time, two tiles' boxes in flight together.
// found(u, t, mask): victim u of the group has eliminators `mask` (not 0) in tile t; returns whether that settles it.
template <bool IOU, class Found>
__device__ __forceinline__ void place_scan_group(const PlaceFrame &p, const PlaceTest &test, const PlaceVictim (&v)[kPlaceGroup], int members,
                                                 int lane, Found found)
{
    constexpr int G = kPlaceGroup, C = 2;
    unsigned settled = 0;
#pragma unroll 1
    for (int s = 0; s < p.tiles; s += C * kTile) {
        unsigned long long reach[C][G];
        {
            float4 h[C];
            uint2 hi[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int t = s + c * kTile + lane;
                h[c] = p.hull[t < p.tiles ? t : p.tiles - 1];
                hi[c] = p.tile[t < p.tiles ? t : p.tiles - 1];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    reach[c][u] = 0;
                    if (u < members && ((settled >> u) & 1u) == 0)
                        reach[c][u] = __ballot(nms_place_reaches<IOU>(s + c * kTile + lane, p.tiles, v[u].box, v[u].T, v[u].upper, h[c],
                                                                      __uint_as_float(hi[c].x), hi[c].y, test.offset));
                }
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            unsigned long long left = 0;
#pragma unroll
            for (int u = 0; u < G; ++u) left |= reach[c][u];
#pragma unroll 1
            while (left != 0) {
                constexpr int K = 2;
                int t[K];
                float4 b[K];
                float T[K];
                unsigned up[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    t[k] = left != 0 ? __builtin_ctzll(left) : -1;
                    left &= left - 1;  // (0 stays 0)
                    const int r = (s + c * kTile + (t[k] < 0 ? t[0] : t[k])) * kTile + lane;
                    b[k] = p.box[r];
                    T[k] = p.T[r];
                    up[k] = p.upper[r];
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (t[k] < 0) break;
                    const int tile = s + c * kTile + t[k];
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        if (((reach[c][u] >> t[k]) & 1ull) == 0) continue;  // wave-uniform
                        const unsigned long long m = place_eliminators<IOU>(p, test, v[u], tile * kTile + lane, b[k], T[k], up[k]);
                        if (m != 0 && found(u, tile, m)) {
                            settled |= 1u << u;
                            reach[c][u] = 0;
                            left &= reach[c][0] | reach[c][1] | reach[c][2] | reach[c][3];
                        }
                    }
                }
            }
        }
    }
}

// The paper's rule from the table: a victim survives unless some better-ranked box eliminates it.  A workgroup of W wavefronts
// per tile of victims: first the tile's own boxes (lane = victim; neighbours are what eliminates most), then the victims left,
// up to four at a time, lane = outranking box, against the tiles that reach them.
template <int W, bool IOU>
__global__ void __launch_bounds__(W * 64)
place_scan_kernel(const int32_t *__restrict__ counts, int n_max, int n_pad, PlaceTest test, PlaceTable tab,
                  uint8_t *__restrict__ keep_out)
{
    __shared__ unsigned long long dead_s;
    const int f = blockIdx.x;
    const int t = blockIdx.y;
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_f = frame_count(counts, f, n_max);
    if (t * kTile >= n_f) return;
    const PlaceFrame p = place_frame(tab, f, n_f, n_max, n_pad);
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const bool labelled = test.classes != nullptr;

    if (threadIdx.x == 0) dead_s = 0ull;
    const int row = t * kTile + lane;
    const bool there = row < n_f;
    const float4 mine = p.box[row];
    const float mine_T = p.T[row];
    const unsigned mine_upper = p.upper[row];
    const unsigned mine_index = p.index[there ? row : n_f - 1];
    const int mine_label = labelled ? p.label[row] : 0;
    const float mine_area = ((mine.z - mine.x) + test.offset) * ((mine.w - mine.y) + test.offset);
    lds_barrier();

    // ---- the tile's own boxes
    {
        unsigned long long gone = 0;
#pragma unroll 2
        for (int i = 0; i < kTile / W; ++i) {
            const int k = wave + W * i;
            const float4 c = make_float4(lane_value(mine.x, k), lane_value(mine.y, k), lane_value(mine.z, k), lane_value(mine.w, k));
            const float inter = nms_place_inter(mine, c, test.offset);
            unsigned long long hit = __ballot(inter >= (IOU ? fmaxf(lane_value(mine_T, k), mine_T) : lane_value(mine_T, k)));
            hit &= __ballot((unsigned)__builtin_amdgcn_readlane((int)mine_upper, k) < mine_upper);  // (equal scores: below)
            if (labelled) hit &= __ballot(__builtin_amdgcn_readlane(mine_label, k) == mine_label);
            if (IOU && (hit & ~gone) != 0) hit &= __ballot((double)inter >= test.boundary * (double)((mine_area + lane_value(mine_area, k)) - inter));
            gone |= hit;
        }
        if (lane == 0 && gone != 0) atomicOr(&dead_s, gone);
    }
    lds_barrier();
    const unsigned long long alive = ~dead_s & __ballot(there);
    if (wave == 0 && there && !((alive >> lane) & 1ull)) keep_f[mine_index] = 0;

    // ---- the victims left; this wavefront's: every W-th group of them
    const unsigned nth = __builtin_amdgcn_mbcnt_hi((unsigned)(alive >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)alive, 0u));
    constexpr int G = kPlaceGroup;
    const int left = __builtin_popcountll(alive);
    const int group = left >= W * G ? G : (left > W ? 2 : 1);
    unsigned long long todo = __ballot(((alive >> lane) & 1ull) != 0 && (int)(nth / (unsigned)(group == G ? G : 1) / (unsigned)(group == 2 ? 2 : 1)) % W == wave);
    while (todo != 0) {
        PlaceVictim v[G];
        int members = 0;
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const bool is = todo != 0 && u < group;
            const int at = todo != 0 ? __builtin_ctzll(todo) : 0;
            if (is) {
                todo &= todo - 1;
                ++members;
            }
            v[u].box = make_float4(lane_value(mine.x, at), lane_value(mine.y, at), lane_value(mine.z, at), lane_value(mine.w, at));
            v[u].upper = (unsigned)__builtin_amdgcn_readlane((int)mine_upper, at);
            v[u].index = (unsigned)__builtin_amdgcn_readlane((int)mine_index, at);
            v[u].T = lane_value(mine_T, at);
            v[u].area = lane_value(mine_area, at);
            v[u].label = __builtin_amdgcn_readlane(mine_label, at);
            v[u].row = t * kTile + at;
        }
        unsigned dead = 0;
        place_scan_group<IOU>(p, test, v, members, lane, [&](int u, int, unsigned long long) __attribute__((always_inline)) {
            dead |= 1u << u;
            return true;
        });
        if (lane < members) {
            unsigned e = v[0].index;
#pragma unroll
            for (int u = 1; u < G; ++u) e = lane == u ? v[u].index : e;
            keep_f[e] = ((dead >> lane) & 1u) != 0 ? 0 : 1;
        }
    }
}

// ----------------------------------------------------------------------------- greedy rule in order of place

// The sequential rule needs, for every box, the better-ranked boxes that would eliminate it.  Under IoU these are few
// (1.3 per box on anchors, 8 on clustered detections), and in order of place they lie in one to six tiles: a launch writes them
// down per row, as lane masks with their tiles, and another settles the rows of a frame.  One frame of 4096 clustered boxes: table
// 8 us, relation 7.6, resolve 10.4 (which one workgroup does: its loads and the rounds), 27.5 for the call against 36.0 with
// ranks, mask and sweep.
//
// Per row: the first kRelationWords masks and a byte each for their tiles (bit 7 of the last: there are more), the further
// masks behind those of all rows, in the order of the tiles named in `summary` (a bit per tile, S words).
constexpr int kRelationWords = 4;

struct PlaceRelation {
    unsigned long long *first;    // [frames][n_pad][kRelationWords]; 0: none
    unsigned long long *further;  // [frames][n_pad][n_pad / 64 - kRelationWords]
    unsigned *at;                 // [frames][n_pad]
    unsigned long long *summary;  // [frames][n_pad][S]
    int S;
};

// W wavefronts per tile of victims (M of them in a group), parts workgroups per tile.  The masks of a victim are collected in the lanes
// of a register and stored together: a store per mask would have every load of the next tiles wait for it.
template <int W, int M>
__global__ void __launch_bounds__(W * 64)
place_relation_kernel(const int32_t *__restrict__ counts, int n_max, int n_pad, int parts_log2, PlaceTest test, PlaceTable tab, PlaceRelation rel)
{
    const int f = blockIdx.x;
    const int t = blockIdx.y >> parts_log2, part = blockIdx.y & ((1 << parts_log2) - 1);
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_f = frame_count(counts, f, n_max);
    if (t * kTile >= n_f) return;
    const PlaceFrame p = place_frame(tab, f, n_f, n_max, n_pad);
    const bool labelled = test.classes != nullptr;
    const int T = n_pad / kTile;
    const int row = t * kTile + lane;
    const bool there = row < n_f;
    const float4 mine = p.box[row];
    const float mine_T = p.T[row];
    const unsigned mine_upper = p.upper[row];
    const unsigned mine_index = p.index[there ? row : n_f - 1];
    const int mine_label = labelled ? p.label[row] : 0;
    const float mine_area = ((mine.z - mine.x) + test.offset) * ((mine.w - mine.y) + test.offset);
    constexpr int G = kPlaceGroup;
#pragma unroll 1
    for (int i0 = (part * W + wave) * M; i0 < kTile; i0 += (W << parts_log2) * M) {
        const int r0 = t * kTile + i0;
        if (r0 >= n_f) break;
        const int members = n_f - r0 < M ? n_f - r0 : M;
        PlaceVictim v[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int at = i0 + (u < M ? u : 0);
            v[u].box = make_float4(lane_value(mine.x, at), lane_value(mine.y, at), lane_value(mine.z, at), lane_value(mine.w, at));
            v[u].upper = (unsigned)__builtin_amdgcn_readlane((int)mine_upper, at);
            v[u].index = (unsigned)__builtin_amdgcn_readlane((int)mine_index, at);
            v[u].T = lane_value(mine_T, at);
            v[u].area = lane_value(mine_area, at);
            v[u].label = __builtin_amdgcn_readlane(mine_label, at);
            v[u].row = t * kTile + at;
        }
        unsigned long long sum[2][G] = {};
        int found[G] = {};
        unsigned w_lo[G] = {}, w_hi[G] = {}, tiles_of[G] = {};
        unsigned long long *further_f = rel.further + ((size_t)f * n_pad + r0) * (size_t)(T > kRelationWords ? T - kRelationWords : 0);
        place_scan_group<true>(p, test, v, members, lane, [&](int u, int tile, unsigned long long m) __attribute__((always_inline)) {
            if (tile < kTile) sum[0][u] |= 1ull << tile;
            else sum[1][u] |= 1ull << (tile - kTile);
            const int k = found[u]++;
            if (k < kRelationWords) {
                const bool here = lane == k;
                w_lo[u] = here ? (unsigned)m : w_lo[u];
                w_hi[u] = here ? (unsigned)(m >> 32) : w_hi[u];
                tiles_of[u] |= (unsigned)tile << (8 * k);
            } else {
                tiles_of[u] |= 0x80000000u;
                if (lane == 0) further_f[(size_t)u * (T - kRelationWords) + k - kRelationWords] = m;
            }
            return false;
        });
#pragma unroll
        for (int u = 0; u < M; ++u)
            if (u < members && lane < kRelationWords)
                rel.first[((size_t)f * n_pad + r0 + u) * kRelationWords + lane] = ((unsigned long long)w_hi[u] << 32) | w_lo[u];
        if (lane < members) {
            unsigned long long w0 = sum[0][0], w1 = sum[1][0];
            unsigned at = tiles_of[0];
#pragma unroll
            for (int u = 1; u < M; ++u) {
                w0 = lane == u ? sum[0][u] : w0;
                w1 = lane == u ? sum[1][u] : w1;
                at = lane == u ? tiles_of[u] : at;
            }
            const size_t r = (size_t)f * n_pad + r0 + lane;
            rel.at[r] = at;
            rel.summary[r * rel.S] = w0;
            if (rel.S > 1) rel.summary[r * rel.S + 1] = w1;
        }
    }
}

// A row without eliminators is kept; of the others a row with a kept eliminator is out, a row none of whose eliminators is kept or
// open is kept, until no row is open.  A workgroup per frame, R tiles of 64 rows per wavefront (frames of at most 1024 R boxes),
// lane = row; the states of the tiles are words in LDS.  A wavefront looks at its open rows, again while that settles some;
// the best-ranked open row of the frame has no open eliminator, so something is settled between any two barriers, and the rounds end.
constexpr int kResolveWaves = 16;

template <int R>
__global__ void __launch_bounds__(kResolveWaves * 64)
place_resolve_kernel(const int32_t *__restrict__ counts, int n_max, int n_pad, const unsigned *__restrict__ index, PlaceRelation rel,
                     uint8_t *__restrict__ keep_out)
{
    constexpr int kTiles = kResolveWaves * R, K = kRelationWords;
    __shared__ unsigned long long open_s[kTiles], kept_s[kTiles];
    const int f = blockIdx.x;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    if (n_f == 0) return;
    const int T = n_pad / kTile;

    unsigned long long word[R][K];
    unsigned at[R], index_of[R];
    unsigned long long open[R], kept[R];  // wave-uniform: the state of the tile
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = (wave + kResolveWaves * i) * kTile + lane;
        const size_t r = (size_t)f * n_pad + (row < n_f ? row : 0);
        const ulonglong2 *w = reinterpret_cast<const ulonglong2 *>(rel.first + r * K);
        const ulonglong2 a = w[0], b = w[1];
        word[i][0] = a.x, word[i][1] = a.y, word[i][2] = b.x, word[i][3] = b.y;
        at[i] = rel.at[r];
        index_of[i] = index[(size_t)f * n_max + (row < n_f ? row : 0)];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int t = wave + kResolveWaves * i;
        const bool there = t * kTile + lane < n_f;
        open[i] = __ballot(there && (word[i][0] | word[i][1] | word[i][2] | word[i][3]) != 0);
        kept[i] = __ballot(there) & ~open[i];
        if (lane == 0) {
            open_s[t] = open[i];
            kept_s[t] = kept[i];
        }
    }
    __syncthreads();
    auto load = [&](const unsigned long long *p) __attribute__((always_inline)) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    for (;;) {
        bool any;
        for (int pass = 0; pass < 8; ++pass) {  // (the bound only lets the others' results in through a barrier now and then)
            bool settled = false;
            any = false;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (open[i] == 0) continue;  // wave-uniform
                const int t = wave + kResolveWaves * i;
                const bool mine = (open[i] >> lane) & 1ull;
                unsigned long long is_open = 0ull, is_out = 0ull;
                if (mine) {
                    // open is read before kept, and written after it: a row that is no longer open by then has its kept bit
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (word[i][k] != 0) is_open |= word[i][k] & load(&open_s[(at[i] >> (8 * k)) & 127u]);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (word[i][k] != 0) is_out |= word[i][k] & load(&kept_s[(at[i] >> (8 * k)) & 127u]);
                    if ((at[i] >> 31) != 0 && is_out == 0 && is_open == 0) {  // further masks
                        const size_t r = (size_t)f * n_pad + t * kTile + lane;
                        const unsigned long long *more = rel.further + r * (size_t)(T - K);
                        int k = 0;
                        for (int half = 0; half < rel.S; ++half) {
                            unsigned long long s = rel.summary[r * rel.S + half];
                            while (s != 0 && is_out == 0) {
                                const int tt = __builtin_ctzll(s) + kTile * half;
                                s &= s - 1;
                                if (k >= K) {
                                    const unsigned long long w = more[k - K];
                                    is_open |= w & load(&open_s[tt]);
                                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                                    is_out |= w & load(&kept_s[tt]);
                                }
                                ++k;
                            }
                        }
                    }
                }
                const unsigned long long now_out = __ballot(mine && is_out != 0);
                const unsigned long long now_kept = __ballot(mine && is_out == 0 && is_open == 0);
                if ((now_out | now_kept) != 0) {
                    settled = true;
                    kept[i] |= now_kept;
                    open[i] &= ~(now_out | now_kept);
                    if (lane == 0) {
                        __hip_atomic_store(&kept_s[t], kept[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __hip_atomic_store(&open_s[t], open[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
                any = any || open[i] != 0;
            }
            if (!settled) break;
        }
        if (__syncthreads_or(any ? 1 : 0) == 0) break;
    }
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int row = (wave + kResolveWaves * i) * kTile + lane;
        if (row < n_f) keep_f[index_of[i]] = (uint8_t)((kept[i] >> lane) & 1ull);
    }
}

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
// each pass.  GREEDY: for the relation launch.  With E = 16 boxes, cells and first places are 96 of the 128 registers that
// sixteen wavefronts leave each; the MULTI form (frames beyond 16,384 boxes) spills 13 (56 bytes a lane) and takes 1 x 32,768 in 49 us (104 before).
template <int E, bool MULTI, bool IOU, bool GREEDY>
__global__ void __launch_bounds__(kSortThreads)
place_sort_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ counts,
                  int n_max, int n_pad, int share, PlaceTest test, PlaceTable tab, unsigned *__restrict__ crowded, uint8_t *__restrict__ keep_out)
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
    // (coordinates that are not finite: a box counted under one cell and placed under another would leave a place unwritten)
    static_assert(kSortShare == kSortThreads, "a place per thread");
    sh.index[tid] = 0u;
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
        const unsigned e = there ? sh.index[i] : 0u;
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
        nms_place_hull_add<IOU>(h, T_hull, v, T, there);
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
            if (GREEDY && lo + i == 0) crowded[f] = 0u;  // (for the relation launch; where it is not wanted even the branch costs 2 %)
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

// What a group of victims is tested against: the tiles that reach one of them, 128 tiles at a time, K tiles' boxes in flight together.
// found(u, t, mask): victim u of the group has eliminators `mask` (not 0) in tile t; returns whether that settles it.
// many(u, k): k tiles of the 128 at hand reach victim u; returns whether that settles it.
template <bool IOU, int K, class Many, class Found>
__device__ __forceinline__ void place_scan_group(const PlaceFrame &p, const PlaceTest &test, const PlaceVictim (&v)[kPlaceGroup], int members,
                                                 int lane, Many many, Found found)
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
                const unsigned long long lanes = s + c * kTile < p.tiles ? nms_place_tile_lanes(s + c * kTile, p.tiles) : 0ull;
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    reach[c][u] = 0;
                    if (u < members && ((settled >> u) & 1u) == 0)
                        reach[c][u] = __ballot(nms_place_reaches<IOU>(v[u].box, v[u].T, v[u].upper, h[c], __uint_as_float(hi[c].x), hi[c].y, test.offset)) & lanes;
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                int k = 0;
#pragma unroll
                for (int c = 0; c < C; ++c) k += __builtin_popcountll(reach[c][u]);
                if (k != 0 && many(u, k)) {  // wave-uniform
                    settled |= 1u << u;
#pragma unroll
                    for (int c = 0; c < C; ++c) reach[c][u] = 0;
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
        place_scan_group<IOU, 2>(
            p, test, v, members, lane, [](int, int) __attribute__((always_inline)) { return false; },
            [&](int u, int, unsigned long long) __attribute__((always_inline)) {
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

// The sequential rule needs, for every box, the better-ranked boxes that would eliminate it.  Under IoU these are mostly few
// (1.3 per box on anchors, 8 on clustered detections), and in order of place they lie in one to six tiles: a launch writes them
// down per row, as lane masks with their tiles, and another settles the rows of a frame.  Where thousands of candidates crowd
// around few objects a row has them in dozens of tiles; such a crowded row keeps the first kRelationMasks masks only, so that the
// relation stays bounded, and what then cannot be settled from masks is walked in rank order.
//
// A row's masks lie as nms_relation_block says (columns, so that the lanes of a tile read one together); a byte each for their tiles.
// A victim that more than kCrowdedReach tiles reach and that kCrowdedTile of its own tile's boxes overlap far enough is crowded without a look at
// them all: clusters are reached by six tiles, and what many tiles reach without such neighbours (boxes of very different sizes) has few eliminators.
constexpr int kCrowdedReach = 20, kCrowdedTile = 16;
constexpr int kSampleTiles = 16;
constexpr unsigned kRowCrowded = 0x80u;   // of PlaceRelation::at[].x: the row has more masks than are kept
constexpr unsigned kRowMore = 0x8000u;    // of the same: masks behind the first four
constexpr unsigned kNoTile = 0x80u;       // of the bytes behind the first four: no mask

struct PlaceRelation {
    unsigned long long *words;  // [frames] blocks of n_pad / 64 * n_pad words
    uint4 *at;                  // [frames][n_pad]
    unsigned *crowded;          // [frames] crowded ones of the rows that are sampled: the first wavefront's in each of the first kSampleTiles tiles
    int32_t *left;              // [frames] boxes of the frames that the rounds have left open (0: settled), frames beyond NMS_SORT_CHUNK boxes
};

// W wavefronts per tile of victims (M of them in a group), parts workgroups per tile.  The masks of a victim are collected in the lanes
// of a register and stored together: a store per mask would have every load of the next tiles wait for it.  In large batches (M = 4), whose
// workgroups come one after the other, the tiles still to come are not related at all once half of the rows sampled
// are crowded: the frame will be walked.  (A count of all crowded rows is 4096 atomics on one address, 45 us.)
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
    const unsigned crowded_rows = __hip_atomic_load(rel.crowded + f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float4 mine = p.box[row];
    const float mine_T = p.T[row];
    const unsigned mine_upper = p.upper[row];
    const unsigned mine_index = p.index[there ? row : n_f - 1];
    const int mine_label = labelled ? p.label[row] : 0;
    const float mine_area = ((mine.z - mine.x) + test.offset) * ((mine.w - mine.y) + test.offset);
    const bool skip = M == 4 && __builtin_amdgcn_readfirstlane((int)crowded_rows) > kSampleTiles * M / 2;
    unsigned long long *first_f = rel.words + (size_t)f * T * n_pad;
    unsigned long long *more_f = first_f + nms_relation_block(n_pad).more;
    constexpr int G = kPlaceGroup;
    unsigned crowded_here = 0;
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
        int found[G] = {};
        unsigned w_lo[G] = {}, w_hi[G] = {}, tile_of[G];
#pragma unroll
        for (int u = 0; u < G; ++u) tile_of[u] = lane < kRelationWords ? 0u : kNoTile;
        unsigned crowded = skip ? (1u << G) - 1u : 0u;
        if (!skip) {
            // a victim that many tiles reach and that a quarter of its own tile would eliminate or be eliminated by: crowded, without a look at them all
            auto many = [&](int u, int k) __attribute__((always_inline)) {
                if (k <= kCrowdedReach) return false;
                asm volatile("" ::: "memory");  // keeps this a branch
                const float inter = nms_place_inter(v[u].box, mine, test.offset);
                unsigned long long near = __ballot(inter >= fmaxf(mine_T, v[u].T)) & __ballot((double)inter >= test.boundary * (double)((v[u].area + mine_area) - inter));
                if (labelled) near &= __ballot(mine_label == v[u].label);
                if (__builtin_popcountll(near) < kCrowdedTile) return false;
                crowded |= 1u << u;
                return true;
            };
            place_scan_group<true, M == 4 ? 2 : 4>(p, test, v, members, lane, many, [&](int u, int tile, unsigned long long m) __attribute__((always_inline)) {
                const int k = found[u]++;
                if (k == kRelationMasks) {
                    crowded |= 1u << u;
                    return true;
                }
                const bool here = lane == k;
                w_lo[u] = here ? (unsigned)m : w_lo[u];
                w_hi[u] = here ? (unsigned)(m >> 32) : w_hi[u];
                tile_of[u] = here ? (unsigned)tile : tile_of[u];
                return false;
            });
        }
#pragma unroll
        for (int u = 0; u < M; ++u) {
            if (u < members) {
                const size_t r = (size_t)(r0 + u);
                const unsigned long long w = ((unsigned long long)w_hi[u] << 32) | w_lo[u];
                if (lane < kRelationWords)
                    first_f[r * kRelationWords + lane] = w;
                else if (lane < kRelationMasks && lane < found[u])
                    more_f[(size_t)(lane - kRelationWords) * n_pad + r] = w;
                // four bytes to a word, in the first lane of each four
                unsigned at = tile_of[u] << (8 * (lane & 3));
                at |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)at, 0xb1, 0xf, 0xf, true);  // quad_perm: neighbour
                at |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)at, 0x4e, 0xf, 0xf, true);  // quad_perm: the other pair
                if (lane == 0) {
                    at |= found[u] > kRelationWords ? kRowMore : 0u;
                    if (((crowded >> u) & 1u) != 0) {
                        at |= kRowCrowded;
                        ++crowded_here;
                    }
                }
                if (lane < kRelationMasks && (lane & 3) == 0) reinterpret_cast<unsigned *>(rel.at + (size_t)f * n_pad + r)[lane >> 2] = at;
            }
        }
    }
    if (M == 4 && t < kSampleTiles && wave == 0 && lane == 0 && crowded_here != 0)
        __hip_atomic_fetch_add(rel.crowded + f, crowded_here, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A row without eliminators is kept; of the others a row with a kept eliminator is out, a row all of whose eliminators are out
// is kept, until no row is open or none can be settled any more.  A workgroup per frame, lane = row, up to R neighbouring tiles
// per wavefront (frames of at most 1024 R boxes): chains of eliminators run between neighbours, so that they run inside a wavefront,
// and inside a tile in registers.  The states of the tiles are words in LDS that only ever gain bits: a word read
// late leaves rows open longer and does no harm.  A round ends with a barrier; a round in which nothing was settled is the last one, so
// there are at most as many rounds as rows.
//
// Crowded rows, whose masks are not all there, are not settled here.  What is left open in the end (and what the rounds have not
// settled after kResolveRounds: long chains across wavefronts) is, WALK, put in rank order together with the kept rows that may touch it, and walked
// as in greedy_fused_kernel, by the same workgroup; beyond NMS_SORT_CHUNK boxes the frame is left to the general kernels (rel.left).
//
// What bounds it is one workgroup's chain: loads 3 us, rounds 8 (four to five passes over the rows, issue), stores 1 (1 x 4096 clustered: table 8,
// relation 6, resolve 12; the walk of one object's candidates 25 more: sort 12, ranked rows 3, walk 7).  With the masks in LDS instead of registers and the
// tiles in a loop 16 instead of 12; with the state of three masks or more behind a branch 13.  Frames beyond NMS_SORT_CHUNK boxes spill 12 vector registers.
// The whole call against rank, mask and sweep: nms_use_place_greedy.
constexpr int kResolveWaves = 16;
constexpr int kResolvePasses = 8;    // of a wavefront over its tiles in a round
constexpr int kResolveRounds = 128;  // (in frames with crowded rows kCrowdedRounds: what waits for those settles one by one)
constexpr int kCrowdedRounds = 4;

struct ResolveSort {  // rows in input order, then sorted
    unsigned long long keys[NMS_SORT_CHUNK];
    __align__(16) unsigned hist[kResolveWaves * 256];
    __align__(16) unsigned wbase[kResolveWaves * 256];
    __align__(16) unsigned tot[256];
    unsigned long long match[kResolveWaves * 512];
    unsigned long long bits[kTile];  // by input index: rows of the walk
    unsigned before[kTile];          // of them before each word
};

template <int R, bool AUX, bool WALK>
__global__ void __launch_bounds__(kResolveWaves * 64)
place_resolve_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ counts, int n_max, int n_pad,
                     PlaceTest test, PlaceTable tab, PlaceRelation rel, uint8_t *__restrict__ keep_out)
{
    constexpr int K = kRelationWords, kMore = kRelationMasks - kRelationWords;
    static_assert(!WALK || R * kResolveWaves * kTile == NMS_SORT_CHUNK, "the walk takes frames of one chunk");
    using Walk = WalkShared<kFusedWaves, NMS_SORT_CHUNK>;
    // (the states by themselves: through a reference into the walk's bytes the compiler would reach them by flat loads)
    struct States {
        unsigned long long kept[kResolveWaves * R], out[kResolveWaves * R];
    };
    __shared__ States st_s;
    __shared__ uint16_t index_s[kResolveWaves * 64 * R];  // of the lane's row i: there are no registers for it
    __shared__ unsigned news_s[3];  // of a round: bit 0: something was settled, bit 1: something is open, bit 2: there are crowded rows
    __shared__ __align__(16) unsigned char raw[WALK ? (sizeof(ResolveSort) > sizeof(Walk) ? sizeof(ResolveSort) : sizeof(Walk)) : 16];
    const int f = blockIdx.x;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    if (!WALK && tid == 0) rel.left[f] = 0;
    if (n_f == 0) return;
    const int T = n_pad / kTile;
    const int tiles = (n_f + kTile - 1) / kTile;
    const int per = (tiles + kResolveWaves - 1) / kResolveWaves;  // tiles of a wavefront, <= R
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const unsigned *index_f = tab.index + (size_t)f * n_max;
    const unsigned long long *first_f = rel.words + (size_t)f * T * n_pad;
    const unsigned long long *more_f = first_f + nms_relation_block(n_pad).more;
    const uint4 *at_f = rel.at + (size_t)f * n_pad;

    unsigned long long word[R][K], own[R];  // masks in other tiles, in the row's own
    unsigned at[R];
    unsigned long long open[R], kept[R], crowd[R];  // wave-uniform: the state of the tile; its crowded rows
    auto row_of = [&](int i) __attribute__((always_inline)) { return (wave * per + i) * kTile + lane; };
    auto index_of = [&](int i) __attribute__((always_inline)) { return (unsigned)index_s[i * kResolveWaves * 64 + tid]; };
    auto has = [&](int i) __attribute__((always_inline)) { return i < per && row_of(i) < n_f; };
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const size_t r = has(i) ? (size_t)row_of(i) : 0;
        const ulonglong2 *w = reinterpret_cast<const ulonglong2 *>(first_f + r * K);
        const ulonglong2 a = w[0], b = w[1];
        word[i][0] = a.x, word[i][1] = a.y, word[i][2] = b.x, word[i][3] = b.y;
        at[i] = reinterpret_cast<const unsigned *>(at_f + r)[0];
        index_s[i * kResolveWaves * 64 + tid] = (uint16_t)index_f[r];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int t = wave * per + i;
        const bool there = has(i);
        const unsigned long long rows = __ballot(there);
        crowd[i] = __ballot(there && (at[i] & kRowCrowded) != 0);
        open[i] = __ballot(there && (word[i][0] | word[i][1] | word[i][2] | word[i][3]) != 0) | crowd[i];
        kept[i] = rows & ~open[i];
        own[i] = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool is_own = ((at[i] >> (8 * k)) & 127u) == (unsigned)t;
            own[i] |= is_own ? word[i][k] : 0ull;
            word[i][k] = is_own ? 0ull : word[i][k];
        }
        if (lane == 0 && i < per && t < tiles) {
            st_s.kept[t] = kept[i];
            st_s.out[t] = ~rows;
        }
    }
    if (tid < 3) news_s[tid] = 0u;
    lds_barrier();
    struct State {
        unsigned long long kept, out;
    };
    auto state = [&](unsigned tile) __attribute__((always_inline)) {
        return State{__hip_atomic_load(&st_s.kept[tile], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP),
                     __hip_atomic_load(&st_s.out[tile], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)};
    };
    auto scalar = [&](unsigned long long x) __attribute__((always_inline)) {
        return ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((int)x);
    };
    bool open_left = false;
#pragma unroll 1
    for (int round = 0;; ++round) {
        unsigned news = 0;
#pragma unroll 1
        for (int pass = 0; pass < kResolvePasses; ++pass) {  // (the bound lets the others' results in through a barrier now and then)
            bool settled = false;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                if (scalar(open[i] & ~crowd[i]) == 0) continue;
                const int t = wave * per + i;
                const bool mine = ((open[i] & ~crowd[i]) >> lane) & 1ull;
                unsigned long long is_out = 0, is_open = 0;
                {
                    unsigned tiles_of = at[i];
                    asm volatile("" : "+v"(tiles_of));  // (addresses kept from pass to pass would take what registers there are)
                    State st[K];
#pragma unroll
                    for (int k = 0; k < K; ++k) st[k] = state((tiles_of >> (8 * k)) & 127u);  // (no mask: tile 0, to no effect)
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        is_out |= word[i][k] & st[k].kept;
                        is_open |= word[i][k] & ~(st[k].kept | st[k].out);
                    }
                }
                // the further masks: once a round, and where the first ones hold nothing open
                const bool look = mine && (at[i] & kRowMore) != 0 && is_out == 0 && (pass == 0 || is_open == 0);
                if (__ballot(look) != 0) {
                    asm volatile("" ::: "memory");  // keeps this a branch
                    if (look) {
                        unsigned r = (unsigned)(t * kTile + lane);
                        asm volatile("" : "+v"(r));  // (nor these addresses)
#pragma unroll 1
                        for (int j = 0; j < kMore; j += 4) {
                            const unsigned tiles_of = reinterpret_cast<const unsigned *>(at_f + r)[1 + j / 4];
                            unsigned long long w[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                w[k] = ((tiles_of >> (8 * k)) & 0xffu) != kNoTile ? more_f[(size_t)(j + k) * n_pad + r] : 0ull;
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const State st = state((tiles_of >> (8 * k)) & 127u);
                                is_out |= w[k] & st.kept;
                                is_open |= w[k] & ~(st.kept | st.out);
                            }
                            if ((tiles_of >> 24) == kNoTile || is_out != 0) break;
                        }
                    }
                }
                const unsigned long long active = open[i] & ~crowd[i];
                const unsigned long long go_out = __ballot(is_out != 0) & active, may_stay = __ballot(is_open == 0) & active;
                unsigned long long now_open = scalar(open[i]), now_kept = scalar(kept[i]);
                for (;;) {  // the tile's own rows: at most 64 times
                    const unsigned long long o = (go_out | __ballot((own[i] & now_kept) != 0)) & now_open & ~crowd[i];
                    const unsigned long long k = __ballot((own[i] & (now_open | now_kept)) == 0) & may_stay & now_open & ~o;
                    if ((o | k) == 0) break;
                    now_kept |= k;
                    now_open &= ~(o | k);
                }
                if (now_open != open[i]) {
                    settled = true;
                    open[i] = now_open;
                    kept[i] = now_kept;
                    if (lane == 0) {
                        const int in_tile = n_f - t * kTile;
                        const unsigned long long rows = in_tile >= kTile ? ~0ull : (1ull << in_tile) - 1ull;
                        __hip_atomic_store(&st_s.kept[t], now_kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_store(&st_s.out[t], ~(rows & (now_open | now_kept)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                }
            }
            if (__builtin_amdgcn_readfirstlane(settled ? 1 : 0) == 0) break;
            news |= 1u;
        }
        {
            unsigned long long any = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) any |= open[i];
            news |= any != 0 ? 2u : 0u;
            unsigned long long any_crowd = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) any_crowd |= crowd[i];
            news |= any_crowd != 0 ? 4u : 0u;
        }
        if (tid == 0) news_s[(round + 1) % 3] = 0u;
        if (lane == 0 && news != 0) atomicOr(&news_s[round % 3], news);
        lds_barrier();
        const unsigned all = (unsigned)__builtin_amdgcn_readfirstlane((int)news_s[round % 3]);
        if ((all & 2u) == 0) break;
        if ((all & 1u) == 0 || round + 1 >= ((all & 4u) != 0 ? kCrowdedRounds : kResolveRounds)) {
            open_left = true;
            break;
        }
    }
    if (!open_left) {  // uniform
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (has(i)) keep_f[index_of(i)] = (uint8_t)((kept[i] >> lane) & 1ull);
        return;
    }
    if constexpr (!WALK) {
        if (tid == 0) rel.left[f] = n_f;
    } else {
        // ---- the open rows, and the kept ones that reach a tile with open rows, in input order
        ResolveSort &so = *reinterpret_cast<ResolveSort *>(raw);
        const unsigned long long open_tiles = __ballot(lane < tiles && ~(st_s.kept[lane < tiles ? lane : 0] | st_s.out[lane < tiles ? lane : 0]) != 0);
        lds_barrier();  // (the states are not read any more)
        if (tid < kTile) so.bits[tid] = 0ull;
        unsigned long long walked[R];
        {
            const PlaceFrame p = place_frame(tab, f, n_f, n_max, n_pad);
            const float4 hull = p.hull[lane < tiles ? lane : 0];
            const float least = __uint_as_float(p.tile[lane < tiles ? lane : 0].x);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                walked[i] = open[i];
                if (kept[i] == 0) continue;  // wave-uniform
                const float4 mine = p.box[has(i) ? row_of(i) : 0];
                const float mine_T = p.T[has(i) ? row_of(i) : 0];
                for (unsigned long long todo = kept[i]; todo != 0; todo &= todo - 1) {
                    const int k = __builtin_ctzll(todo);
                    const float4 c = make_float4(lane_value(mine.x, k), lane_value(mine.y, k), lane_value(mine.z, k), lane_value(mine.w, k));
                    if ((__ballot(nms_place_reaches<true>(c, lane_value(mine_T, k), ~0u, hull, least, 0u, test.offset)) & open_tiles) != 0)
                        walked[i] |= todo & (0ull - todo);
                }
            }
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if ((walked[i] >> lane) & 1ull) __hip_atomic_fetch_or(&so.bits[index_of(i) / 64u], 1ull << (index_of(i) % 64u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        lds_barrier();
        const unsigned in_word = (unsigned)__builtin_popcountll(so.bits[lane]);
        const unsigned upto = wave_inclusive_sum(in_word);
        const int m = __builtin_amdgcn_readlane((int)upto, 63);
        if (wave == 0) so.before[lane] = upto - in_word;
        lds_barrier();
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if ((walked[i] >> lane) & 1ull) {
                const unsigned long long below = so.bits[index_of(i) / 64u] & ((1ull << (index_of(i) % 64u)) - 1ull);
                so.keys[so.before[index_of(i) / 64u] + (unsigned)__builtin_popcountll(below)] = nms_rank_key(scores[(size_t)f * n_max + index_of(i)], index_of(i));
            }
        }
        lds_barrier();

        // ---- in rank order, the ranked rows into the frame's block
        unsigned key[4], idx[4];
        int e[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            e[q] = wave * 256 + q * 64 + lane;
            const unsigned long long v = e[q] < m ? so.keys[e[q]] : kSentinel;
            key[q] = (unsigned)(v >> 32);
            idx[q] = (unsigned)v;
        }
        radix_rank_large<kResolveWaves>(key, idx, e, m, so.keys, so.hist, so.tot, so.wbase, so.match);
        float4 *sorted_f = reinterpret_cast<float4 *>(rel.words + (size_t)f * T * n_pad + nms_relation_block(n_pad).ranked);
        int32_t *order_f = reinterpret_cast<int32_t *>(sorted_f + n_pad);
        float *score_f = reinterpret_cast<float *>(order_f + n_pad);
        int32_t *label_f = reinterpret_cast<int32_t *>(score_f + n_pad);
        for (int r = tid; r < m; r += kResolveWaves * 64) {
            const unsigned from = (unsigned)so.keys[r];
            sorted_f[r] = reinterpret_cast<const float4 *>(boxes)[(size_t)f * n_max + from];
            order_f[r] = (int32_t)from;
            if (AUX) score_f[r] = scores[(size_t)f * n_max + from];
            if (AUX && test.classes != nullptr) label_f[r] = test.classes[(size_t)f * n_max + from];
        }
        __syncthreads();
        const FusedVariant v = {nullptr, nullptr, test.boundary, test.offset, (test.ties_ignore ? kExTiesIgnore : 0) | (test.classes != nullptr ? kExClasses : 0)};
        walk_frame<true, true, kExBoundary, AUX>(*reinterpret_cast<Walk *>(raw), reinterpret_cast<const float *>(sorted_f), order_f, score_f, label_f,
                                                 m, n_max, n_pad, NmsThetaConst{}, v, keep_f);
#pragma unroll
        for (int i = 0; i < R; ++i)  // (behind the barriers after the walk's zero fill)
            if ((kept[i] >> lane) & 1ull) keep_f[index_of(i)] = 1;
    }
}

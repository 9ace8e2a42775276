// Part of nms_kernels.hip (included there, inside its anonymous namespace): classic greedy rule on the mask: block-wise sweep and the apply kernel between blocks.
#pragma once

// ----------------------------------------------------------------------------- greedy sweep

// The classic sequential procedure on the same mask: rank r survives iff no SURVIVING
// better-ranked box eliminates it.  (Not what the paper's Algorithm 2 computes -- there
// every better-ranked box counts -- but the rule its introduction describes; offered as a
// selectable reduce.)  The state of the procedure lives in keep_out itself (0 = known dead).
//
// greedy_sweep_kernel settles one block of up to kSweepTiles tile rows (4096 ranks) per
// launch, one workgroup of sixteen wavefronts per frame.  Wavefront w owns the four tile rows
// 4w .. 4w+3 of the block (a lane: one row of each), and the wavefronts settle theirs in turn:
//   - rows already marked dead by earlier survivors are out; among the rest of a tile, the
//     survivors are the unique solution of  kept[r] = alive[r] and no kept c < r of this tile
//     hits r,  found by iterating that equation from kept = alive until it stops changing (row r
//     is final after r+1 rounds at most; typically a few rounds); then they are applied to the
//     later ones of the four tiles;
//   - the four words of survivors go to LDS, and behind a barrier the later wavefronts apply
//     them to their own rows: dead |= (mask word of the column tile) & kept, sixteen coalesced
//     512-byte reads per wavefront.
// What bounds it is the chain of steps, each with a barrier and at least one LDS round trip: sixteen
// steps of 256 rows instead of sixty-four of one tile row (one frame of 4096 boxes, IoU, the whole
// call: 71.7 -> 35.8 us).  The mask words do
// not depend on the steps, only what is done with them does: a wavefront has the words of the next
// two steps in flight, so memory latency stays off the chain.
// Frames with more than one block alternate with greedy_apply_kernel, which applies a settled
// block's survivors to every later row in parallel.
// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every
// global load in flight, which would put the look-ahead fetches back on the dependent chain.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kSweepTiles = 64;
constexpr int kSweepOwned = 4;                              // tile rows of a wavefront, settled in one step
constexpr int kSweepWaves = kSweepTiles / kSweepOwned;

template <bool FIRST>
__global__ void __launch_bounds__(kSweepWaves * 64)
greedy_sweep_kernel(const unsigned long long *__restrict__ mask, const int32_t *__restrict__ order,
                    const int32_t *__restrict__ counts, int n_max, int n_pad, int t0, int fill, uint8_t *__restrict__ keep_out)
{
    __shared__ unsigned long long kept_s[kSweepTiles];
    const int f = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_f = frame_count(counts, f, n_max);
    const int tiles_f = (n_f + kTile - 1) / kTile;
    const int t1 = t0 + kSweepTiles < tiles_f ? t0 + kSweepTiles : tiles_f;  // this launch settles tiles t0 .. t1-1
    const unsigned long long *m = mask + (size_t)f * ((size_t)(n_pad / kTile) * n_pad);
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const int32_t *order_f = order + (size_t)f * n_max;
    if (FIRST && fill)
        for (int i = n_f + (int)threadIdx.x; i < n_max; i += blockDim.x) keep_f[i] = 0;  // slots beyond the count
    if (t0 >= t1) return;  // uniform
    const int steps = (t1 - t0 + kSweepOwned - 1) / kSweepOwned;  // wavefronts that own tiles of this frame
    const int own = t0 + kSweepOwned * wave;                      // first owned tile row

    // a tile beyond the block's last is read as a copy of that one; its rows do not exist
    auto word_at = [&](int tc, int tr) __attribute__((always_inline)) {
        const int c = tc < t1 ? tc : t1 - 1, r = tr < t1 ? tr : t1 - 1;
        return m[(size_t)c * n_pad + r * kTile + lane];
    };
    // words of the owned rows against the four column tiles of step s; every call issues the same
    // sixteen loads, so that the wait for one step's words leaves the next step's in flight
    auto fetch = [&](unsigned long long (&w)[kSweepOwned][kSweepOwned], int s) __attribute__((always_inline)) {
        const int ss = s < wave ? s : 0;
#pragma unroll
        for (int c = 0; c < kSweepOwned; ++c)
#pragma unroll
            for (int i = 0; i < kSweepOwned; ++i) w[c][i] = word_at(t0 + kSweepOwned * ss + c, own + i);
    };

    int my_index[kSweepOwned];  // input index of this lane's row of each owned tile (-1: no such row)
    bool dead[kSweepOwned];
    unsigned long long inner[kSweepOwned][kSweepOwned];  // [c][i], c <= i: the owned tiles among themselves
    if (wave < steps) {
#pragma unroll
        for (int i = 0; i < kSweepOwned; ++i) {
            const int r = (own + i) * kTile + lane;
            my_index[i] = (own + i < t1 && r < n_f) ? order_f[r] : -1;
        }
#pragma unroll
        for (int c = 0; c < kSweepOwned; ++c)
#pragma unroll
            for (int i = c; i < kSweepOwned; ++i) inner[c][i] = word_at(own + c, own + i);
        // the first block starts with every row alive, later blocks read what the apply kernel left in keep_out
#pragma unroll
        for (int i = 0; i < kSweepOwned; ++i) dead[i] = my_index[i] < 0 || (!FIRST && keep_f[my_index[i] < 0 ? 0 : my_index[i]] == 0);
    }

    auto apply = [&](const unsigned long long (&w)[kSweepOwned][kSweepOwned], int s) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kSweepOwned; ++c) {
            const unsigned long long kept = kept_s[kSweepOwned * s + c];
#pragma unroll
            for (int i = 0; i < kSweepOwned; ++i) dead[i] = dead[i] || (w[c][i] & kept) != 0;
        }
    };
    // Every wavefront passes `steps` barriers: one behind each step before its own, its own, and the rest.
    int s = 0;
    if (wave < steps && wave > 0) {
        unsigned long long even[kSweepOwned][kSweepOwned], odd[kSweepOwned][kSweepOwned];
        fetch(even, 0);
        fetch(odd, 1);
#pragma unroll 1
        for (;;) {
            lds_barrier();
            apply(even, s);
            if (++s == wave) break;
            fetch(even, s + 1);
            lds_barrier();
            apply(odd, s);
            if (++s == wave) break;
            fetch(odd, s + 1);
        }
    }
    if (wave < steps) {
        unsigned long long kept[kSweepOwned];
#pragma unroll
        for (int i = 0; i < kSweepOwned; ++i) {
#pragma unroll
            for (int c = 0; c < i; ++c) dead[i] = dead[i] || (inner[c][i] & kept[c]) != 0;
            const bool alive = !dead[i];
            kept[i] = __ballot(alive);
            for (int round = 0; round < kTile; ++round) {
                const unsigned long long next = __ballot(alive && (inner[i][i] & kept[i]) == 0);
                if (next == kept[i]) break;
                kept[i] = next;
            }
            if (lane == 0) kept_s[kSweepOwned * wave + i] = kept[i];
        }
        lds_barrier();
        ++s;
#pragma unroll
        for (int i = 0; i < kSweepOwned; ++i)
            if (my_index[i] >= 0) keep_f[my_index[i]] = (uint8_t)((kept[i] >> lane) & 1u);
    }
    for (; s < steps; ++s) lds_barrier();
}

// Applies the survivors of the settled block of tile rows t0 .. t0+kSweepTiles-1 to every
// later row: a row with a surviving eliminator in the block is marked dead in keep_out.
// After the first block (FIRST) every later row is written, 1 = alive so far, which
// initialises the state.  One wavefront per later tile row, four per workgroup; the block's
// survivor words are rebuilt from keep_out into LDS by each workgroup.
template <bool FIRST>
__global__ void __launch_bounds__(256)
greedy_apply_kernel(const unsigned long long *__restrict__ mask, const int32_t *__restrict__ order,
                    const int32_t *__restrict__ counts, int n_max, int n_pad, int t0, uint8_t *__restrict__ keep_out)
{
    __shared__ unsigned long long kept_s[kSweepTiles];
    const int f = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_f = frame_count(counts, f, n_max);
    const int first_row_tile = t0 + kSweepTiles + (int)blockIdx.x * 4;
    if (first_row_tile * kTile >= n_f) return;  // whole workgroup beyond the count (then the block below is full)
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const int32_t *order_f = order + (size_t)f * n_max;
    for (int w = wave; w < kSweepTiles; w += 4) {
        const int r = (t0 + w) * kTile + lane;  // < n_f: a later tile row holds boxes, so the block is full
        const unsigned long long kept = __ballot(keep_f[order_f[r]] != 0);
        if (lane == 0) kept_s[w] = kept;
    }
    __syncthreads();
    const int j = first_row_tile + wave;
    const int row = j * kTile + lane;
    if (j * kTile >= n_f) return;
    const unsigned long long *col = mask + (size_t)f * ((size_t)(n_pad / kTile) * n_pad) + (size_t)t0 * n_pad + row;
    unsigned long long acc = 0;
#pragma unroll 8
    for (int w = 0; w < kSweepTiles; ++w) acc |= col[(size_t)w * n_pad] & kept_s[w];
    if (row < n_f) {
        if (FIRST)
            keep_f[order_f[row]] = acc != 0 ? 0 : 1;
        else if (acc != 0)
            keep_f[order_f[row]] = 0;
    }
}

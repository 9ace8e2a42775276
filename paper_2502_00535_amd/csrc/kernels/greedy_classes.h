// Part of nms_kernels.hip (included there, inside its anonymous namespace): greedy rule with class labels: every class by a wavefront of its own.
#pragma once

// ----------------------------------------------------------------------------- greedy rule, class by class

// With labels a box eliminates boxes of its own label only, so the sequential rule falls apart into
// one short procedure per label.  A workgroup puts the ranked boxes of its frame into 256 bins by
// label (one pass of a stable counting sort, so a bin stays in rank order) and each
// wavefront settles whole bins, without a barrier: 64 rows at a time, the bin's survivors so far
// against them, then the rows among themselves in rank order.  Twenty labels leave a twentieth of the
// pairs, and the bins of a frame run side by side where the walk of greedy_fused_kernel is one chain
// through all tiles (128 ragged frames of 3000 boxes, IoU, 20 labels, the whole call: 749 -> 69 us, and
// 65 once the rank step writes the labels in rank order).
//
// A bin is found by a hash of the label, so one bin may hold several labels: the label test stays, and
// any labels give the same result.  A bin is one wavefront's work and grows with the square of its
// size; a frame with a bin of more than nms_class_bin_limit() rows is walked instead, here and at once:
// in a launch of its own the walk starts when the last bin of the batch is done, and costs its 4 us also when
// there is nothing to do (171 x 768, three labels, frames of both kinds: 106 / 167 us, here 60 / 83;
// 128 x 3000, 20 labels 75 / 72, here 73 / 71).
//
// LDS: a bin's survivors are kept, packed, at the front of its own stretch of the tables; the tile in
// work sits right behind them (survivors + rows of the tile never exceed the rows seen so far).
constexpr int kClassBins = 256;

__device__ __forceinline__ unsigned class_bin(int label)
{
    unsigned x = (unsigned)label;
    x ^= x >> 16;
    x ^= x >> 8;
    return x & (kClassBins - 1);
}

// Putting the ranks of a frame into bins by W wavefronts.
template <int W>
struct ClassSort {
    unsigned long long match[256 * W];   // a wavefront's lane masks by bin
    unsigned hist[256 * W];              // its counts by bin, then the boxes of the bin in the wavefronts before
    __align__(16) unsigned tot[256];
};

template <int N>
struct ClassTables {
    float4 box[N];
    float T[N];
    int label[N];
    uint16_t rank[N];
};

template <int W, int N>
union ClassShared {
    ClassSort<W> sort;
    ClassTables<N> tables;
    WalkShared<W, N> walk;
};

// W: wavefronts of the workgroup; frames of at most N boxes, N = 64, 128 or 256 W.  Grid: frames * parts workgroups;
// each takes every parts-th bin of its frame.
template <bool IOU, int W, int N>
__global__ void __launch_bounds__(W * 64, 4)  // (a fourth wavefront per SIMD costs W = 4, N = 1024 a register spilled)
greedy_classes_kernel(const float *__restrict__ sorted5, const int32_t *__restrict__ order, const int32_t *__restrict__ counts,
                      int n_max, int n_pad, int parts, NmsThetaConst th, FusedVariant opt, uint8_t *__restrict__ keep_out)
{
    constexpr int kThreads = W * 64;
    static_assert(kThreads >= kClassBins, "a thread per bin");
    __shared__ __align__(16) unsigned char raw[sizeof(ClassShared<W, N>)];
    ClassSort<W> &so = reinterpret_cast<ClassShared<W, N> *>(raw)->sort;
    ClassTables<N> &tb = reinterpret_cast<ClassShared<W, N> *>(raw)->tables;
    __shared__ uint16_t ids[N];  // ranks, bin by bin
    __shared__ int start[kClassBins + 1];
    __shared__ int next_bin;
    const int f = blockIdx.x / parts;
    const int part = blockIdx.x % parts;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    const float4 *box4 = reinterpret_cast<const float4 *>(sorted5 + (size_t)f * 5 * n_pad);
    const int32_t *order_f = order + (size_t)f * n_max;
    const int32_t *label_f = opt.ranked_label + (size_t)f * n_pad;
    const float *score_f = opt.ranked_score + (size_t)f * n_pad;
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    const bool ties_ignore = (opt.flags & kExTiesIgnore) != 0;

    // a box's place in its bin: the boxes of the bin in the wavefronts before, in this wavefront's registers before, in the lanes before
    constexpr int kPer = N / kThreads;
    unsigned bin_of[kPer], place[kPer];
    {
        unsigned long long *tab = so.match + wave * 256;
        unsigned *mine = so.hist + wave * 256;
        for (int i = lane; i < 256; i += 64) {
            tab[i] = 0ull;
            mine[i] = 0u;
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int e = (wave * kPer + q) * 64 + lane;
            bin_of[q] = e < n_f ? class_bin(label_f[e]) : (unsigned)kClassBins;  // (no box)
        }
        // (the fences only keep the compiler from reordering: a wavefront's LDS instructions execute in order)
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const bool real = bin_of[q] < kClassBins;
            const unsigned b = bin_of[q] & (kClassBins - 1);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (real) __hip_atomic_fetch_or(&tab[b], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const unsigned long long same = __hip_atomic_load(&tab[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            const unsigned before = __hip_atomic_load(&mine[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const unsigned below = (unsigned)__builtin_popcountll(same & ((1ull << lane) - 1ull));
            place[q] = before + below;
            if (real && below == 0) {
                __hip_atomic_store(&mine[b], before + (unsigned)__builtin_popcountll(same), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                __hip_atomic_store(&tab[b], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
        }
    }
    __syncthreads();
    if (tid < kClassBins) {
        unsigned run = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const unsigned t = so.hist[w * 256 + tid];
            so.hist[w * 256 + tid] = run;
            run += t;
        }
        so.tot[tid] = run;
    }
    __syncthreads();
    if (wave == 0) {
        const uint4 all = reinterpret_cast<const uint4 *>(so.tot)[lane];
        const int sum = (int)(all.x + all.y + all.z + all.w);
        const int before = (int)wave_inclusive_sum((unsigned)sum) - sum;
        start[4 * lane] = before;
        start[4 * lane + 1] = before + (int)all.x;
        start[4 * lane + 2] = before + (int)(all.x + all.y);
        start[4 * lane + 3] = before + (int)(all.x + all.y + all.z);
        if (lane == 0) {
            start[kClassBins] = n_f;
            next_bin = part;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (bin_of[q] < kClassBins)
            ids[start[bin_of[q]] + (int)(so.hist[wave * 256 + bin_of[q]] + place[q])] = (uint16_t)((wave * kPer + q) * 64 + lane);
    __syncthreads();
    // (a barrier: the sort's part of the LDS is free from here on)
    const bool oversized = __syncthreads_or(tid < kClassBins && start[tid + 1] - start[tid] > nms_class_bin_limit(n_f)) != 0;
    if (oversized) {
        if (part == 0)
            walk_frame<true, IOU, kExBoundary, true>(reinterpret_cast<ClassShared<W, N> *>(raw)->walk, sorted5 + (size_t)f * 5 * n_pad, order_f,
                                                     score_f, label_f, n_f, n_max, n_pad, th, opt, keep_f);
        return;
    }
    if (part == 0)
        for (int i = n_f + tid; i < n_max; i += kThreads) keep_f[i] = 0;

    for (;;) {
        int bin = 0;
        if (lane == 0) bin = __hip_atomic_fetch_add(&next_bin, parts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        bin = __builtin_amdgcn_readfirstlane(bin);
        if (bin >= kClassBins) break;
        const int first = __builtin_amdgcn_readfirstlane(start[bin]);
        const int size = __builtin_amdgcn_readfirstlane(start[bin + 1]) - first;
        if (size <= 0) continue;

        // a lane's row of the next tile, fetched a tile ahead
        float4 row_box;
        int row_rank, row_index, row_label;
        float row_score;
        auto fetch = [&](int t0) __attribute__((always_inline)) {
            row_rank = ids[first + (t0 + lane < size ? t0 + lane : size - 1)];
            row_box = box4[row_rank];
            row_index = order_f[row_rank];
            row_label = label_f[row_rank];
            row_score = ties_ignore ? score_f[row_rank] : 0.0f;
        };
        // entry `at` of the tables as an outranking box: what the first test needs, and the rest
        auto first_entry = [&](int at) __attribute__((always_inline)) {
            const float4 b = tb.box[at];
            FusedCandidate c;
            c.x1 = b.x, c.y1 = b.y, c.x2 = b.z, c.y2 = b.w;
            c.T = tb.T[at];
            c.area = c.score = 0.0f;
            c.label = 0;
            return c;
        };
        auto complete = [&](FusedCandidate &c, int at) __attribute__((always_inline)) {
            c.area = ((c.x2 - c.x1) + opt.offset) * ((c.y2 - c.y1) + opt.offset);
            c.label = tb.label[at];
            if (ties_ignore) c.score = score_f[tb.rank[at]];
        };
        fetch(0);
        int kept_rows = 0;  // the bin's survivors so far
        for (int t0 = 0; t0 < size; t0 += kTile) {
            const int rows = size - t0 < kTile ? size - t0 : kTile;
            const bool real = lane < rows;
            const float4 v = row_box;
            const int v_rank = row_rank, v_index = row_index, v_label = row_label;
            const float v_score = row_score;
            const float v_area = ((v.z - v.x) + opt.offset) * ((v.w - v.y) + opt.offset);
            const float v_T = fused_threshold<true, IOU>(v_area, opt.boundary);
            if (t0 + kTile < size) fetch(t0 + kTile);
            unsigned long long open = rows == kTile ? ~0ull : (1ull << rows) - 1ull;  // rows that no survivor has eliminated
            const int tile_at = first + kept_rows;
            // a wavefront's LDS instructions execute in order: the fences only keep the compiler from moving them
            if (real) {
                tb.box[tile_at + lane] = v;
                tb.T[tile_at + lane] = v_T;
                tb.label[tile_at + lane] = v_label;
                tb.rank[tile_at + lane] = (uint16_t)v_rank;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            // the survivors so far, four at a time (the last one again where the count ends)
            for (int j = 0; j < kept_rows && open != 0; j += 4) {
                FusedCandidate c[4];
                unsigned long long word[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) c[k] = first_entry(first + (j + k < kept_rows ? j + k : kept_rows - 1));
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    word[k] = __ballot(fused_first<true, IOU, kExBoundary, true>(v, v_area, v_T, v_score, v_label, c[k], 0.0f, opt));
                if (((word[0] | word[1] | word[2] | word[3]) & open) != 0) {
                    asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        word[k] &= open;
                        if (word[k] != 0) {
                            complete(c[k], first + (j + k < kept_rows ? j + k : kept_rows - 1));
                            open &= ~fused_second<IOU, true>(word[k], v, v_area, v_score, v_label, c[k], opt);
                        }
                    }
                }
            }
            // the rows among themselves: the first tests of four rows side by side, then in rank order
            for (int j = 0; j < rows; j += 4) {
                if (((open >> j) & 15ull) == 0) continue;
                FusedCandidate c[4];
                unsigned long long word[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) c[k] = first_entry(tile_at + (j + k < rows ? j + k : rows - 1));
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    word[k] = __ballot(fused_first<true, IOU, kExBoundary, true>(v, v_area, v_T, v_score, v_label, c[k], 0.0f, opt));
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int r = j + k;  // < 64; a row at or beyond `rows` is not open
                    word[k] &= open & (r == kTile - 1 ? 0ull : ~0ull << (r + 1));
                    if (((open >> r) & 1ull) != 0 && word[k] != 0) {
                        asm volatile("" ::: "memory");  // keeps this a branch
                        complete(c[k], tile_at + (r < rows ? r : rows - 1));
                        open &= ~fused_second<IOU, true>(word[k], v, v_area, v_score, v_label, c[k], opt);
                    }
                }
            }
            const bool kept = ((open >> lane) & 1ull) != 0;
            if (real) keep_f[v_index] = kept ? 1 : 0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (kept) {
                const int at = tile_at + __builtin_popcountll(open & ((1ull << lane) - 1ull));
                tb.box[at] = v;
                tb.T[at] = v_T;
                tb.label[at] = v_label;
                tb.rank[at] = (uint16_t)v_rank;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            kept_rows += __builtin_popcountll(open);
        }
    }
}

// Part of nms_kernels.hip (included there, inside its anonymous namespace): rank step of small batches: ranks counted over the whole chip, no sort.
#pragma once

// ----------------------------------------------------------------------------- rank by counting

// The rank of a box is the number of boxes that outrank it.  A sort of one chunk is the work of one
// workgroup -- a chain of thirteen barriers, 16 us at 4096 boxes however few frames there are --, whereas
// counting is n compares per box that depend on nothing: two VALU instructions per pair (compare, add
// with carry), spread over as many workgroups as the chip holds.  It wins until the pairs take longer
// than the chain: see nms_use_count_rank.
//
// A workgroup stages the keys of its whole frame in LDS and ranks kElems neighbouring elements of the
// input.  lane = (element, group); wavefronts and groups share the other keys out in units of four
// (one 16-byte LDS read, the same address for all lanes of a group), and their counts meet in LDS.
// kElems: 64, or 16 and four groups (nms_count_rank_elements).  Two elements per lane (128), which a read
// serves eight compares instead of four, gain only where the sort is as quick (120 x 500 boxes 5.7 us
// against 6.8 with 64 elements, sorted 6.8; 64 x 500 4.3 against 4.5; 8 x 3000 9.8 against 9.6).
// Equal keys: the lower index first, so the keys before the workgroup's elements count when they are
// not larger, the keys behind them when they are smaller, and only its own elements need the index.
// Integer keys: ranks are a permutation whatever the bits of the scores are.
constexpr int kCountThreads = 1024;
constexpr int kCountWaves = kCountThreads / 64;

template <int kElems>
__global__ void __launch_bounds__(kCountThreads)
rank_count_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ counts,
                  int n_max, int n_pad, int32_t *__restrict__ order, float *__restrict__ sorted5,
                  uint8_t *__restrict__ keep_preset, RankExtras ex)
{
    static_assert(kElems <= 64, "one element per lane");
    constexpr int kGroups = 64 / kElems;
    __shared__ uint4 keys4[kChunk / 4];
    __shared__ int partial[kCountWaves][kElems];
    unsigned *keys = reinterpret_cast<unsigned *>(keys4);
    const int f = blockIdx.y;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    const int e0 = blockIdx.x * kElems;
    const float *scores_f = scores + (size_t)f * n_max;
    float *sorted_f = sorted5 + (size_t)f * 5 * n_pad;

    // box, score and label of the element this thread writes out at the end: fetched now, used then
    const int e_mine = e0 + tid;
    float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
    float s_mine = -INFINITY;
    int label = 0;
    if (tid < kElems && e_mine < n_f) {
        b = reinterpret_cast<const float4 *>(boxes + (size_t)f * n_max * 4)[e_mine];
        if (ex.score != nullptr) {
            s_mine = scores_f[e_mine];
            if (ex.classes != nullptr) label = ex.classes[(size_t)f * n_max + e_mine];
        }
    }
    if (e0 < n_f) {  // uniform
        const int units = (n_f + 3) / 4;
        for (int i = tid; i < 4 * units; i += kCountThreads)
            keys[i] = i < n_f ? (unsigned)(nms_rank_key(scores_f[i], (unsigned)i) >> 32) : ~0u;  // (behind the last element: smaller than none)
        __syncthreads();
        const int e = e0 + lane % kElems;
        const unsigned mine = keys[e < n_f ? e : e0];
        int before = 0;
        const int first = wave * kGroups + lane / kElems;  // this lane's first unit
        constexpr int kStride = kCountWaves * kGroups;
        const int own = e0 / 4;                            // units [own, own_end): the workgroup's own elements
        const int own_end = own + kElems / 4 < units ? own + kElems / 4 : units;
#pragma unroll 2
        for (int u = first; u < own; u += kStride) {
            const uint4 k = keys4[u];
            before += k.x <= mine;
            before += k.y <= mine;
            before += k.z <= mine;
            before += k.w <= mine;
        }
        for (int u = own + first; u < own_end; u += kStride) {
            const uint4 k = keys4[u];
            before += k.x < mine || (k.x == mine && 4 * u < e);
            before += k.y < mine || (k.y == mine && 4 * u + 1 < e);
            before += k.z < mine || (k.z == mine && 4 * u + 2 < e);
            before += k.w < mine || (k.w == mine && 4 * u + 3 < e);
        }
#pragma unroll 2
        for (int u = own_end + first; u < units; u += kStride) {
            const uint4 k = keys4[u];
            before += k.x < mine;
            before += k.y < mine;
            before += k.z < mine;
            before += k.w < mine;
        }
#pragma unroll
        for (int step = kElems; step < 64; step <<= 1) before += __shfl_xor(before, step);
        if (lane < kElems) partial[wave][lane] = before;
        __syncthreads();
    }
    if (tid >= kElems || e_mine >= n_pad) return;
    int r = e_mine;  // rows beyond the count hold padding, in place
    if (e_mine < n_f) {
        r = 0;
#pragma unroll
        for (int w = 0; w < kCountWaves; ++w) r += partial[w][tid];
        emit_ranked_box(b, e_mine, r, n_pad, order + (size_t)f * n_max, sorted_f, nullptr, nullptr, 0.0);
    } else {
        emit_padding_row(e_mine, n_pad, sorted_f, nullptr, nullptr);
    }
    if (ex.score != nullptr) {
        const size_t at = (size_t)f * n_pad + r;
        ex.score[at] = s_mine;
        if (ex.classes != nullptr) ex.label[at] = label;
        ex.area[at] = ((b.z - b.x) + ex.offset) * ((b.w - b.y) + ex.offset);
    }
    if (keep_preset != nullptr && e_mine < n_max) keep_preset[(size_t)f * n_max + e_mine] = e_mine < n_f ? 1 : 0;
}

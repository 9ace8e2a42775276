// Part of nms_kernels.hip (included there, inside its anonymous namespace): greedy rule on frames of at most 192 boxes in one launch (all variants).
#pragma once

// ----------------------------------------------------------------------------- greedy rule, small frames

// Rank step, mask and sweep of a short frame are three launches of 3 to 5 us that do next to nothing.  Here one
// workgroup does all of it in LDS: ranks by counting (four threads per box, as in rank_count_kernel), the boxes to
// their ranks, the words of the mask (lane = outranking box, a wavefront per 16 rows of a tile of the ranked
// triangle; the pair tests are those of the walk, fused_word), and the sweep by one wavefront, tile by tile, as
// in greedy_sweep_kernel.  What bounds it is that chain: 6.3 us for a call at 70 boxes, of which the call itself is 6; 8.8 at
// 50 x 160, where the three launches take 12.2.
template <int N, bool EX, bool IOU, int MODE, bool AUX>
__global__ void __launch_bounds__(4 * N)
greedy_small_kernel(const float *__restrict__ boxes, const float *__restrict__ scores, const int32_t *__restrict__ classes,
                    const int32_t *__restrict__ counts, int n_max, NmsThetaConst th, FusedVariant opt, uint8_t *__restrict__ keep_out)
{
    constexpr int W = N / 16, kTiles = (N + kTile - 1) / kTile;
    static_assert(kTiles <= 3 && N % kTile == 0, "pairs of tiles");
    constexpr bool kUseT = MODE == kExBoundary && (!IOU || AUX);
    __shared__ uint4 keys4[N / 4];
    __shared__ float4 box[N];
    __shared__ float T[N], area[N], score[N];
    __shared__ int label[N];
    __shared__ uint16_t index[N];
    __shared__ unsigned long long words[N][kTiles];
    unsigned *keys = reinterpret_cast<unsigned *>(keys4);
    const int f = blockIdx.x;
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_f = frame_count(counts, f, n_max);
    const float *score_f = scores + (size_t)f * n_max;
    uint8_t *keep_f = keep_out + (size_t)f * n_max;
    for (int i = n_f + tid; i < n_max; i += 4 * N) keep_f[i] = 0;
    if (n_f == 0) return;
    const bool labelled = AUX && (opt.flags & kExClasses) != 0;

    const int e = tid >> 2;  // this thread's box, shared with its three neighbours
    float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
    float s = 0.0f;
    int l = 0;
    if ((tid & 3) == 0 && e < n_f) {
        b = reinterpret_cast<const float4 *>(boxes)[(size_t)f * n_max + e];
        if (AUX) s = score_f[e];
        if (labelled) l = classes[(size_t)f * n_max + e];
    }
    if (tid < N) keys[tid] = tid < n_f ? (unsigned)(nms_rank_key(score_f[tid], (unsigned)tid) >> 32) : ~0u;
    lds_barrier();
    int before = 0;
    {
        const unsigned mine = keys[e < n_f ? e : 0];
        for (int u = tid & 3; 4 * u < n_f; u += 4) {  // (equal keys: the lower index first; behind the last box: smaller than none)
            const uint4 k = keys4[u];
            before += k.x < mine || (k.x == mine && 4 * u < e);
            before += k.y < mine || (k.y == mine && 4 * u + 1 < e);
            before += k.z < mine || (k.z == mine && 4 * u + 2 < e);
            before += k.w < mine || (k.w == mine && 4 * u + 3 < e);
        }
        before += __builtin_amdgcn_update_dpp(0, before, 0xb1, 0xf, 0xf, true);  // quad_perm: neighbour
        before += __builtin_amdgcn_update_dpp(0, before, 0x4e, 0xf, 0xf, true);  // quad_perm: the other pair
    }
    if ((tid & 3) == 0 && e < n_f) {
        const float a = EX ? ((b.z - b.x) + opt.offset) * ((b.w - b.y) + opt.offset) : nms_box_area(b.x, b.y, b.z, b.w);
        box[before] = b;
        area[before] = a;
        T[before] = kUseT ? fused_threshold<EX, IOU>(a, EX ? opt.boundary : th.m) : 0.0f;
        score[before] = s;
        label[before] = l;
        index[before] = (uint16_t)e;
    }
    lds_barrier();

    auto entry = [&](int r) __attribute__((always_inline)) {
        FusedCandidate c;
        const float4 v = box[r];
        c.x1 = v.x, c.y1 = v.y, c.x2 = v.z, c.y2 = v.w;
        c.area = area[r];
        c.T = T[r];
        c.score = AUX ? score[r] : 0.0f;
        c.label = AUX ? label[r] : 0;
        return c;
    };
    // ---- the mask: 16 rows of a tile of the ranked triangle at a time
    const int tiles = (n_f + kTile - 1) / kTile;
    for (int item = wave; item < 2 * tiles * (tiles + 1); item += W) {
        const int pair = item >> 2;
        const int tr = pair < 1 ? 0 : (pair < 3 ? 1 : 2);
        const int tc = pair - tr * (tr + 1) / 2;
        const FusedCandidate c = entry(tc * kTile + lane);  // (what lies behind the last box outranks none)
        const int r0 = tr * kTile + 16 * (item & 3);
#pragma unroll 4
        for (int k = 0; k < 16; ++k) {
            const int r = r0 + k < n_f ? r0 + k : n_f - 1;  // (the last row again)
            const FusedCandidate v = entry(r);
            const unsigned long long open = tr == tc ? (1ull << (r & (kTile - 1))) - 1ull : ~0ull;
            const unsigned long long word = fused_word<EX, IOU, MODE, AUX>(open, make_float4(v.x1, v.y1, v.x2, v.y2), v.area, v.T, v.score,
                                                                           v.label, c, th.theta, opt);
            if (lane == 0 && r0 + k < n_f) words[r][tc] = word;
        }
    }
    lds_barrier();
    if (wave != 0) return;

    // ---- the sweep
    unsigned long long kept[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
        kept[t] = 0ull;
        if (t * kTile < n_f) {  // uniform
            const int r = t * kTile + lane;
            bool alive = r < n_f;
            unsigned long long own = 0ull;
            if (alive) {
#pragma unroll
                for (int c = 0; c < t; ++c) alive = alive && (words[r][c] & kept[c]) == 0;
                own = words[r][t];
            }
            kept[t] = __ballot(alive);
            for (int round = 0; round < kTile; ++round) {
                const unsigned long long next = __ballot(alive && (own & kept[t]) == 0);
                if (next == kept[t]) break;
                kept[t] = next;
            }
            if (r < n_f) keep_f[index[r]] = (uint8_t)((kept[t] >> lane) & 1ull);
        }
    }
}

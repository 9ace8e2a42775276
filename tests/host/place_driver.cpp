// Host checks of nms_place.h, which the kernels in order of place share.
//   place_driver reach        frames of 1 to 128 tiles with boxes of every size, infinite ones and such whose area overflows among them:
//                             reach words as the kernels form them (64 lanes at a time, lanes behind the last tile read the last one);
//                             prints "words <n> outside <n>": bits of lanes that are no tile
//   place_driver bins         labels -8 .. 511 and their bins
//   place_driver tiles        random tiles of outranking boxes and victims: a pair that eliminates, by the definition (float32, IEEE division), in a tile that does not
//                             reach the victim is a violation; a box under its own T that eliminates is one too.  Prints, per form, "form violations hits reached of"
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "../../paper_2502_00535_amd/csrc/nms_place.h"

struct Box {
    float x, y, z, w;
};
static const int kTile = 64;

struct Tile {
    Box hull;
    float T;
    uint32_t best;
};

// The hull of the boxes at rows 64 t .. of a frame of n, as place_sort_kernel stores it.
template <bool IOU>
static Tile make_tile(const std::vector<Box> &box, const std::vector<float> &T, const std::vector<uint32_t> &upper, int n, int t)
{
    Box h = {INFINITY, INFINITY, INFINITY, INFINITY};
    Tile r;
    r.T = INFINITY;
    r.best = ~0u;
    for (int i = t * kTile; i < (t + 1) * kTile; ++i) {
        const bool there = i < n;
        nms_place_hull_add<IOU>(h, r.T, there ? box[i] : Box{0.f, 0.f, 0.f, 0.f}, there ? T[i] : INFINITY, there);
        if (there) r.best = std::min(r.best, upper[i]);
    }
    r.hull = {h.x, h.y, -h.z, -h.w};
    return r;
}

template <bool IOU>
static void reach(std::mt19937 &rng, long &words, long &outside)
{
    std::uniform_real_distribution<float> u(0.0f, 1.0f);
    for (int tiles = 1; tiles <= 128; ++tiles) {
        const int n = (tiles - 1) * kTile + 1 + (int)(rng() % kTile);
        const float off = IOU && rng() % 2 ? 0.0f : 1.0f;
        const double boundary = 0.45;
        std::vector<Box> box(n);
        std::vector<float> T(n);
        std::vector<uint32_t> upper(n);
        for (int i = 0; i < n; ++i) {
            const float x = 1000.0f * u(rng), y = 1000.0f * u(rng);
            box[i] = {x, y, x + 1.0f + 90.0f * u(rng), y + 1.0f + 90.0f * u(rng)};
            const int kind = (int)(rng() % 40);
            if (kind == 0) box[i].z = INFINITY;
            if (kind == 1) box[i].x = -INFINITY, box[i].w = INFINITY;
            if (kind == 2) box[i] = {-1e30f, -1e30f, 1e30f, 1e30f};
            if (kind == 3) box[i] = {INFINITY, INFINITY, INFINITY, INFINITY};
            T[i] = nms_place_threshold<IOU>(((box[i].z - box[i].x) + off) * ((box[i].w - box[i].y) + off), boundary);
            upper[i] = (uint32_t)rng();
        }
        std::vector<Tile> tile(tiles);
        for (int t = 0; t < tiles; ++t) tile[t] = make_tile<IOU>(box, T, upper, n, t);
        for (int v = 0; v < n; v += 3) {
            for (int s = 0; s < tiles; s += kTile) {
                unsigned long long word = 0;
                for (int lane = 0; lane < kTile; ++lane) {
                    const int t = s + lane;
                    const Tile &c = tile[t < tiles ? t : tiles - 1];
                    if (nms_place_reaches<IOU>(box[v], T[v], upper[v], c.hull, c.T, c.best, off)) word |= 1ull << lane;
                }
                word &= nms_place_tile_lanes(s, tiles);
                ++words;
                if (tiles - s < kTile && (word >> (tiles - s)) != 0) ++outside;
            }
        }
    }
}

// The definition: the outranking box c eliminates v, compare >= or > (gt).
static bool eliminates(const Box &v, const Box &c, bool iou, bool gt, float off, float theta)
{
    volatile float iw = std::max(0.0f, (std::min(v.z, c.z) - std::max(v.x, c.x)) + off);
    volatile float ih = std::max(0.0f, (std::min(v.w, c.w) - std::max(v.y, c.y)) + off);
    volatile float inter = iw * ih;
    volatile float wc = (c.z - c.x) + off, hc = (c.w - c.y) + off, wv = (v.z - v.x) + off, hv = (v.w - v.y) + off;
    volatile float ac = wc * hc, av = wv * hv;
    volatile float sum = av + ac;
    volatile float denom = iou ? sum - inter : (float)ac;
    volatile float q = inter / denom;
    return gt ? q > theta : !(q < theta);
}

// The rounding boundary of the division next to theta, below it for >=, above it for >.
static double boundary_of(float theta, bool gt)
{
    uint32_t b;
    std::memcpy(&b, &theta, sizeof b);
    b = gt ? b + 1u : b - 1u;
    float other;
    std::memcpy(&other, &b, sizeof other);
    return 0.5 * ((double)theta + (double)other);
}

template <bool IOU>
static void tiles_form(std::mt19937 &rng, bool gt, float off, const char *name)
{
    std::uniform_real_distribution<float> u(0.0f, 1.0f);
    const float thetas[] = {0.3f, 0.45f, 0.5f, 0.7f, 1.0f, 0x1p-40f, 0.01f, 1.3f, 0x1p20f, 0.25f};
    long violations = 0, hits = 0, reached = 0, asked = 0;
    for (int round = 0; round < 6000; ++round) {
        const float theta = thetas[rng() % 10];
        const double boundary = boundary_of(theta, gt);
        const float scale = std::ldexp(1.0f, (int)(rng() % 40) - 10), size = std::ldexp(1.0f, (int)(rng() % 14) - 6);
        const bool grid = rng() % 2, steered = rng() % 2, flat = IOU && off == 0.0f && rng() % 4 == 0;
        const float cx = scale * (u(rng) - 0.5f), cy = scale * (u(rng) - 0.5f);
        auto box = [&](float spread) {
            float x = cx + spread * (u(rng) - 0.5f), y = cy + spread * (u(rng) - 0.5f), w = size * u(rng), h = size * u(rng);
            if (grid) x = std::floor(x), y = std::floor(y), w = std::floor(w), h = std::floor(h);
            if (off == 0.0f && !flat) w += size * 0.01f + 0x1p-20f * scale, h += size * 0.01f + 0x1p-20f * scale;  // extents above 0
            Box b = {x, y, x + w, y + h};
            if (flat && rng() % 3 == 0) b.z = b.x;  // no area
            return b;
        };
        const int n = 1 + (int)(rng() % kTile);
        std::vector<Box> box_c(n);
        std::vector<float> T(n);
        std::vector<uint32_t> upper(n);
        for (int i = 0; i < n; ++i) {
            box_c[i] = box(size * 3.0f);
            T[i] = nms_place_threshold<IOU>(((box_c[i].z - box_c[i].x) + off) * ((box_c[i].w - box_c[i].y) + off), boundary);
            upper[i] = (uint32_t)rng() % 16;
        }
        const Tile t = make_tile<IOU>(box_c, T, upper, n, 0);
        for (int k = 0; k < 12; ++k) {
            Box v = box(size * 3.0f);
            if (steered) {  // a victim that just reaches, or is, a box of the tile
                const Box &c = box_c[rng() % n];
                const float w = c.z - c.x, h = c.w - c.y;
                v = {c.x + w * (rng() % 3 == 0 ? 0.0f : theta < 1.0f ? 1.0f - theta : 0.0f), c.y, c.z, c.w + (rng() % 4 == 0 ? h : 0.0f)};
                if (!(v.z >= v.x)) v = c;
            }
            const uint32_t v_upper = (uint32_t)rng() % 16;
            const float v_T = nms_place_threshold<IOU>(((v.z - v.x) + off) * ((v.w - v.y) + off), boundary);
            const bool reach = nms_place_reaches<IOU>(v, v_T, v_upper, t.hull, t.T, t.best, off);
            reached += reach;
            ++asked;
            for (int i = 0; i < n; ++i) {
                if (upper[i] > v_upper || !eliminates(v, box_c[i], IOU, gt, off, theta)) continue;
                ++hits;
                const float inter = nms_place_inter(v, box_c[i], off);
                const bool first_test = inter >= (IOU ? std::max(T[i], v_T) : T[i]);
                const bool no_area = IOU && !(T[i] > 0.0f && v_T > 0.0f);  // (decided by the tile's reach alone: 0 / 0)
                if (!reach || (!first_test && !no_area)) ++violations;
            }
        }
    }
    std::printf("%s %ld %ld %ld %ld\n", name, violations, hits, reached, asked);
}

int main(int argc, char **argv)
{
    std::mt19937 rng(7);
    if (argc > 1 && std::strcmp(argv[1], "reach") == 0) {
        long words = 0, outside = 0;
        reach<false>(rng, words, outside);
        reach<true>(rng, words, outside);
        std::printf("words %ld outside %ld\n", words, outside);
        return 0;
    }
    if (argc > 1 && std::strcmp(argv[1], "tiles") == 0) {
        tiles_form<false>(rng, false, 1.0f, "area_ge");
        tiles_form<false>(rng, true, 1.0f, "area_gt");
        tiles_form<true>(rng, false, 1.0f, "iou_ge_1");
        tiles_form<true>(rng, true, 1.0f, "iou_gt_1");
        tiles_form<true>(rng, false, 0.0f, "iou_ge_0");
        tiles_form<true>(rng, true, 0.0f, "iou_gt_0");
        return 0;
    }
    if (argc > 1 && std::strcmp(argv[1], "bins") == 0) {
        for (int label = -8; label < 512; ++label) std::printf("%d %u\n", label, nms_place_bin(label));
        return 0;
    }
    return 2;
}

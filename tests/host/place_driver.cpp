// Host checks of nms_place.h, which the kernels in order of place share.
//   place_driver reach        frames of 1 to 128 tiles with boxes of every size, infinite ones and such whose area overflows among them:
//                             reach words as the kernels form them (64 lanes at a time, lanes behind the last tile read the last one);
//                             prints "words <n> outside <n>": bits of lanes that are no tile
//   place_driver bins         labels -8 .. 511 and their bins
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
    if (argc > 1 && std::strcmp(argv[1], "bins") == 0) {
        for (int label = -8; label < 512; ++label) std::printf("%d %u\n", label, nms_place_bin(label));
        return 0;
    }
    return 2;
}

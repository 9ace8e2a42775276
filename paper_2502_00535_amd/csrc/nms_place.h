// What the kernels in order of place rely on when they leave pairs out: the least intersection that may eliminate, the hull of a
// tile of outranking boxes, and whether the tile can hold an eliminator of a victim.  Plain functions, shared by the kernels
// and compilable by a host compiler alone (the host tests run them without a GPU).
//
// min, max and the rounded float32 subtraction, addition and multiplication are monotone, and a box of the tile lies inside its
// hull: the float32 intersection of victim and hull, by the operations of the pair test, is no smaller than with any box of the
// tile.  Where it stays below the least T of the tile, no pair test of the tile succeeds.
#pragma once

#include <math.h>
#include <stdint.h>
#include <string.h>

#include "nms_pair.h"

// The float32 below which an intersection with a box eliminates nothing: the value that decides (outranking area), or, under
// IoU, a bound that no union undercuts: the union is no smaller than either box but for the rounding of its two operations,
// which the factor covers.  Under IoU 0 for a box without area.
template <bool IOU>
NMS_HD float nms_place_threshold(float area, double boundary)
{
    if (!IOU) return nms_pair_threshold(area, boundary);
    const double t = boundary * (double)area * (1.0 - 0x1p-21);
    float t1 = (float)t;
    if ((double)t1 > t) {  // next float32 down (t > 0)
        uint32_t b;
        memcpy(&b, &t1, sizeof b);
        b -= 1u;
        memcpy(&t1, &b, sizeof t1);
    }
    return t1 > 0.0f ? t1 : 0.0f;
}

// Intersection of a victim and an outranking box (or a hull); B: x, y, z, w = x1, y1, x2, y2.
template <class B>
NMS_HD float nms_place_inter(const B &v, const B &c, float off)
{
    const float iw = (fminf(v.z, c.z) - fmaxf(v.x, c.x)) + off;  // one floor is enough where T > 0: see nms_pair.h
    const float ih = fmaxf(0.0f, (fminf(v.w, c.w) - fmaxf(v.y, c.y)) + off);
    return iw * ih;
}

// One row of a tile taken into its hull: h = (least x1, least y1, least -x2, least -y2), least = the least T.  A row that is not
// there changes nothing.  IOU: a box without area (no positive T) may eliminate what it does not touch: its tile reaches everything.
template <bool IOU, class B>
NMS_HD void nms_place_hull_add(B &h, float &least, const B &v, float T, bool there)
{
    const bool odd = IOU && there && !(T > 0.0f);
    const float far = odd ? -INFINITY : INFINITY;
    h.x = fminf(h.x, there && !odd ? v.x : far);
    h.y = fminf(h.y, there && !odd ? v.y : far);
    h.z = fminf(h.z, there && !odd ? -v.z : far);
    h.w = fminf(h.w, there && !odd ? -v.w : far);
    least = fminf(least, odd ? -INFINITY : (there ? T : INFINITY));
}

// Can a tile hold a box that is ranked before the victim and eliminates it?  hull, tile_T, best: the tile's; best, v_upper: upper
// halves of rank keys.
template <bool IOU, class B>
NMS_HD bool nms_place_reaches(const B &v, float v_T, uint32_t v_upper, const B &hull, float tile_T, uint32_t best, float off)
{
    const float inter = nms_place_inter(v, hull, off);
    const float least = IOU ? (tile_T < 0.0f ? tile_T : fmaxf(tile_T, v_T)) : tile_T;
    return (inter >= least) & (best <= v_upper);
}

// Which of the 64 lanes stand for a tile when they look at the tiles first, first + 1, .. (first < tiles).  No T can say that: an
// intersection with an infinite box, or one whose area overflows, reaches infinity too.
NMS_HD unsigned long long nms_place_tile_lanes(int first, int tiles)
{
    return tiles - first >= 64 ? ~0ull : (1ull << (tiles - first)) - 1ull;
}

// Bin of a label, one of sixteen.  With bits 4 to 7 of the label it tells 0 to 255 apart, and neither labels with equal low bits nor
// labels with equal high bits share one (by the low bits alone, labels that are multiples of 16 did: 100 x 2000 boxes with
// nine of them 108 us, now 61, 20 x 4096 73 and 33).
NMS_HD unsigned nms_place_bin(int label)
{
    return ((unsigned)label ^ ((unsigned)label >> 4)) & 15u;
}

// Host check that the pair test is monotone in the victim's box: a box that eliminates a victim passes the same test against any box
// around the victim.  Reads lines "theta cx1 cy1 cx2 cy2 k" followed by k victims; prints "violations <n> hits <n>".
#include <cstdio>
#include <vector>
#include <algorithm>
#include "../../paper_2502_00535_amd/csrc/nms_pair.h"

int main()
{
    float theta, c[4];
    int k;
    long violations = 0, hits = 0;
    while (std::scanf("%f %f %f %f %f %d", &theta, c, c + 1, c + 2, c + 3, &k) == 6) {
        std::vector<float> v(4 * (size_t)k);
        for (float &x : v)
            if (std::scanf("%f", &x) != 1) return 1;
        float h[4] = {INFINITY, INFINITY, -INFINITY, -INFINITY};
        for (int i = 0; i < k; ++i) {
            h[0] = std::min(h[0], v[4 * i]), h[1] = std::min(h[1], v[4 * i + 1]);
            h[2] = std::max(h[2], v[4 * i + 2]), h[3] = std::max(h[3], v[4 * i + 3]);
        }
        const NmsThetaConst th = nms_make_theta_const(theta);
        const float T = nms_pair_threshold(nms_box_area(c[0], c[1], c[2], c[3]), th.m);
        const bool passes = nms_eliminates_fast(h[0], h[1], h[2], h[3], c[0], c[1], c[2], c[3], T);
        for (int i = 0; i < k; ++i)
            if (nms_eliminates_fast(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3], c[0], c[1], c[2], c[3], T)) {
                ++hits;
                violations += passes ? 0 : 1;
            }
    }
    std::printf("violations %ld hits %ld\n", violations, hits);
    return 0;
}

// Head groups or stage kernels for a C = 1280 layer (mid_preferred): at sizes where both were timed and differ by more than 3 %, the
// rule takes the faster one. Host code only.
#include <cstdio>

#include "taq_internal.h"

struct Point {
    int H, packed, B, N;
    double groups, stages;  // us per call
};

int main() {
    const Point points[] = {
        {8, 1, 1, 496, 21.9, 26.1},  {8, 1, 1, 512, 18.4, 25.8},  {8, 1, 1, 528, 29.3, 26.5},  {8, 1, 1, 544, 27.4, 26.5},  {8, 1, 1, 640, 25.8, 26.8},
        {8, 1, 1, 656, 29.8, 27.0},  {8, 1, 1, 768, 26.1, 26.9},  {8, 1, 1, 784, 30.5, 27.7},  {8, 1, 1, 848, 33.1, 27.9},  {8, 1, 1, 1024, 30.1, 28.2},
        {8, 1, 2, 317, 25.5, 26.8},  {8, 1, 4, 189, 25.3, 27.0},  {8, 1, 8, 77, 25.3, 26.5},   {8, 1, 2, 509, 29.8, 28.2},  {8, 1, 4, 253, 30.0, 28.1},
        {8, 1, 5, 109, 28.6, 26.3},  {8, 0, 1, 496, 24.5, 26.7},  {8, 0, 1, 512, 20.5, 26.4},  {8, 0, 1, 576, 30.0, 27.6},  {8, 0, 1, 768, 29.9, 27.9},
        {20, 1, 1, 400, 16.8, 23.1}, {20, 1, 1, 784, 25.6, 26.6}, {20, 1, 1, 832, 25.3, 26.9}, {20, 1, 1, 848, 30.8, 27.2}, {20, 1, 1, 864, 28.7, 27.0},
        {20, 1, 4, 205, 25.4, 26.8}, {20, 1, 1, 896, 25.9, 27.2}, {20, 1, 1, 912, 31.6, 27.5}, {20, 1, 3, 285, 28.7, 27.0}, {20, 1, 1, 1008, 32.7, 27.4},
        {20, 0, 1, 400, 18.5, 23.6}, {20, 0, 1, 432, 24.2, 23.3}, {20, 0, 1, 496, 26.7, 24.6}, {20, 0, 1, 640, 23.3, 25.3}, {20, 0, 1, 656, 27.6, 25.6},
        {20, 0, 1, 704, 24.2, 25.6}, {20, 0, 4, 189, 24.1, 25.5}, {20, 0, 1, 784, 28.7, 27.4}, {20, 0, 1, 832, 29.9, 27.6}, {20, 0, 3, 269, 29.0, 27.6},
    };
    int bad = 0;
    for (const Point& p : points) {
        taq_shape s = {};
        s.B = p.B; s.N = p.N; s.C = 1280; s.H = p.H; s.T = 77; s.Cc = 768;
        s.bits_kv = s.bits_prob = s.bits_q = s.bits_proj = 8;
        s.w_layout = p.packed;
        if (!taq::mid_supported(s) || taq::mid_preferred(s) != (p.groups < p.stages)) {
            std::fprintf(stderr, "%d heads, %s weights, %d x %d tokens: groups %.1f us, stages %.1f us\n", p.H, p.packed ? "packed" : "row-major", p.B, p.N, p.groups, p.stages);
            ++bad;
        }
    }
    if (!bad) std::puts("mid_rule: ok");
    return bad != 0;
}

// Kernels of the full-precision path and the token sweep that sizes select: at sizes where the forms were timed in turn on one card, the form that
// the rule takes is the fastest, or within the 2 % by which repeated timings differ. Host code only.
#include <cstdio>

#include "taq_internal.h"

static int bad = 0;
static void check(const char* what, int a, int b, double taken, double best) {
    if (taken <= 1.02 * best) return;
    std::fprintf(stderr, "%s, %d x %d: %.1f us, the fastest %.1f us\n", what, a, b, taken, best);
    ++bad;
}

// launch_gemm_f16, us per sweep of 2 x rows / 2 image tokens and 5 text tokens (9 at 12000 x 96), with small and with large tiles
struct Product {
    int rows, C;
    double small, large;
};
static const Product products[] = {
    {320, 1280, 80.4, 87.6},  {480, 1280, 85.7, 90.8},  {640, 1280, 92.5, 96.7},  {800, 1280, 100.0, 104.0}, {864, 1280, 104.2, 104.3},
    {992, 1280, 106.6, 106.1}, {1120, 1280, 113.7, 113.0}, {1280, 1280, 118.7, 116.8}, {1440, 1280, 128.9, 124.8}, {1600, 1280, 134.0, 130.6},
    {640, 640, 70.7, 73.6},   {1216, 640, 79.6, 82.8},  {1600, 640, 86.7, 89.0},  {1760, 640, 88.6, 89.1},  {1984, 640, 93.6, 94.6},
    {2240, 640, 99.9, 99.9},  {2560, 640, 100.9, 100.1}, {3200, 640, 112.1, 109.0}, {1280, 320, 68.9, 71.0}, {2432, 320, 75.3, 76.1},
    {3200, 320, 80.2, 80.4},  {3520, 320, 85.5, 85.5},  {4480, 320, 91.1, 90.3},  {5120, 320, 92.8, 91.0},  {6400, 320, 101.6, 99.8},
    {12000, 96, 86.0, 87.0},
    {4256, 96, 61.1, 61.9},   {8096, 96, 67.2, 67.4},   {10656, 96, 69.6, 70.2},  {14912, 96, 75.7, 75.3},  {800, 960, 121.3, 125.1},
    {1056, 960, 135.3, 137.4}, {1312, 960, 147.4, 147.4}, {1920, 960, 189.1, 186.5}, {1504, 512, 72.1, 76.1}, {1984, 512, 81.1, 82.8},
    {2784, 512, 88.2, 87.3},  {4000, 512, 109.6, 105.5},
};

int main() {
    for (const Product& p : products)
        check("sweep, fp16 product", p.rows, p.C, taq::gemm_f16_small(p.rows, p.C) ? p.small : p.large, p.small < p.large ? p.small : p.large);
    if (!bad) std::puts("fullprec_rule: ok");
    return bad != 0;
}

// Two claims that the exact quantizers rest on, over all their cases, on the host in float32:
//   half_row (csrc/taq_device.h): the code of an fp16 value is rint of one product, where 127 does not divide the significand of the row's largest
//     value; every significand of a largest value against every fp16 value below it, and with the factor one unit off either way (its reciprocal
//     comes from the hardware's approximation)
//   div_grid: the division by 127 and by 7, for every float from 0 to infinity: with an argument all of them (a minute), otherwise every significand
//     of the binades up to 2^-86, where quotient or remainder may be subnormal, of a few in the middle, where a power of two changes nothing, and
//     of the last three
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <thread>

#include "taq_device.h"

using taq::div_grid;

static float as_float(uint32_t u) {
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}
static uint32_t as_bits(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    return u;
}

// the definition: rint(fl(fl(x * 127) / amax)); the fast path: the low byte of fma(x, m, 1.5 * 2^23)
static int defined(float x, float amax) { return (int)std::rint((x * 127.0f) / amax); }
static int fast(float x, float m) { return (int8_t)as_bits(std::fma(x, m, 12582912.0f)); }

int main(int argc, char** argv) {
    (void)argv;
    const bool all = argc > 1;
    long bad = 0;
    for (int A = 1024; A < 2048; ++A) {  // amax = A, times a power of two, which changes nothing; subnormal ones are among them with fewer bits
        const float amax = (float)A;
        const float c = 127.0f / amax, scale = div_grid(amax, 127.f);
        if (taq::half_row(c, scale, amax).doubt != (A % 127 == 0)) ++bad;
        if (A % 127 == 0) continue;
        for (int off = -1; off <= 1; ++off) {
            const float m = taq::half_row(as_float(as_bits(c) + off), scale, amax).m;
            for (int shift = 0; shift < 40; ++shift) {  // x = X 2^-shift <= amax
                bool any = false;
                for (int X = 1024; X < 2048; ++X) {
                    const float x = std::ldexp((float)X, -shift);
                    if (x > amax) break;
                    const int want = defined(x, amax);
                    any |= want != 0;
                    if (want != fast(x, m) || -want != fast(-x, m)) ++bad;
                }
                if (!any) break;  // (smaller ones are zeros too)
            }
        }
    }
    if (bad) std::fprintf(stderr, "rows of fp16 values: %ld codes\n", bad);
    std::atomic<int> next{0};
    std::atomic<long> wrong{0};
    auto binades = [&]() {  // (subnormal numbers are slow on the host)
        for (int e; (e = next++) < 255;) {
            if (!all && e > 40 && e < 252 && e % 50) continue;
            for (float d : {127.f, 7.f})
                for (uint32_t u = (uint32_t)e << 23; u < (uint32_t)(e + 1) << 23; ++u) {
                    const float x = as_float(u), q = div_grid(x, d), want = x / d;
                    if (as_bits(q) != as_bits(want) && wrong++ < 20) std::fprintf(stderr, "%a / %g: %a, not %a\n", x, d, q, want);
                }
        }
    };
    std::thread threads[8];
    for (std::thread& t : threads) t = std::thread(binades);
    for (std::thread& t : threads) t.join();
    bad += wrong;
    const float inf = INFINITY;
    for (float d : {127.f, 7.f})
        if (div_grid(inf, d) != inf) ++bad;
    if (!bad) std::puts("grid_quotients: ok");
    return bad != 0;
}

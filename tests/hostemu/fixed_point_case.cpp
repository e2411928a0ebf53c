// The scatter pass's float-to-integer conversion against exact arithmetic: prints
// every (v, e) of its list where fixed_point is not the rounded product, or not 0 where
// that is no integer below 2^62; exits 1 if there is one.
#include "emu.h"
#include "bwd_pixel.h"

static long long want(float v, int e) {
    const float x = rintf(ldexpf(v, e));
    if (!(fabsf(x) < 0x1p62f)) return 0;
    return (long long)x;   // (in range: exact)
}

int main() {
    int bad = 0;
    long long n = 0;
    auto one = [&](float v, int e) {
        ++n;
        const long long g = vct::fixed_point(v, e), w = want(v, e);
        if (g != w && ++bad < 20) printf("fixed_point(%a, %d) = %lld, expected %lld\n", v, e, g, w);
    };
    const float inf = INFINITY;
    for (int e : {-40, 0, 17, 31, 61})
        for (float v : {0.0f, -0.0f, inf, -inf, (float)NAN, -(float)NAN, FLT_MAX, -FLT_MAX, FLT_MIN, 1e-45f}) one(v, e);
    // powers of two and their neighbours, halves (ties to even), odd multiples of 2^31 (ties of the split)
    for (int p = -3; p <= 64; ++p)
        for (float m : {1.0f, 1.5f, 1.25f, 1.75f, 2.5f, 5.0f, 0x1.fffffep0f, 0x1.000002p0f, 0x1.800002p0f, 0x1.7ffffep0f})
            for (int e : {0, 5, 31, 61}) {
                one(ldexpf(m, p - e), e);
                one(-ldexpf(m, p - e), e);
            }
    for (int k = 1; k < 4096; k += 2) {
        one((float)k, 31);
        one(-(float)k, 31);
    }
    unsigned int s = 12345;
    for (int i = 0; i < 4000000; ++i) {
        s = s * 1664525u + 1013904223u;
        const float m = __uint_as_float((s >> 9) | 0x3f800000u);
        s = s * 1664525u + 1013904223u;
        const int p = (int)((s >> 8) % 66u) - 3, e = (int)((s >> 20) % 70u) - 5;
        one(ldexpf((s & 0x80u) ? -m : m, p - e), e);
    }
    printf("%lld values, %d wrong\n", n, bad);
    return bad != 0;
}

// Twiddle constants w = exp(+2 pi i n / L) as c (1 + i t), from compile-time series.
#pragma once

#include <cstdint>

namespace epic {

struct Root {
    float t, c;
};

// |x| <= pi, 2 n / L <= 1 / 2: exact to FP64 rounding before they are rounded to FP32.
constexpr double kPi = 3.14159265358979323846;
constexpr double series_cos(double x) {
    double s = 1.0, t = 1.0;
    for (int k = 1; k < 24; ++k) {
        t *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
        s += t;
    }
    return s;
}
constexpr double series_sin(double x) {
    double s = x, t = x;
    for (int k = 1; k < 24; ++k) {
        t *= -x * x / ((2.0 * k) * (2.0 * k + 1.0));
        s += t;
    }
    return s;
}
// What is applied is c and the product c t, the same for every sample, so a constant's
// error does not average out over time.  Rounding c and t each for itself leaves two
// roundings in c t (2.9-3.1e-8 RMS over the roots of 128, 256 and 512, the worst
// 7.5e-8); the pair (t, c) nearest to w among the nine c next to the rounded
// cosine is as near as the rounded (cos, sin) are (2.1e-8, the worst 3.9e-8).
constexpr Root root_of(int n, int L) {
    if (4 * n == L) return Root{0x1p40f, 0x1p-40f};
    const double x = 2.0 * kPi * n / L, cx = series_cos(x), sx = series_sin(x);
    Root best{0.f, 0.f};
    double least = 2.0;
    for (int k = -4; k <= 4; ++k) {
        const float c = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, (float)cx) + (uint32_t)k);
        const float t = (float)(sx / (double)c);
        const double ec = (double)c - cx, es = (double)c * (double)t - sx;
        if (ec * ec + es * es < least) {
            least = ec * ec + es * es;
            best = Root{t, c};
        }
    }
    return best;
}

}  // namespace epic

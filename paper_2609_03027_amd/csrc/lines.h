// Short transforms in registers (positive exponent, natural order) and their
// twiddle constants, shared by the fused and staged kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "roots.h"

namespace epic {

// ---------------------------------------------------------------- complex
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 mul_i(float2 a) { return make_float2(-a.y, a.x); }

// Length-R DFT with the positive exponent, natural order in and out:
// v[p] <- sum_q v[q] exp(+2 pi i p q / R).
template <int R> __device__ __forceinline__ void dft(float2 *v);

template <> __device__ __forceinline__ void dft<4>(float2 *v) {
    const float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const float2 t2 = cadd(v[1], v[3]), t3 = mul_i(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
}

template <> __device__ __forceinline__ void dft<8>(float2 *v) {
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    dft<4>(e);
    dft<4>(o);
    const float h = 0.70710678118654752440f;
    // o1 *= (1+i)/sqrt2, o2 *= i, o3 *= (-1+i)/sqrt2
    o[1] = make_float2((o[1].x - o[1].y) * h, (o[1].x + o[1].y) * h);
    o[2] = mul_i(o[2]);
    o[3] = make_float2(-(o[3].x + o[3].y) * h, (o[3].x - o[3].y) * h);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        v[p] = cadd(e[p], o[p]);
        v[p + 4] = csub(e[p], o[p]);
    }
}

// Length-8 DFT of v[q] w^q: every twiddle goes into the radix-2 butterfly that
// follows it.  With w = c (1 + i t), a +- w b takes two fused multiply-adds for
// u = (1 + i t) b and four for a +- c u, so the transform with its seven
// twiddles costs 72 instructions instead of 52 + 28.  c = 0 is held as c =
// 2^-40, t = 2^40, whose products are exact.  |t b| may pass FP32's range where
// |b| does not (above 2^87): for transforms whose |E|^2 has to fit FP32, not for
// those that return E.
struct Tw8 {
    Root w4, w2, w1, w1e;                // w^4, w^2, w, w exp(2 pi i / 8)
};
__device__ __forceinline__ void bfly(float2 &a, float2 &b, Root r) {
    const float u = fmaf(-r.t, b.y, b.x), v = fmaf(r.t, b.x, b.y);
    b = make_float2(fmaf(-r.c, u, a.x), fmaf(-r.c, v, a.y));
    a = make_float2(fmaf(r.c, u, a.x), fmaf(r.c, v, a.y));
}
__device__ __forceinline__ void bfly_i(float2 &a, float2 &b, Root r) {     // a +- i w b
    const float u = fmaf(-r.t, b.y, b.x), v = fmaf(r.t, b.x, b.y);
    b = make_float2(fmaf(r.c, v, a.x), fmaf(-r.c, u, a.y));
    a = make_float2(fmaf(-r.c, v, a.x), fmaf(r.c, u, a.y));
}
// The last two stages: e[q] = v[q] + w^4 v[q+4], o[q] = v[q] - w^4 v[q+4].
__device__ __forceinline__ void dft8_tail(float2 *v, float2 *e, float2 *o, Root w2, Root w1, Root w1e) {
    bfly(e[0], e[2], w2);
    bfly(e[1], e[3], w2);
    bfly(e[0], e[1], w1);
    bfly_i(e[2], e[3], w1);
    bfly_i(o[0], o[2], w2);
    bfly_i(o[1], o[3], w2);
    bfly(o[0], o[1], w1e);
    bfly_i(o[2], o[3], w1e);
    v[0] = e[0];
    v[4] = e[1];
    v[2] = e[2];
    v[6] = e[3];
    v[1] = o[0];
    v[5] = o[1];
    v[3] = o[2];
    v[7] = o[3];
}
__device__ __forceinline__ void dft8_tw(float2 *v, const Tw8 &w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) bfly(v[q], v[q + 4], w.w4);
    float2 e[4] = {v[0], v[1], v[2], v[3]}, o[4] = {v[4], v[5], v[6], v[7]};
    dft8_tail(v, e, o, w.w2, w.w1, w.w1e);
}
// The same with w = exp(2 pi i / 16): the first stage's twiddle is i.
__device__ __forceinline__ void dft8_root16(float2 *v) {
    float2 e[4], o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        e[q] = cadd(v[q], mul_i(v[q + 4]));
        o[q] = csub(v[q], mul_i(v[q + 4]));
    }
    dft8_tail(v, e, o, Root{1.f, 0.70710678118654752440f},
              Root{0.41421356237309504880f, 0.92387953251128675613f},
              Root{2.41421356237309504880f, 0.38268343236508977173f});
}

// Length 4 likewise, w^2 and w: 24 instructions instead of 16 + 12.
struct Tw4 {
    Root w2, w1;
};
__device__ __forceinline__ void dft4_tw(float2 *v, const Tw4 &w) {
    bfly(v[0], v[2], w.w2);
    bfly(v[1], v[3], w.w2);
    bfly(v[0], v[1], w.w1);
    bfly_i(v[2], v[3], w.w1);
    const float2 t = v[1];              // (X0, X2, X1, X3) -> natural order
    v[1] = v[2];
    v[2] = t;
}

constexpr Tw8 tw8_of(int n, int L) {     // 8 divides L
    return Tw8{root_of(4 * n, L), root_of(2 * n, L), root_of(n, L), root_of(n + L / 8, L)};
}
constexpr Tw4 tw4_of(int n, int L) { return Tw4{root_of(2 * n, L), root_of(n, L)}; }
struct RootTables {
    Tw8 r8[16];                          // exp(+2 pi i n / 128): 64-point lines take even n
    Tw4 r4[8];                           // exp(+2 pi i n / 32): 16-point lines take even n
    Tw4 r96[24], r48[12];                // exp(+2 pi i n / 96), exp(+2 pi i n / 48)
};
constexpr RootTables root_tables() {
    RootTables t{};
    for (int n = 0; n < 16; ++n) t.r8[n] = tw8_of(n, 128);
    for (int n = 0; n < 8; ++n) t.r4[n] = tw4_of(n, 32);
    for (int n = 0; n < 24; ++n) t.r96[n] = tw4_of(n, 96);
    for (int n = 0; n < 12; ++n) t.r48[n] = tw4_of(n, 48);
    return t;
}
__constant__ constexpr RootTables kRoots = root_tables();

// Twiddles of an M-point line's second step on the block of frequency p.
template <int M> struct LineTw;
template <> struct LineTw<64> {
    using T = Tw8;
    static __device__ __forceinline__ T at(int p) { return kRoots.r8[2 * p]; }
};
template <> struct LineTw<32> {
    using T = Tw4;
    static __device__ __forceinline__ T at(int p) { return kRoots.r4[p]; }
};
template <> struct LineTw<16> {
    using T = Tw4;
    static __device__ __forceinline__ T at(int p) { return kRoots.r4[2 * p]; }
};
__device__ __forceinline__ void dft_tw(float2 *v, const Tw8 &w) { dft8_tw(v, w); }
__device__ __forceinline__ void dft_tw(float2 *v, const Tw4 &w) { dft4_tw(v, w); }

// a exp(+2 pi i m / 16), m a constant after unrolling
__device__ __forceinline__ float2 rot16(float2 a, int m) {
    constexpr float c1 = 0.92387953251128675613f, s1 = 0.38268343236508977173f;
    constexpr float h = 0.70710678118654752440f;
    switch (m) {
        case 0: return a;
        case 1: return cmul(a, make_float2(c1, s1));
        case 2: return cmul(a, make_float2(h, h));
        case 3: return cmul(a, make_float2(s1, c1));
        case 4: return mul_i(a);
        case 6: return cmul(a, make_float2(-h, h));
        default: return cmul(a, make_float2(-c1, -s1));     // 9
    }
}

// Length 16 as 4 x 4, constant twiddles between the steps.
__device__ __forceinline__ void dft16(float2 *v) {
    float2 y[4][4];                     // [j][p]: step 1 over v[j + 4 q]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) y[j][q] = v[j + 4 * q];
        dft<4>(y[j]);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float2 z[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = rot16(y[j][p], j * p);
        dft<4>(z);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[p + 4 * k] = z[k];
    }
}

// Length 16 with input twiddles w^q: 192 instructions instead of 152 + 60.
struct Tw16 {
    Root w8, w4, w2, w2e;                // w^8, w^4, w^2, w^2 exp(2 pi i / 8)
    Root w1[4];                          // w exp(2 pi i p / 16)
};
constexpr Tw16 tw16_of(int n, int L) {   // 16 divides L
    return Tw16{root_of(8 * n, L), root_of(4 * n, L), root_of(2 * n, L), root_of(2 * n + L / 8, L),
                {root_of(n, L), root_of(n + L / 16, L), root_of(n + L / 8, L),
                 root_of(n + 3 * L / 16, L)}};
}
__device__ __forceinline__ void dft16_tw(float2 *v, const Tw16 &w) {
    float2 y[4][4];                     // [j][p]: v[j + 4 q] w^(4 q), the factor w^j left out
    const Tw4 w44{w.w8, w.w4};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) y[j][q] = v[j + 4 * q];
        dft4_tw(y[j], w44);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {       // input twiddle W = w exp(2 pi i p / 16)
        float2 a = y[0][p], b = y[1][p], c = y[2][p], d = y[3][p];
        const Root sq = (p & 1) ? w.w2e : w.w2;    // W^2, for p >= 2 without its factor i
        if (p < 2) {
            bfly(a, c, sq);
            bfly(b, d, sq);
        } else {
            bfly_i(a, c, sq);
            bfly_i(b, d, sq);
        }
        bfly(a, b, w.w1[p]);
        bfly_i(c, d, w.w1[p]);
        v[p] = a;
        v[p + 8] = b;
        v[p + 4] = c;
        v[p + 12] = d;
    }
}
__device__ __forceinline__ void dft_tw(float2 *v, const Tw16 &w) { dft16_tw(v, w); }

}  // namespace epic

// Low-bitwidth EPIC path (precision EPIC_FIXED16) on 64 x 64 grids, the size
// of the FPGA prototype's transform core (Sec. 3): integer gridding with
// 8+8-bit kernel weights, a rounding shift to 16-bit grid values, and a 2D
// radix-2 decimation-in-frequency FFT in 16-bit fixed point with a scaling
// bit per stage, round-half-up and saturation between stages (Sec. 3: the
// FFT core takes different scaling schemes).  The Eq. 2 products of the
// integer sky values are summed exactly in 64-bit integers, each time slice's
// sums leave as FP64 (exact below 2^53), and their total does not depend on the
// order; one reduce scales it back to image units and adds it to the FP32
// accumulator.
//
// Arithmetic, per sample and feed (all integer):
//   G'[j]  = sum_a conj(q_a(j)) (-1)^(jx+jy) E_a            (exact, int32)
//   G16[j] = sat16(rsh(G'[j], sg))
//   stage s of an axis, pair (a, c) = (x[b+i], x[b+i+h]), h = 64 / 2^(s+1):
//     a <- sat16(rsh(a + c, sh_s)),  c <- sat16(rsh((a - c) w_{i 2^s}, ts + sh_s))
//   rsh(x, k) = (x + 2^(k-1)) >> k (k > 0), x (k = 0); w_n = rint(2^ts e^{+2 pi i n/64}).
// Rows (along x) take scaling bits 0-5, columns bits 6-11; the outputs are
// in bit-reversed order on both axes.  The (-1)^j factor makes the plain
// transform give the Eq. 2 products of the centred one of Eq. 1.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace epic {

namespace {
constexpr int FN = 64, FT = 512, FROW = 65;

typedef short s16x2 __attribute__((ext_vector_type(2)));

// A complex 16-bit value stays one register (re & 0xffff) | im << 16 from the
// stage to the products: sums and differences are packed 16-bit operations,
// complex products two-element dot products with an int32 accumulator.
__device__ __forceinline__ uint32_t pack16(int r, int i) {
    return ((uint32_t)r & 0xffffu) | ((uint32_t)i << 16);
}
__device__ __forceinline__ s16x2 pk(uint32_t v) { return __builtin_bit_cast(s16x2, v); }
__device__ __forceinline__ uint32_t un(s16x2 v) { return __builtin_bit_cast(uint32_t, v); }
// c + a.lo b.lo + a.hi b.hi, modulo 2^32
__device__ __forceinline__ int dot2(uint32_t a, uint32_t b, int c) {
    return __builtin_amdgcn_sdot2(pk(a), pk(b), c, false);
}
// The same where the result fits int32: the saturating form takes its third
// operand from any register, the plain one overwrites it (a copy per use).
__device__ __forceinline__ int dot2_fit(uint32_t a, uint32_t b, int c) {
    return __builtin_amdgcn_sdot2(pk(a), pk(b), c, true);
}
// (sat16(r), sat16(i))
__device__ __forceinline__ uint32_t sat_pack(int r, int i) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pk_i16(r, i));
}
__device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b) {
    return un(__builtin_elementwise_add_sat(pk(a), pk(b)));
}
__device__ __forceinline__ uint32_t sub_sat(uint32_t a, uint32_t b) {
    return un(__builtin_elementwise_sub_sat(pk(a), pk(b)));
}
__device__ __forceinline__ uint32_t half_floor(uint32_t a) { return un(pk(a) >> (short)1); }
// (im of a, re of a): the halves swapped
__device__ __forceinline__ uint32_t swap16(uint32_t a) { return __builtin_amdgcn_alignbit(a, a, 16); }

// sat16(rsh(a + c, SH)) per half.  Halving: a + c = 2 (a | c) - (a ^ c), so
// floor((a + c + 1) / 2) = (a | c) - floor((a ^ c) / 2), always in range.
template <bool SH> __device__ __forceinline__ uint32_t sum16(uint32_t a, uint32_t c) {
    if (!SH) return add_sat(a, c);
    return un(pk(a | c) - pk(half_floor(a ^ c)));
}
// sat16(rsh(a - c, SH)) per half.  Halving: a - c + 1 = 2 (a & ~c) - (a ^ c) + 1,
// so floor((a - c + 1) / 2) = (a & ~c) - floor((a ^ c) / 2), which reaches
// 32768 (a = 32767, c = -32768): the last subtraction saturates.
template <bool SH> __device__ __forceinline__ uint32_t dif16(uint32_t a, uint32_t c) {
    if (!SH) return sub_sat(a, c);
    return sub_sat(a & ~c, half_floor(a ^ c));
}

// A twiddle as the four dot-product operands (wr, -wi), (-wr, wi), (wi, wr),
// (-wi, -wr): |w| <= 2^14, so every half is exact.
struct TwW {
    uint32_t p, pn, q, qn;
};
__device__ __forceinline__ TwW tw_operands(int2 w) {
    return TwW{pack16(w.x, -w.y), pack16(-w.x, w.y), pack16(w.y, w.x), pack16(-w.y, -w.x)};
}

// One radix-2 DIF butterfly of the definition above, t = ts + SH, rnd =
// 2^(t-1).  The product (a - c) w is a w + c (-w); with |wr| + |wi| <=
// sqrt(2) 2^14 + 1, a w + rnd stays below 2^30 and the whole below 2^31.
template <bool SH>
__device__ __forceinline__ void bfly(uint32_t &a, uint32_t &c, const TwW &w, int t, int rnd) {
    const int vr = dot2(c, w.pn, dot2_fit(a, w.p, rnd));
    const int vi = dot2(c, w.qn, dot2_fit(a, w.q, rnd));
    a = sum16<SH>(a, c);
    c = sat_pack(vr >> t, vi >> t);
}
// w = 2^ts: rsh((a - c) 2^ts, ts + sh) = rsh(a - c, sh)
template <bool SH> __device__ __forceinline__ void bfly_1(uint32_t &a, uint32_t &c) {
    const uint32_t d = dif16<SH>(a, c);
    a = sum16<SH>(a, c);
    c = d;
}
// w = i 2^ts: (re, im) = (c.im - a.im, a.re - c.re), rounded the same way
template <bool SH> __device__ __forceinline__ void bfly_i(uint32_t &a, uint32_t &c) {
    const uint32_t d = dif16<SH>(__builtin_amdgcn_alignbit(a, c, 16), __builtin_amdgcn_alignbit(c, a, 16));
    a = sum16<SH>(a, c);
    c = d;
}

// Stages 0-2 of an axis on the 8 elements j + 8 m (m = 0..7) of a line:
// stage 0 pairs (m, m+4) with twiddle index j + 8 m; stage 1 pairs
// (m, m+2), m in {0, 1, 4, 5}, index 2 (j + 8 (m & 1)); stage 2 pairs
// (m, m+1), m even, index 4 j.  wa[0..3] = w_{j+8m}, wa[4..5] =
// w_{2(j+8b)}, wa[6] = w_{4j}.  Every stage exists with and without halving;
// the scaling bits are uniform, so a stage costs one scalar branch.
template <int ST, bool SH>
__device__ __forceinline__ void stage_a(uint32_t *v, const TwW *wa, int ts, const int *rn) {
    const int t = ts + (SH ? 1 : 0), rnd = rn[SH ? 1 : 0];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        if (ST == 0 && m < 4) bfly<SH>(v[m], v[m + 4], wa[m], t, rnd);
        if (ST == 1 && (m & 2) == 0) bfly<SH>(v[m], v[m + 2], wa[4 + (m & 1)], t, rnd);
        if (ST == 2 && (m & 1) == 0) bfly<SH>(v[m], v[m + 1], wa[6], t, rnd);
    }
}
// Stages 3-5 of an axis on the 8 elements 8 q + m: stage 3 pairs (m, m+4)
// with index 8 m; stage 4 pairs (m, m+2), m in {0, 1, 4, 5}, index
// 16 (m & 1); stage 5 pairs (m, m+1), index 0.  wb = w_8, w_24.
template <int ST, bool SH>
__device__ __forceinline__ void stage_b(uint32_t *v, const TwW *wb, int ts, const int *rn) {
    const int t = ts + (SH ? 1 : 0), rnd = rn[SH ? 1 : 0];
    if (ST == 3) {
        bfly_1<SH>(v[0], v[4]);
        bfly<SH>(v[1], v[5], wb[0], t, rnd);
        bfly_i<SH>(v[2], v[6]);
        bfly<SH>(v[3], v[7], wb[1], t, rnd);
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        if (ST == 4 && (m & 3) == 0) bfly_1<SH>(v[m], v[m + 2]);
        if (ST == 4 && (m & 3) == 1) bfly_i<SH>(v[m], v[m + 2]);
        if (ST == 5 && (m & 1) == 0) bfly_1<SH>(v[m], v[m + 1]);
    }
}
// Stages s0 .. s0 + 2 of the mask on both feeds.  ALL: every bit is set.
template <int P, bool ALL>
__device__ __forceinline__ void stages_012(uint32_t *x, uint32_t *y, const TwW *wa, int ts,
                                           const int *rn, uint32_t mask) {
#define EPIC_STAGE(F, ST, W)                       \
    if (ALL || ((mask >> ST) & 1u)) {              \
        F<ST, true>(x, W, ts, rn);                 \
        if (P == 2) F<ST, true>(y, W, ts, rn);     \
    } else {                                       \
        F<ST, false>(x, W, ts, rn);                \
        if (P == 2) F<ST, false>(y, W, ts, rn);    \
    }
    EPIC_STAGE(stage_a, 0, wa)
    EPIC_STAGE(stage_a, 1, wa)
    EPIC_STAGE(stage_a, 2, wa)
}
template <int P, bool ALL>
__device__ __forceinline__ void stages_345(uint32_t *x, uint32_t *y, const TwW *wb, int ts,
                                           const int *rn, uint32_t mask) {
    EPIC_STAGE(stage_b, 3, wb)
    EPIC_STAGE(stage_b, 4, wb)
    EPIC_STAGE(stage_b, 5, wb)
#undef EPIC_STAGE
}

__device__ __forceinline__ int brev6(int p) { return (int)(__brev((unsigned)p) >> 26); }

__device__ __forceinline__ int2 uni2(int2 v) {
    return make_int2(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y));
}
}  // namespace

// One workgroup per (channel, time slice); 512 threads; j = tid / 64 is the
// wave index, so pass-A twiddles are wave-uniform.  Gather entry (uint2): x =
// element | cell << 14 | last-tap-of-cell << 31, y = the conjugate weight
// q' = conj(q) (-1)^(jx+jy) as the dot-product operand (q'r, -q'i).  Every
// entry stores the running sum, so the loop has no per-lane branches: a cell's
// last tap to the cell, the others to column 64, which no pass reads.
// The first 2 EB entries of a lane stay in registers for the whole sample loop
// (they are the same every sample; 256 elements with a
// 3 x 3 kernel fill five, and no entries are read then), and each sample's
// voltages are loaded during the sample before.  The Eq. 2 products are formed
// as unsigned 32-bit integers (the cross products with a bias of 2^31 - 1, so
// that x = y = -32768 - 32768 i still fits) and summed in 64 bits.  With
// `autos` (A <= 512) the self-term sums are added here.
// part: double [slice][item][P == 2 ? 4 : 1][4096] sums in natural pixel
// order; slices with no samples write zeros.
//
// Bound: vector issue.  A thread and sample takes about 12 instructions per
// butterfly with a general twiddle (4 packed for the sum, 4 dot products, 2
// shifts and 1 saturating pack for the product) and 6 with a unit one, about
// 1200 in all.  64 channels, 256 elements, K = 2, 8+8 bits, 1000 samples: 1.17 ms
// with the reduce, 2.05 ms with every part unpacked to 32 bits, FP64 product
// sums, entries read from L2 one by one and a separate self-term pass.
//
// ALL: every stage halves (the default mask), so the stages need no branches.
template <int P, bool ALL>
__global__ __launch_bounds__(FT) __attribute__((amdgpu_waves_per_eu(4))) void k_fixed64(
    const FusedItem *__restrict__ items, int n_items, const uint2 *__restrict__ entries,
    const uint8_t *__restrict__ volt, int64_t volt_t_stride, int A, int n_time, int t_per_slice,
    const int2 *__restrict__ tw, int ts, uint32_t mask, int sg, double *__restrict__ part, int vb,
    int32_t *__restrict__ autos) {
    constexpr int NPROD = P == 2 ? 4 : 1;
    constexpr int EB = 3;
    extern __shared__ uint2 smem[];
    uint2 *grid = smem;                  // [64][65] cells
    uint2 *stage = smem + FN * FROW;     // [A] staged voltages
    const int item = blockIdx.x % n_items, slice = blockIdx.x / n_items;
    const FusedItem it = items[item];
    const int tid = threadIdx.x;
    const int line = tid & 63;
    const int j = __builtin_amdgcn_readfirstlane(tid >> 6);

    TwW wa[7], wb[2];
#pragma unroll
    for (int m = 0; m < 4; ++m) wa[m] = tw_operands(uni2(tw[j + 8 * m]));
    wa[4] = tw_operands(uni2(tw[2 * j]));
    wa[5] = tw_operands(uni2(tw[2 * (j + 8)]));
    wa[6] = tw_operands(uni2(tw[4 * j]));
    wb[0] = tw_operands(uni2(tw[8]));
    wb[1] = tw_operands(uni2(tw[24]));

    for (int i = tid; i < FN * FROW; i += FT) grid[i] = make_uint2(0u, 0u);
    uint32_t acc[8][NPROD], acch[8][NPROD];      // 64-bit sums, low and high halves
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
        for (int q = 0; q < NPROD; ++q) acc[m][q] = acch[m][q] = 0u;

    const int t0 = slice * t_per_slice;
    const int t1 = min(n_time, t0 + t_per_slice);
    const uint8_t *vbase = volt + (int64_t)it.c * P * A * vb;
    const uint2 *ent = entries + it.entry_off + tid;
    const int n_iter = it.n_iter;
    auto entry = [&](int k) {
        // past the list: no weight, not a cell's last tap, the unread column
        return k < n_iter ? ent[(int64_t)k * FT] : make_uint2((uint32_t)FN << 14, 0u);
    };
    uint2 held[2 * EB];
#pragma unroll
    for (int k = 0; k < 2 * EB; ++k) held[k] = entry(k);
    // this sample's voltages of element tid, loaded one sample ahead
    uint32_t rx = 0u, ry = 0u;
    if (tid < A && t0 < t1) {
        const uint8_t *v0 = vbase + (int64_t)t0 * volt_t_stride;
        rx = volt_raw(v0, tid, vb);
        ry = P == 2 ? volt_raw(v0, A + tid, vb) : 0u;
    }
    int sa[NPROD];
#pragma unroll
    for (int q = 0; q < NPROD; ++q) sa[q] = 0;
    const int half = (1 << sg) >> 1;
    // rounding terms without and with halving; kept in vector registers, since
    // a dot product takes one scalar operand (the twiddle)
    int rn[2] = {1 << (ts - 1), 1 << ts};
    asm volatile("" : "+v"(rn[0]), "+v"(rn[1]));
    for (int t = t0; t < t1; ++t) {
        const uint8_t *vt = vbase + (int64_t)t * volt_t_stride;
        if (tid < A) {
            const int2 x = volt_dec(rx, vb);
            const int2 y = P == 2 ? volt_dec(ry, vb) : make_int2(0, 0);
            stage[tid] = make_uint2(pack16(x.x, x.y), pack16(y.x, y.y));
            if (autos) {
                sa[0] += x.x * x.x + x.y * x.y;
                if (P == 2) {
                    sa[1] += y.x * y.x + y.y * y.y;
                    sa[2] += x.x * y.x + x.y * y.y;
                    sa[3] += x.y * y.x - x.x * y.y;
                }
            }
        }
        for (int a = tid + FT; a < A; a += FT) {
            const int2 x = volt_at(vt, a, vb);
            const int2 y = P == 2 ? volt_at(vt, A + a, vb) : make_int2(0, 0);
            stage[a] = make_uint2(pack16(x.x, x.y), pack16(y.x, y.y));
        }
        __syncthreads();
        if (t + 1 < t1 && tid < A) {
            rx = volt_raw(vt + volt_t_stride, tid, vb);
            ry = P == 2 ? volt_raw(vt + volt_t_stride, A + tid, vb) : 0u;
        }
        {
            int sxr = half, sxi = half, syr = half, syi = half;
            uint2 e[EB];
            for (int k0 = 0; k0 < n_iter; k0 += EB) {
                if (k0 < 2 * EB) {
#pragma unroll
                    for (int k = 0; k < EB; ++k) {
                        // decoded per sample: hoisted out of the loop the
                        // addresses and swapped operands would take three
                        // registers an entry
                        e[k] = k0 ? held[EB + k] : held[k];
                        asm volatile("" : "+v"(e[k].x), "+v"(e[k].y));
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < EB; ++k) e[k] = entry(k0 + k);
                }
                uint2 v[EB];
#pragma unroll
                for (int k = 0; k < EB; ++k) v[k] = stage[e[k].x & 0x3FFFu];
#pragma unroll
                for (int k = 0; k < EB; ++k) {
                    const uint32_t wp = e[k].y;                             // (q'r, -q'i)
                    const uint32_t wq = un(pk(swap16(wp)) * s16x2{-1, 1});  // (q'i, q'r)
                    sxr = dot2(v[k].x, wp, sxr);
                    sxi = dot2(v[k].x, wq, sxi);
                    if (P == 2) {
                        syr = dot2(v[k].y, wp, syr);
                        syi = dot2(v[k].y, wq, syi);
                    }
                    grid[(e[k].x >> 14) & 0x1FFFu] = make_uint2(
                        sat_pack(sxr >> sg, sxi >> sg), P == 2 ? sat_pack(syr >> sg, syi >> sg) : 0u);
                    const bool last = (e[k].x >> 31) != 0u;
                    sxr = last ? half : sxr;
                    sxi = last ? half : sxi;
                    syr = last ? half : syr;
                    syi = last ? half : syi;
                }
            }
        }
        __syncthreads();
        // rows (along x): stages 0-2 on elements j + 8 m of row `line`
        {
            uint32_t vx[8], vy[8];
            const int base = line * FROW + j;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint2 g = grid[base + 8 * m];
                vx[m] = g.x;
                vy[m] = g.y;
            }
            stages_012<P, ALL>(vx, vy, wa, ts, rn, mask);
#pragma unroll
            for (int m = 0; m < 8; ++m) grid[base + 8 * m] = make_uint2(vx[m], vy[m]);
        }
        __syncthreads();
        // rows: stages 3-5 on elements 8 j + m
        {
            uint32_t vx[8], vy[8];
            const int base = line * FROW + 8 * j;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint2 g = grid[base + m];
                vx[m] = g.x;
                vy[m] = g.y;
            }
            stages_345<P, ALL>(vx, vy, wb, ts, rn, mask);
#pragma unroll
            for (int m = 0; m < 8; ++m) grid[base + m] = make_uint2(vx[m], vy[m]);
        }
        __syncthreads();
        // columns (along y): stages 0-2 on rows j + 8 m of column `line`
        {
            uint32_t vx[8], vy[8];
            const int base = j * FROW + line;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint2 g = grid[base + 8 * m * FROW];
                vx[m] = g.x;
                vy[m] = g.y;
            }
            stages_012<P, ALL>(vx, vy, wa, ts, rn, mask >> 6);
#pragma unroll
            for (int m = 0; m < 8; ++m) grid[base + 8 * m * FROW] = make_uint2(vx[m], vy[m]);
        }
        __syncthreads();
        // columns: stages 3-5 on rows 8 j + m, then the Eq. 2 products; the
        // grid is left zeroed for the next gather (the staging barrier of
        // the next sample orders these writes before it)
        {
            uint32_t vx[8], vy[8];
            const int base = 8 * j * FROW + line;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint2 g = grid[base + m * FROW];
                vx[m] = g.x;
                vy[m] = g.y;
                grid[base + m * FROW] = make_uint2(0u, 0u);
            }
            stages_345<P, ALL>(vx, vy, wb, ts, rn, mask >> 6);
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint32_t x = vx[m], y = vy[m];
                uint32_t pr[4];
                pr[0] = (uint32_t)dot2(x, x, 0);
                if (P == 2) {
                    pr[1] = (uint32_t)dot2(y, y, 0);
                    pr[2] = (uint32_t)dot2(x, y, 0x7fffffff);
                    // xi yr - xr yi = xi yr + xr (~yi + 1)
                    pr[3] = (uint32_t)dot2(swap16(x), y ^ 0xffff0000u,
                                           (int)((uint32_t)((int)(x << 16) >> 16) + 0x7fffffffu));
                }
#pragma unroll
                for (int q = 0; q < NPROD; ++q)
                    acch[m][q] += __builtin_add_overflow(acc[m][q], pr[q], &acc[m][q]);
            }
        }
    }
    // position (8 j + m, line) holds frequency (brev(8 j + m), brev(line))
    double *dst = part + ((int64_t)slice * n_items + item) * NPROD * FN * FN;
    const int kx = brev6(line);
    const int64_t bias = (int64_t)max(0, t1 - t0) * 0x7fffffff;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int ky = brev6(8 * j + m);
#pragma unroll
        for (int q = 0; q < NPROD; ++q)
            dst[(int64_t)q * FN * FN + ky * FN + kx] =
                (double)((int64_t)(((uint64_t)acch[m][q] << 32) | acc[m][q]) - (q >= 2 ? bias : 0));
    }
    if (autos && tid < A) {
        int32_t *d = autos + ((int64_t)it.c * A + tid) * NPROD;
#pragma unroll
        for (int q = 0; q < NPROD; ++q) atomicAdd(d + q, sa[q]);
    }
}

// acc[img_off + q N^2 + pixel] += fl32(2^exp2 sum over slices of part).  The
// slice sums are exact integers, so their order does not matter.
__global__ void k_fixed_reduce(const FusedItem *__restrict__ items, int n_items, int n_slices,
                               int nprod, const double *__restrict__ part, double scale,
                               float *__restrict__ acc) {
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    const int q = blockIdx.y, item = blockIdx.z;
    if (pix >= FN * FN) return;
    double s = 0.0;
    for (int k = 0; k < n_slices; ++k)
        s += part[(((int64_t)k * n_items + item) * nprod + q) * FN * FN + pix];
    float *a = acc + items[item].img_off + (int64_t)q * FN * FN + pix;
    *a += (float)(s * scale);
}

// ------------------------------------------------------------ host build
int fixed_kernel_shift(const std::vector<double> &w) {
    double m = 0.0;
    for (double v : w) m = std::max(m, std::fabs(v));
    if (m == 0.0) return 0;
    int s = 40;
    while (m * std::ldexp(1.0, s) >= 127.5) --s;
    return s;
}

// Gather tables, twiddles and slice count; the weights w are already the
// effective (quantised) ones, q 2^-sw.
epic_status fixed_build(epic_plan p, const std::vector<int> &j0, const std::vector<double> &w,
                        hipStream_t s) {
    FixedPlan &F = p->fixed;
    const int A = p->A, K = p->K, C = p->C;
    const double up = std::ldexp(1.0, F.sw);
    const int vmax = p->vb == 2 ? 128 : 8;
    std::vector<FusedItem> items;
    std::vector<uint4> all;
    int64_t bmax = 0;
    for (int c = 0; c < C; ++c) {
        std::vector<GatherTap> taps;
        std::vector<int64_t> bound(FN * FN, 0);
        for (int a = 0; a < A; ++a) {
            const int jx0 = j0[((size_t)c * A + a) * 2], jy0 = j0[((size_t)c * A + a) * 2 + 1];
            for (int dy = 0; dy < K; ++dy)
                for (int dx = 0; dx < K; ++dx) {
                    const int jx = jx0 + dx, jy = jy0 + dy;
                    const size_t wi = (((size_t)c * A + a) * K * K + dy * K + dx) * 2;
                    const int qr = (int)std::nearbyint(w[wi] * up);
                    const int qi = (int)std::nearbyint(w[wi + 1] * up);
                    const int sg = ((jx + jy) & 1) ? -1 : 1;
                    GatherTap tp{};
                    tp.cell = jy * FROW + jx;
                    tp.ant = a;
                    // conj(q) (-1)^(jx+jy) as the operand (re, -im)
                    tp.wr = __builtin_bit_cast(float, ((uint32_t)(sg * qr) & 0xffffu) |
                                                          ((uint32_t)(sg * qi) << 16));
                    taps.push_back(tp);
                    bound[jy * FN + jx] += (int64_t)(std::abs(qr) + std::abs(qi)) * vmax;
                }
        }
        for (int64_t b : bound) bmax = std::max(bmax, b);
        FusedItem fi{};
        fi.c = c;
        fi.N = FN;
        fi.R = 1;
        fi.entry_off = (int64_t)all.size();
        fi.n_iter = lpt_pack(taps, FT, all);
        fi.img_off = p->ch[c].img_off;
        items.push_back(fi);
    }
    // the exact gridded sums are formed in int32
    if (bmax > 2147483647 - 65536)
        return fail(EPIC_ERR_UNSUPPORTED, "gridded sums could exceed 32 bits");
    if (F.sg < 0) {
        int sgv = 0;
        while (((bmax + ((int64_t{1} << sgv) >> 1)) >> sgv) > 32767) ++sgv;
        F.sg = sgv;
    }
    if (bmax + ((int64_t{1} << F.sg) >> 1) > 2147483647)
        return fail(EPIC_ERR_UNSUPPORTED, "gridded sums could exceed 32 bits with this grid shift");
    std::vector<int2> tw(FN / 2);
    for (int n = 0; n < FN / 2; ++n) {
        const double ang = 2.0 * M_PI * (double)n / (double)FN;
        tw[n] = make_int2((int)std::nearbyint(std::cos(ang) * std::ldexp(1.0, F.ts)),
                          (int)std::nearbyint(std::sin(ang) * std::ldexp(1.0, F.ts)));
    }
    int n_sh = 0;
    for (int b = 0; b < 12; ++b) n_sh += (F.mask >> b) & 1u;
    F.exp2 = 2 * (n_sh + F.sg - F.sw);
    // time slices: about 1024 workgroups in all, partial sums at most 256 MiB
    const int nprod = p->n_prod;
    const int64_t per_slice = (int64_t)C * nprod * FN * FN * (int64_t)sizeof(double);
    int S = std::max(1, (1024 + C - 1) / C);
    S = (int)std::min<int64_t>(S, std::max<int64_t>(1, (int64_t{256} << 20) / per_slice));
    F.slices = S;
    F.part_bytes = per_slice * S;
    F.n_items = C;
    // {element | last << 31, cell, operand} -> the kernel's 8-byte entries
    std::vector<uint2> packed(all.size());
    for (size_t i = 0; i < all.size(); ++i) {
        const uint32_t cell = (all[i].x >> 31) ? all[i].y : (uint32_t)(i % FN) * FROW + FN;
        packed[i] = make_uint2((all[i].x & 0x80003FFFu) | (cell << 14), all[i].z);
    }
    epic_status st;
    if ((st = F.items.alloc(sizeof(FusedItem) * items.size()))) return st;
    if ((st = F.entries.alloc(sizeof(uint2) * packed.size()))) return st;
    if ((st = F.tw.alloc(sizeof(int2) * tw.size()))) return st;
    EPIC_HIP(hipMemcpyAsync(F.items.p, items.data(), sizeof(FusedItem) * items.size(),
                            hipMemcpyHostToDevice, s));
    EPIC_HIP(hipMemcpyAsync(F.entries.p, packed.data(), sizeof(uint2) * packed.size(),
                            hipMemcpyHostToDevice, s));
    EPIC_HIP(hipMemcpyAsync(F.tw.p, tw.data(), sizeof(int2) * tw.size(), hipMemcpyHostToDevice, s));
    EPIC_HIP(hipStreamSynchronize(s));
    return EPIC_OK;
}

// dry: only give the kernel its LDS allowance (done before a graph capture).
epic_status fixed_accumulate(epic_plan p, epic_acc acc, const uint8_t *d_volt, int n_time,
                             hipStream_t s, bool dry) {
    const FixedPlan &F = p->fixed;
    const size_t lds = sizeof(uint2) * ((size_t)FN * FROW + (size_t)p->A);
    const bool halve = F.mask == 0xFFFu;
    auto kern = p->P == 2 ? (halve ? k_fixed64<2, true> : k_fixed64<2, false>)
                          : (halve ? k_fixed64<1, true> : k_fixed64<1, false>);
    epic_status st = lds_ready(reinterpret_cast<const void *>(kern), lds);
    if (st || dry) return st;
    // one element per thread: the kernel adds the self-term sums itself
    int32_t *autos = p->A <= FT ? acc->d_autos.as<int32_t>() : nullptr;
    const int tps = (n_time + F.slices - 1) / F.slices;
    const int used = (n_time + tps - 1) / tps;            // slices with samples
    double *part = acc->d_work.as<double>();
    dim3 grid((unsigned)(F.n_items * used));
    hipLaunchKernelGGL(kern, grid, dim3(FT), lds, s, F.items.as<FusedItem>(), F.n_items,
                       F.entries.as<uint2>(), d_volt, p->vstride(), p->A, n_time, tps,
                       F.tw.as<int2>(), F.ts, F.mask, F.sg, part, p->vb, autos);
    EPIC_HIP(hipGetLastError());
    dim3 rg(FN * FN / 256, p->n_prod, F.n_items);
    hipLaunchKernelGGL(k_fixed_reduce, rg, dim3(256), 0, s, F.items.as<FusedItem>(), F.n_items,
                       used, p->n_prod, part, std::ldexp(1.0, F.exp2), acc->d_acc.as<float>());
    EPIC_HIP(hipGetLastError());
    return autos ? EPIC_OK : autos_accumulate(p, acc, d_volt, n_time, s);
}

}  // namespace epic

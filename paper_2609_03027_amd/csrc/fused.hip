// Fused EPIC path: per time sample, gridding (Eq. 1 inner sum), the spatial
// transform (Eq. 1 outer sum) and the polarisation products (Eq. 2) stay in
// LDS and registers; only the time sums leave the chip.
//
// Decomposition.  With the centred transform of Eq. 1 written on integer
// indices,
//   E[k] = sum_j G[j] exp(+2 pi i (k - N/2)(j - N/2) / N)
//        = (-1)^k c_N sum_j (-1)^j G[j] exp(+2 pi i k j / N)     (per axis)
// and the factor (-1)^k c_N has modulus one and is the same for both feeds,
// so it cancels in |E|^2 and Ex conj(Ey).  Splitting k = R k' + o with
// N = R M,
//   sum_j (-1)^j G[j] e^{2 pi i (R k' + o) j / N}
//     = sum_{m<M} e^{2 pi i k' m / M} sum_{j = m mod M} (-1)^j e^{2 pi i o j / N} G[j],
// i.e. each output class o in [0, R)^2 is an M x M transform of a grid folded
// modulo M whose weights carry (-1)^(jx+jy) exp(+2 pi i (o . j) / N).  The
// plan folds those factors into the gather weights, so the kernel only ever
// runs M x M transforms (M = 16, 32, 64) with no index shifts.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <queue>

#include <mutex>

#include "internal.h"
#include "lines.h"
#include "slices.h"

namespace epic {

template <int M> struct FCfg;
template <> struct FCfg<64> { static constexpr int T = 512, RA = 8, RB = 8, ROW = 65; };
template <> struct FCfg<32> { static constexpr int T = 128, RA = 8, RB = 4, ROW = 33; };
template <> struct FCfg<16> { static constexpr int T = 64, RA = 4, RB = 4, ROW = 17; };

// Grid storage in LDS: with two feeds each element is a float4 (X re, X im,
// Y re, Y im), so one 16-byte access serves both feeds; one feed is float2.
template <int P> struct Grid;
template <> struct Grid<2> {
    float4 *g;
    __device__ __forceinline__ void load(int i, float2 &x, float2 &y) const {
        const float4 v = g[i];
        x = make_float2(v.x, v.y);
        y = make_float2(v.z, v.w);
    }
    __device__ __forceinline__ void store(int i, float2 x, float2 y) const {
        g[i] = make_float4(x.x, x.y, y.x, y.y);
    }
    __device__ __forceinline__ void zero(int i) const { g[i] = make_float4(0.f, 0.f, 0.f, 0.f); }
};
template <> struct Grid<1> {
    float2 *g;
    __device__ __forceinline__ void load(int i, float2 &x, float2 &) const { x = g[i]; }
    __device__ __forceinline__ void store(int i, float2 x, float2) const { g[i] = x; }
    __device__ __forceinline__ void zero(int i) const { g[i] = make_float2(0.f, 0.f); }
};

// ------------------------------------------------------- line transforms
// In place over one axis of an M x M grid stored with row pitch ROW.  Pass A
// (radix RA, stride M/RA) leaves frequency p of span position j at j + p M/RA;
// pass B (radix RB, stride 1) multiplies element q of block p by exp(+2 pi i
// p q / M) on the way into its butterflies.  After both passes position n of
// the axis holds frequency n / RB + RA (n % RB).
template <int M, int P, bool ALONG_X>
__device__ __forceinline__ void pass_a(Grid<P> g, int tid) {
    constexpr int RA = FCfg<M>::RA, ROW = FCfg<M>::ROW, S = M / RA;
    const int line = tid % M, j = tid / M;
    const int base = ALONG_X ? line * ROW + j : j * ROW + line;
    constexpr int step = ALONG_X ? S : S * ROW;
    float2 v0[RA], v1[RA];
#pragma unroll
    for (int q = 0; q < RA; ++q) g.load(base + q * step, v0[q], v1[q]);
    dft<RA>(v0);
    if (P == 2) dft<RA>(v1);
#pragma unroll
    for (int q = 0; q < RA; ++q) g.store(base + q * step, v0[q], v1[q]);
}

// Butterflies of pass B per thread, and their twiddles.
template <int M> constexpr int kNB = M * M / (FCfg<M>::RB * FCfg<M>::T);
template <int M> using PassTw = typename LineTw<M>::T[kNB<M>];

template <int M, int P, bool ALONG_X>
__device__ __forceinline__ void pass_b(Grid<P> g, int tid, const PassTw<M> &tw) {
    constexpr int T = FCfg<M>::T, RB = FCfg<M>::RB, ROW = FCfg<M>::ROW;
#pragma unroll
    for (int k = 0; k < kNB<M>; ++k) {
        const int u = tid + k * T;
        const int line = u % M, blk = u / M;
        const int base = ALONG_X ? line * ROW + blk * RB : blk * RB * ROW + line;
        constexpr int step = ALONG_X ? 1 : ROW;
        float2 v0[RB], v1[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) g.load(base + q * step, v0[q], v1[q]);
        dft_tw(v0, tw[k]);
        if (P == 2) dft_tw(v1, tw[k]);
#pragma unroll
        for (int q = 0; q < RB; ++q) g.store(base + q * step, v0[q], v1[q]);
    }
}

template <int M> __device__ __forceinline__ int unscramble(int n) {
    return n / FCfg<M>::RB + FCfg<M>::RA * (n % FCfg<M>::RB);
}

// Last pass (B along y) fused with the Eq. 2 products: the thread's
// butterflies end in registers, so their outputs go straight into its
// accumulators av[k RB + q] and the grid is left zeroed for the next gather.
// Output q of butterfly k sits at row blk RB + q, column line.
template <int M, int P, int NPROD>
__device__ __forceinline__ void pass_b_products(Grid<P> g, int tid, const PassTw<M> &tw,
                                                float (*av)[NPROD]) {
    constexpr int T = FCfg<M>::T, RB = FCfg<M>::RB, ROW = FCfg<M>::ROW;
#pragma unroll
    for (int k = 0; k < kNB<M>; ++k) {
        const int u = tid + k * T;
        const int line = u % M, blk = u / M;
        const int base = blk * RB * ROW + line;
        float2 v0[RB], v1[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) g.load(base + q * ROW, v0[q], v1[q]);
        dft_tw(v0, tw[k]);
        if (P == 2) dft_tw(v1, tw[k]);
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            g.zero(base + q * ROW);
            const float2 ex = v0[q];
            float *a = av[k * RB + q];
            a[0] = fmaf(ex.x, ex.x, fmaf(ex.y, ex.y, a[0]));
            if (P == 2) {
                const float2 ey = v1[q];
                a[1] = fmaf(ey.x, ey.x, fmaf(ey.y, ey.y, a[1]));
                a[2] = fmaf(ex.x, ey.x, fmaf(ex.y, ey.y, a[2]));
                a[3] = fmaf(ex.y, ey.x, fmaf(-ex.x, ey.y, a[3]));
            }
        }
    }
}

// Grid position (row, column) of accumulator slot s = k RB + q of a thread.
template <int M>
__device__ __forceinline__ void slot_position(int tid, int s, int &row, int &col) {
    constexpr int T = FCfg<M>::T, RB = FCfg<M>::RB;
    const int u = tid + (s / RB) * T;
    col = u % M;
    row = (u / M) * RB + s % RB;
}

// The rest of a Jones tap (the x <- x term is added by the caller): with the
// staged feeds v = (Ex re, Ex im, Ey re, Ey im) and folded conjugate weights
// from rows e1 = (xy, yx) and e2 = (yy, -), sx += w_xy Ey and
// sy += w_yx Ex + w_yy Ey.
__device__ __forceinline__ void jones_taps(const uint4 *r1, const uint4 *r2, const float4 v,
                                           float2 &sx, float2 &sy) {
    const uint4 e1 = *r1, e2 = *r2;
    const float ar = __uint_as_float(e1.x), ai = __uint_as_float(e1.y);
    const float br = __uint_as_float(e1.z), bi = __uint_as_float(e1.w);
    const float cr = __uint_as_float(e2.x), ci = __uint_as_float(e2.y);
    sx.x = fmaf(-ai, v.w, fmaf(ar, v.z, sx.x));
    sx.y = fmaf(ai, v.z, fmaf(ar, v.w, sx.y));
    sy.x = fmaf(-ci, v.w, fmaf(cr, v.z, fmaf(-bi, v.y, fmaf(br, v.x, sy.x))));
    sy.y = fmaf(ci, v.z, fmaf(cr, v.w, fmaf(bi, v.x, fmaf(br, v.y, sy.y))));
}

// One sample's gather.  Each lane owns whole cells; it loads GB entries at
// once (their L2 latencies overlap) and then applies them.  Every entry
// stores the running sum to its cell (the cell's last entry leaves the full
// sum, padding entries write a slot no pass reads) and the last one restarts
// it, so the loop body has no per-lane branches.  Entry: x = element |
// last-tap-of-cell << 31, y = LDS index of the folded cell, z/w = folded
// complex weight; with Jones kernels rows 1 and 2 follow at +T and +2T.
constexpr int GB = 8;   // gather entries in flight per lane

// The entry addresses do not change from sample to sample; the offset
// passes through an empty asm so the loads are not hoisted out of the
// sample loop (holding every entry in registers would cost occupancy).
__device__ __forceinline__ int opaque_zero() {
    int z = 0;
    asm volatile("" : "+v"(z));
    return z;
}

template <int T, bool JN>
__device__ __forceinline__ void gather_load(uint4 (&e)[GB], const uint4 *ent, int k0, int n_iter) {
    const uint4 *p = ent + opaque_zero();
#pragma unroll
    for (int k = 0; k < GB; ++k) e[k] = p[(int64_t)min(k0 + k, n_iter - 1) * (JN ? 3 : 1) * T];
}

// The caller loads the first batch (gather_load(e, ent, 0, n_iter)) ahead of
// the barrier that publishes the staged voltages, so its latency overlaps
// the wait; later batches are loaded here.
template <int T, int P, bool JN>
__device__ __forceinline__ void gather_cells(Grid<P> grid, const uint4 *ent, int n_iter,
                                             const float4 *stage, uint4 (&e)[GB]) {
    float2 sx = make_float2(0.f, 0.f), sy = make_float2(0.f, 0.f);
    for (int k0 = 0; k0 < n_iter; k0 += GB) {
        if (k0) gather_load<T, JN>(e, ent, k0, n_iter);
#pragma unroll
        for (int k = 0; k < GB; ++k) {
            if (k0 + k >= n_iter) break;            // uniform: n_iter is per wave
            const float4 v = stage[e[k].x & 0xFFFFu];
            const float wr = __uint_as_float(e[k].z), wi = __uint_as_float(e[k].w);
            sx.x = fmaf(-wi, v.y, fmaf(wr, v.x, sx.x));
            sx.y = fmaf(wi, v.x, fmaf(wr, v.y, sx.y));
            if (JN) {
                const int64_t r = (int64_t)(k0 + k) * 3 * T;
                jones_taps(ent + r + T, ent + r + 2 * T, v, sx, sy);
            } else if (P == 2) {
                sy.x = fmaf(-wi, v.w, fmaf(wr, v.z, sy.x));
                sy.y = fmaf(wi, v.z, fmaf(wr, v.w, sy.y));
            }
            grid.store(e[k].y, sx, sy);
            const bool last = (e[k].x >> 31) != 0u;
            sx = last ? make_float2(0.f, 0.f) : sx;
            sy = last ? make_float2(0.f, 0.f) : sy;
        }
    }
}

// ------------------------------------------------------------------ kernel
// One workgroup per item (channel c, class o), looping over all n_time
// samples.  Gather entry (uint4): x = element | last-tap-of-cell << 31,
// y = LDS index of the folded cell, z/w = folded complex weight (float bits).
// When `autos` is given (A <= 4 T), the class-(0,0) item of each channel also
// adds the per-element self-term sums S_a^{pq}, exact in int32.  AR is the
// number of element rounds whose self terms a thread keeps (A <= AR * T).
// FR: frame mode -- every frame_len samples the sums are stored to
// frames[t / frame_len] (stride fstride floats) and restarted; acc is not
// touched.  JN: Jones kernels (two feeds) -- each tap has three entry rows
// holding the weights x<-x, x<-y, y<-x, y<-y, and both feeds feed both
// grids.  Time slices: workgroup b takes item b % n_items and samples
// [s tps, (s + 1) tps) of slice s = b / n_items; with `part` given it stores
// its sums to part + s part_stride + it.part_off (k_fused_reduce adds the
// slices), else it adds them to acc.
// The work of one item for samples [t_begin, t_stop), run by the T threads
// tid = 0 .. T - 1 of one workgroup (or of a wave-aligned part of a larger
// one, which then holds every barrier with it): `gsm` is its grid in LDS,
// `stage` the staged voltages of the item's channel (parts running items of
// the same channel may share one stage: they write the same values).  With
// store false the sums and self terms are computed but not written.
template <int M, int P, int AR, bool FR, bool JN>
__device__ __forceinline__ void fused_item(const FusedItem &it,
                                           const uint4 *__restrict__ entries,
                                           const uint8_t *__restrict__ volt,
                                           int64_t volt_t_stride, int A, int t_begin, int t_stop,
                                           float *__restrict__ acc, int32_t *__restrict__ autos,
                                           int frame_len, float *__restrict__ frames,
                                           int64_t fstride, int vb, int slice,
                                           float *__restrict__ part, int64_t part_stride, int tid,
                                           float4 *gsm, float4 *stage, bool store, int n_iter) {
    constexpr int T = FCfg<M>::T;
    constexpr int NPIX = M * M / T;
    constexpr int NPROD = P == 2 ? 4 : 1;
    constexpr int GSZ = M * FCfg<M>::ROW;
    Grid<P> grid;
    grid.g = reinterpret_cast<decltype(grid.g)>(gsm);

    // with M = 64 the block index is the wave index: scalar loads and registers
    PassTw<M> tw;
#pragma unroll
    for (int k = 0; k < kNB<M>; ++k)
        tw[k] = LineTw<M>::at(M == 64 ? __builtin_amdgcn_readfirstlane(tid / M) : (tid + k * T) / M);
    for (int i = tid; i < GSZ; i += T) grid.zero(i);

    float av[NPIX][NPROD];
#pragma unroll
    for (int k = 0; k < NPIX; ++k)
#pragma unroll
        for (int q = 0; q < NPROD; ++q) av[k][q] = 0.f;

    const uint8_t *vbase = volt + (int64_t)it.c * P * A * vb;
    const uint4 *ent = entries + it.entry_off + tid;
    const bool own_autos = store && autos != nullptr && it.ox == 0 && it.oy == 0;
    int sa[AR][NPROD];
#pragma unroll
    for (int k = 0; k < AR; ++k)
#pragma unroll
        for (int q = 0; q < NPROD; ++q) sa[k][q] = 0;

    // this sample's voltages for elements tid + k T, loaded one sample ahead
    // (during the previous sample's gather and transform)
    uint32_t rx[AR], ry[AR];
#pragma unroll
    for (int k = 0; k < AR; ++k) {
        const int a = tid + k * T;
        rx[k] = ry[k] = 0u;
        if (a < A && t_begin < t_stop) {
            const uint8_t *v0 = vbase + (int64_t)t_begin * volt_t_stride;
            rx[k] = volt_raw(v0, a, vb);
            ry[k] = P == 2 ? volt_raw(v0, A + a, vb) : 0u;
        }
    }
    for (int t = t_begin; t < t_stop; ++t) {
        const uint8_t *vt = vbase + (int64_t)t * volt_t_stride;
        uint4 e[GB];
        gather_load<T, JN>(e, ent, 0, n_iter);
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A) {
                const int2 vx = volt_dec(rx[k], vb);
                const int2 vy = P == 2 ? volt_dec(ry[k], vb) : make_int2(0, 0);
                const int xr = vx.x, xi = vx.y, yr = vy.x, yi = vy.y;
                stage[a] = make_float4((float)xr, (float)xi, (float)yr, (float)yi);
                if (own_autos) {
                    sa[k][0] += xr * xr + xi * xi;
                    if (P == 2) {
                        sa[k][1] += yr * yr + yi * yi;
                        sa[k][2] += xr * yr + xi * yi;
                        sa[k][3] += xi * yr - xr * yi;
                    }
                }
            }
        }
        for (int a = tid + AR * T; a < A; a += T) {
            const int2 vx = volt_at(vt, a, vb);
            const int2 vy = P == 2 ? volt_at(vt, A + a, vb) : make_int2(0, 0);
            stage[a] = make_float4((float)vx.x, (float)vx.y, (float)vy.x, (float)vy.y);
        }
        __syncthreads();

        if (t + 1 < t_stop) {
            const uint8_t *vn = vt + volt_t_stride;
#pragma unroll
            for (int k = 0; k < AR; ++k) {
                const int a = tid + k * T;
                if (a < A) {
                    rx[k] = volt_raw(vn, a, vb);
                    ry[k] = P == 2 ? volt_raw(vn, A + a, vb) : 0u;
                }
            }
        }
        gather_cells<T, P, JN>(grid, ent, n_iter, stage, e);
        __syncthreads();

        pass_a<M, P, true>(grid, tid);
        __syncthreads();
        pass_b<M, P, true>(grid, tid, tw);
        __syncthreads();
        pass_a<M, P, false>(grid, tid);
        __syncthreads();
        // last pass + Eq. 2 products; the grid is left zeroed, and the stage
        // barrier of the next sample orders these writes before the gather
        pass_b_products<M, P, NPROD>(grid, tid, tw, av);
        if (FR && (t + 1) % frame_len == 0) {
            const int N = it.N, R = it.R;
            const int64_t plane = (int64_t)N * N;
            float *fr = frames + (int64_t)(t / frame_len) * fstride + it.img_off;
#pragma unroll
            for (int k = 0; k < NPIX; ++k) {
                int row, col;
                slot_position<M>(tid, k, row, col);
                const int ky = R * unscramble<M>(row) + it.oy;
                const int kx = R * unscramble<M>(col) + it.ox;
                float *dst = fr + (int64_t)ky * N + kx;
#pragma unroll
                for (int q = 0; q < NPROD; ++q) {
                    dst[q * plane] = av[k][q];
                    av[k][q] = 0.f;
                }
            }
        }
    }

    const int N = it.N, R = it.R;
    const int64_t plane = (int64_t)N * N;
    if (!FR && store) {
        float *base = part ? part + slice * part_stride + it.part_off : acc + it.img_off;
#pragma unroll
        for (int k = 0; k < NPIX; ++k) {
            int row, col;
            slot_position<M>(tid, k, row, col);
            const int ky = R * unscramble<M>(row) + it.oy;
            const int kx = R * unscramble<M>(col) + it.ox;
            float *dst = base + (int64_t)ky * N + kx;
#pragma unroll
            for (int q = 0; q < NPROD; ++q) {
                if (part)
                    dst[q * plane] = av[k][q];
                else
                    dst[q * plane] += av[k][q];
            }
        }
    }
    if (own_autos) {
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A) {
                int32_t *d = autos + ((int64_t)it.c * A + a) * NPROD;
#pragma unroll
                for (int q = 0; q < NPROD; ++q) atomicAdd(d + q, sa[k][q]);
            }
        }
    }
}

template <int M, int P, int AR, bool FR, bool JN>
__global__ __launch_bounds__(FCfg<M>::T) __attribute__((amdgpu_waves_per_eu(4))) void k_fused(const FusedItem *__restrict__ items,
                                                      const uint4 *__restrict__ entries,
                                                      const uint8_t *__restrict__ volt,
                                                      int64_t volt_t_stride, int A, int n_time,
                                                      float *__restrict__ acc,
                                                      int32_t *__restrict__ autos,
                                                      int frame_len, float *__restrict__ frames,
                                                      int64_t fstride, int vb, int n_items,
                                                      int tps, float *__restrict__ part,
                                                      int64_t part_stride) {
    constexpr int GSZ = M * FCfg<M>::ROW;
    extern __shared__ float4 smem[];
    float4 *stage = reinterpret_cast<float4 *>(reinterpret_cast<float2 *>(smem) + P * GSZ);
    const int slice = blockIdx.x / n_items;
    const FusedItem &it = items[blockIdx.x % n_items];
    if (it.c < 0) return;
    const int t_begin = slice * tps, t_stop = min(n_time, t_begin + tps);
    const int n_iter = it.wave_iter[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
    fused_item<M, P, AR, FR, JN>(it, entries, volt, volt_t_stride, A, t_begin, t_stop, acc, autos,
                                 frame_len, frames, fstride, vb, slice, part, part_stride,
                                 (int)threadIdx.x, smem, stage, true, n_iter);
}

// ------------------------------------------------- persistent work queue
// Every fused class item of a plan in one launch (EPIC_BATCH_QUEUE).  Each
// 512-thread workgroup takes the next unit from a device counter until the
// table is used up, so the exit condition is the same for every wave and no
// workgroup waits for another.  A unit is one 64 x 64 item (all 512 threads),
// or a bundle of four 32 x 32 (128 threads each) or eight 16 x 16 (64 each)
// items of one channel: the parts run side by side, hold every barrier
// together (their sample loops are the same length) and share one staging
// of the channel's voltages (each part writes the same values to it).  Unused
// slots of a bundle rerun its last item without storing.  Units are ordered
// largest transform first.  Self terms come from the separate pass.
constexpr int kQueueGrid = 4224;   // float2 per feed: max(64 x 65, 4 x 32 x 33, 8 x 16 x 17)

// Per size (64, 32, 16): items, entries, samples per slice, slices in use
// and the partial image sets when there is more than one.
struct QueueSizes {
    const FusedItem *it[3];
    const uint4 *e[3];
    float *part[3];
    int64_t pstride[3];
    int tps[3];
    int used[3];
};

template <int P>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_fused_queue(
    const QueueUnit *__restrict__ units, int n_units, unsigned int *__restrict__ head,
    const QueueSizes qs, const uint8_t *__restrict__ volt, int64_t vstride, int A, int n_time,
    int vb, float *__restrict__ acc) {
    extern __shared__ float4 smem[];
    float4 *stage = reinterpret_cast<float4 *>(reinterpret_cast<float2 *>(smem) + P * kQueueGrid);
    // the unit number, after the stage (dynamic LDS only: the whole allowance
    // is given to the dynamic part)
    int &cur = *reinterpret_cast<int *>(stage + A);
    const int tid0 = threadIdx.x;
    for (;;) {
        if (tid0 == 0) cur = (int)atomicAdd(head, 1u);
        __syncthreads();
        const int u = cur;
        __syncthreads();                  // every thread has read cur
        if (u >= n_units) break;          // the same for the whole workgroup
        const QueueUnit *q = units + u;
        const int M = q->M, n = q->n, sl = q->slice;
        // per unit, so the bodies' thread-dependent set-up (twiddles, LDS
        // addresses) is not hoisted out of the unit loop and kept live across it
        const int tid = tid0 + opaque_zero();
        if (M == 64) {
            if (sl >= qs.used[0]) continue;   // a slice beyond this call's samples
            const int t_begin = sl * qs.tps[0], t_stop = min(n_time, t_begin + qs.tps[0]);
            const FusedItem &it = qs.it[0][q->idx[0]];
            const int wi = it.wave_iter[__builtin_amdgcn_readfirstlane(tid >> 6)];
            fused_item<64, P, 1, false, false>(it, qs.e[0], volt, vstride, A, t_begin, t_stop,
                                               acc, nullptr, 0, nullptr, 0, vb, sl, qs.part[0],
                                               qs.pstride[0], tid, smem, stage, true, wi);
        } else if (M == 32) {
            if (sl >= qs.used[1]) continue;
            const int t_begin = sl * qs.tps[1], t_stop = min(n_time, t_begin + qs.tps[1]);
            // sub-group index and grid base are wave-uniform
            const int sub = __builtin_amdgcn_readfirstlane(tid >> 7);
            const FusedItem &it = qs.it[1][q->idx[min(sub, n - 1)]];
            const int wi = it.wave_iter[__builtin_amdgcn_readfirstlane((tid & 127) >> 6)];
            float4 *g = reinterpret_cast<float4 *>(reinterpret_cast<float2 *>(smem) +
                                                   sub * P * 32 * FCfg<32>::ROW);
            fused_item<32, P, 1, false, false>(it, qs.e[1], volt, vstride, A, t_begin, t_stop,
                                               acc, nullptr, 0, nullptr, 0, vb, sl, qs.part[1],
                                               qs.pstride[1], tid & 127, g, stage, sub < n, wi);
        } else {
            if (sl >= qs.used[2]) continue;
            const int t_begin = sl * qs.tps[2], t_stop = min(n_time, t_begin + qs.tps[2]);
            const int sub = __builtin_amdgcn_readfirstlane(tid >> 6);
            const FusedItem &it = qs.it[2][q->idx[min(sub, n - 1)]];
            float4 *g = reinterpret_cast<float4 *>(reinterpret_cast<float2 *>(smem) +
                                                   sub * P * 16 * FCfg<16>::ROW);
            // parts of different channels stage into their own slot after
            // the eight 16 x 16 grids (inside the grid area the other sizes use)
            float4 *st = q->own_stage ? reinterpret_cast<float4 *>(reinterpret_cast<float2 *>(smem) +
                                                                   8 * P * 16 * FCfg<16>::ROW) +
                                            sub * A
                                      : stage;
            fused_item<16, P, 1, false, false>(it, qs.e[2], volt, vstride, A, t_begin, t_stop,
                                               acc, nullptr, 0, nullptr, 0, vb, sl, qs.part[2],
                                               qs.pstride[2], tid & 63, g, st, sub < n,
                                               it.n_iter);
        }
        __syncthreads();                  // the unit's last LDS reads before the next unit
    }
}

__global__ void k_queue_reset(unsigned int *head) { *head = 0u; }

// ------------------------------------------------- paired-class kernel
// For N = 2 M grids (M = 64) whose element rows span at most M rows and two
// feeds, classes (ox, 0) and (ox, 1) share everything up to the y-pass.  With
// the rows counted from the first one an element touches (which multiplies
// both feeds' output by the same phase), row m of class oy carries the factor
// exp(+2 pi i oy m / N), which commutes with the transform along x.  One
// workgroup per (channel, ox) grids once, transforms along x once, and along y
// once per class.
//
// A wave owns eight whole rows in the x-pass and eight whole columns in the
// y-pass, so both radix-8 steps of an axis exchange inside the wave (LDS
// operations of one wave execute in order: no barrier).  Two grids in LDS
// alternate between samples, and a sample takes two barriers:
//   phase 1: y-pass and products of sample t (grid t & 1, own columns), and
//            the gather of sample t + 1 into the other grid;
//   phase 2: x-pass of sample t + 1 (own rows), staging of sample t + 2.
// In phase 1 the waves 0-3 (one per SIMD) gather first and the waves 4-7
// transform first, so that each SIMD has one wave waiting on LDS and one
// issuing arithmetic.  Bound: vector issue, 1019 instructions per thread and
// sample on 8 waves and 4 SIMDs (79 % of the cycles; LDS is busy for 47 %).
// LWA-like station (128 channels, 256 elements), 1000 samples: 4.45 ms (4.6 ms
// with rows and columns in natural order, see pair_pos).  With
// workgroup-wide passes (five barriers a sample, both classes' inputs through
// LDS, 1126 instructions) it took 5.23 ms; 250 samples with Jones kernels 1.27
// against 2.26 ms, where every tap's two further rows waited for L2 in turn.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kPairRow = 65, kPairGrid = 64 * kPairRow;
// elements whose staged voltages fit beside the two grids in a CU's 160 KiB: 1920
constexpr int kPairMaxAnt = 160 * 1024 / 16 - 2 * kPairGrid;

// The gather puts grid row or column m = j + 8 q at position 8 j + q: a 16-byte
// read serves 16 lanes at once, eight rows (or columns) of two neighbouring j,
// whose positions then differ by eight: no bank is met twice.
__host__ __device__ constexpr int pair_pos(int m) { return 8 * (m % 8) + m / 8; }

// y-pass of both classes on the wave's columns and the products; lane = column
// c + 8 j.  Class oy's second step leaves row frequency b + 8 q in accumulator
// oy 8 + q of lane b.  The columns are zeroed.
__device__ __forceinline__ void pair_y(float4 *col, int j, const Tw8 (&tw)[2], float (&av)[16][4]) {
    Grid<2> g;
    g.g = col;
    const int ia = j * kPairRow, ib = j * 8 * kPairRow;
    float2 vx[8], vy[8], ax[8], ay[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        g.load(ib + q * kPairRow, vx[q], vy[q]);
        ax[q] = vx[q];
        ay[q] = vy[q];
    }
    // each exchange's LDS latency is covered by the other class's arithmetic
    auto exchange = [&](float2 *x, float2 *y) {
        wave_sync();
#pragma unroll
        for (int p = 0; p < 8; ++p) g.store(ia + p * 8 * kPairRow, x[p], y[p]);
        wave_sync();
#pragma unroll
        for (int q = 0; q < 8; ++q) g.load(ib + q * kPairRow, x[q], y[q]);
    };
    auto products = [&](const float2 *x, const float2 *y, int s0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float *a = av[s0 + q];
            a[0] = fmaf(x[q].x, x[q].x, fmaf(x[q].y, x[q].y, a[0]));
            a[1] = fmaf(y[q].x, y[q].x, fmaf(y[q].y, y[q].y, a[1]));
            a[2] = fmaf(x[q].x, y[q].x, fmaf(x[q].y, y[q].y, a[2]));
            a[3] = fmaf(x[q].y, y[q].x, fmaf(-x[q].x, y[q].y, a[3]));
        }
    };
    dft<8>(ax);
    dft<8>(ay);
    exchange(ax, ay);
    dft8_root16(vx);
    dft8_root16(vy);
    exchange(vx, vy);
    dft8_tw(ax, tw[0]);
    dft8_tw(ay, tw[0]);
    products(ax, ay, 0);
    wave_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) g.zero(ib + q * kPairRow);
    dft8_tw(vx, tw[1]);
    dft8_tw(vy, tw[1]);
    products(vx, vy, 8);
}

// x-pass on the wave's rows; lane = row r + 8 j.  The second step stores
// frequency b + 8 q at column b + 8 q: natural order.
__device__ __forceinline__ void pair_x(float4 *row, int j, const Tw8 &tw) {
    Grid<2> g;
    g.g = row;
    float2 vx[8], vy[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) g.load(8 * j + q, vx[q], vy[q]);
    dft<8>(vx);
    dft<8>(vy);
    wave_sync();
#pragma unroll
    for (int p = 0; p < 8; ++p) g.store(j + 8 * p, vx[p], vy[p]);
    wave_sync();
#pragma unroll
    for (int q = 0; q < 8; ++q) g.load(8 * j + q, vx[q], vy[q]);
    wave_sync();
    dft8_tw(vx, tw);
    dft8_tw(vy, tw);
#pragma unroll
    for (int q = 0; q < 8; ++q) g.store(j + 8 * q, vx[q], vy[q]);
}

// A gather entry in registers: element | cell << 16 | last-tap-of-cell << 31.
struct PairTap {
    uint32_t ac;
    float wr, wi;
};
__device__ __forceinline__ PairTap pair_tap(uint4 e) {
    return PairTap{e.x | (e.y << 16), __uint_as_float(e.z), __uint_as_float(e.w)};
}
// With Jones kernels a tap's three rows.
struct JonesTap {
    uint4 r[3];
};

// One sample's gather (see gather_cells); the lists do not change from sample
// to sample, so the first 2 B taps of a lane stay in registers, and a batch's
// staged voltages are read before its first sum.  Longer lists stream from L2.
template <int B>
__device__ __forceinline__ void pair_gather(float4 *grid, const uint4 *ent, int n_iter,
                                            const float4 *stage, const PairTap (&held)[2 * B]) {
    constexpr int T = 512;
    float2 sx = make_float2(0.f, 0.f), sy = make_float2(0.f, 0.f);
    auto batch = [&](const PairTap (&e)[B], int k0) {
        float4 v[B];
#pragma unroll
        for (int k = 0; k < B; ++k) v[k] = stage[e[k].ac & 0xFFFFu];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            if (k0 + k >= n_iter) break;            // uniform: n_iter is per wave
            const float wr = e[k].wr, wi = e[k].wi;
            sx.x = fmaf(-wi, v[k].y, fmaf(wr, v[k].x, sx.x));
            sx.y = fmaf(wi, v[k].x, fmaf(wr, v[k].y, sx.y));
            sy.x = fmaf(-wi, v[k].w, fmaf(wr, v[k].z, sy.x));
            sy.y = fmaf(wi, v[k].z, fmaf(wr, v[k].w, sy.y));
            grid[(e[k].ac >> 16) & 0x7FFFu] = make_float4(sx.x, sx.y, sy.x, sy.y);
            const bool last = (e[k].ac >> 31) != 0u;
            sx = last ? make_float2(0.f, 0.f) : sx;
            sy = last ? make_float2(0.f, 0.f) : sy;
        }
    };
    PairTap e[B];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h * B >= n_iter) break;
#pragma unroll
        for (int k = 0; k < B; ++k) {
            e[k] = held[h * B + k];
            asm volatile("" : "+v"(e[k].ac));       // decoded per sample, not kept decoded
        }
        batch(e, h * B);
    }
    // no load of an entry stays in flight past its batch: the y-pass after the
    // gather would have to wait for it, and so for the newer voltage loads
    for (int k0 = 2 * B; k0 < n_iter; k0 += B) {
        const uint4 *p = ent + opaque_zero();
#pragma unroll
        for (int k = 0; k < B; ++k) e[k] = pair_tap(p[(int64_t)min(k0 + k, n_iter - 1) * T]);
        batch(e, k0);
    }
}

// The Jones gather: B taps of three rows at a time, the next batch (after the
// last one, the next sample's first) loaded while one is applied; nxt holds
// batch 0 on entry and on return.
template <int B>
__device__ __forceinline__ void pair_gather_jones(float4 *grid, const uint4 *ent, int n_iter,
                                                  const float4 *stage, JonesTap (&nxt)[B]) {
    constexpr int T = 512;
    float2 sx = make_float2(0.f, 0.f), sy = make_float2(0.f, 0.f);
    for (int k0 = 0; k0 < n_iter; k0 += B) {
        JonesTap e[B];
        float4 v[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            e[k] = nxt[k];
            v[k] = stage[e[k].r[0].x & 0xFFFFu];
        }
        const uint4 *p = ent + opaque_zero();
        const int k1 = k0 + B < n_iter ? k0 + B : 0;
#pragma unroll
        for (int k = 0; k < B; ++k)
#pragma unroll
            for (int r = 0; r < 3; ++r)
                nxt[k].r[r] = p[(int64_t)(min(k1 + k, n_iter - 1) * 3 + r) * T];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            if (k0 + k >= n_iter) break;            // uniform
            const float wr = __uint_as_float(e[k].r[0].z), wi = __uint_as_float(e[k].r[0].w);
            sx.x = fmaf(-wi, v[k].y, fmaf(wr, v[k].x, sx.x));
            sx.y = fmaf(wi, v[k].x, fmaf(wr, v[k].y, sx.y));
            jones_taps(&e[k].r[1], &e[k].r[2], v[k], sx, sy);
            grid[e[k].r[0].y] = make_float4(sx.x, sx.y, sy.x, sy.y);
            const bool last = (e[k].r[0].x >> 31) != 0u;
            sx = last ? make_float2(0.f, 0.f) : sx;
            sy = last ? make_float2(0.f, 0.f) : sy;
        }
    }
}

// Time slices as in k_fused: workgroup b takes item b % n_items and samples
// [s tps, (s + 1) tps) of slice s = b / n_items, and with `part` given stores
// its sums there for k_fused_reduce.
template <int AR, bool FR, bool JN>
__global__ __launch_bounds__(512) void k_fused_pair(const FusedItem *__restrict__ items,
                                                    const uint4 *__restrict__ entries,
                                                    const uint8_t *__restrict__ volt,
                                                    int64_t volt_t_stride, int A, int n_time,
                                                    float *__restrict__ acc,
                                                    int32_t *__restrict__ autos, int frame_len,
                                                    float *__restrict__ frames, int64_t fstride,
                                                    int vb, int n_items, int tps,
                                                    float *__restrict__ part, int64_t part_stride) {
    constexpr int T = 512;
    extern __shared__ float4 smem[];
    float4 *stage = smem + 2 * kPairGrid;

    const int slice = blockIdx.x / n_items;
    const FusedItem &it = items[blockIdx.x % n_items];
    if (it.c < 0) return;
    // sample numbers that may pass n_time (up to 2^31 - 1 in frame mode) are unsigned
    const int t0 = slice * tps, t1 = (int)min((uint32_t)n_time, (uint32_t)t0 + (uint32_t)tps);
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lo = tid & 7, j = (tid >> 3) & 7;

    const Tw8 tw[2] = {kRoots.r8[2 * j], kRoots.r8[2 * j + 1]};   // x-pass and class 0; class 1
    for (int i = tid; i < 2 * kPairGrid; i += T) smem[i] = make_float4(0.f, 0.f, 0.f, 0.f);

    float av[16][4];
#pragma unroll
    for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) av[k][q] = 0.f;

    const uint8_t *vbase = volt + (int64_t)it.c * 2 * A * vb;
    const uint4 *ent = entries + it.entry_off + tid;
    const int n_iter = it.wave_iter[w];
    const bool own_autos = autos != nullptr && it.ox == 0;
    int sa[AR][4];
    uint32_t rx[AR], ry[AR];             // the next sample's voltages of elements tid + k T
    auto fetch = [&](uint32_t t) {
        const uint8_t *vt = vbase + (int64_t)t * volt_t_stride;
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A && t < (uint32_t)t1) {
                rx[k] = volt_raw(vt, a, vb);
                ry[k] = volt_raw(vt, A + a, vb);
            }
        }
    };
    auto put = [&](uint32_t t) {              // stage sample t, add its self terms
        if (t >= (uint32_t)t1) return;
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A) {
                const int2 vx = volt_dec(rx[k], vb), vy = volt_dec(ry[k], vb);
                const int xr = vx.x, xi = vx.y, yr = vy.x, yi = vy.y;
                stage[a] = make_float4((float)xr, (float)xi, (float)yr, (float)yi);
                if (own_autos) {
                    sa[k][0] += xr * xr + xi * xi;
                    sa[k][1] += yr * yr + yi * yi;
                    sa[k][2] += xr * yr + xi * yi;
                    sa[k][3] += xi * yr - xr * yi;
                }
            }
        }
    };
#pragma unroll
    for (int k = 0; k < AR; ++k) {
        rx[k] = ry[k] = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) sa[k][q] = 0;
    }
    fetch((uint32_t)t0);
    constexpr int HB = JN ? 1 : 5, JB = JN ? 3 : 1;
    PairTap held[2 * HB];
    JonesTap jt[JB];
    if (JN) {
#pragma unroll
        for (int k = 0; k < JB; ++k)
#pragma unroll
            for (int r = 0; r < 3; ++r) jt[k].r[r] = ent[(int64_t)(min(k, n_iter - 1) * 3 + r) * T];
    } else {
#pragma unroll
        for (int k = 0; k < 2 * HB; ++k) held[k] = pair_tap(ent[(int64_t)min(k, n_iter - 1) * T]);
    }
    put((uint32_t)t0);
    fetch((uint32_t)t0 + 1u);
    __syncthreads();

    for (int t = t0 - 1; t < t1; ++t) {
        float4 *cur = smem + (t & 1) * kPairGrid, *oth = smem + ((t + 1) & 1) * kPairGrid;
        // phase 1
        auto gather = [&]() {
            if constexpr (JN)
                pair_gather_jones<JB>(oth, ent, n_iter, stage, jt);
            else
                pair_gather<HB>(oth, ent, n_iter, stage, held);
        };
        if (w < 4 && t + 1 < t1) gather();
        if (t >= t0) pair_y(cur + 8 * w + lo, j, tw, av);
        if (w >= 4 && t + 1 < t1) gather();
        if (FR && t >= t0 && (t + 1) % frame_len == 0) {
            const int N = it.N;
            const int64_t plane = (int64_t)N * N;
            float *fr = frames + (int64_t)(t / frame_len) * fstride + it.img_off;
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int ky = 2 * (j + 8 * (s & 7)) + (s >> 3), kx = 2 * (8 * w + lo) + it.ox;
                float *dst = fr + (int64_t)ky * N + kx;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    dst[p * plane] = av[s][p];
                    av[s][p] = 0.f;
                }
            }
        }
        __syncthreads();
        // phase 2
        if (t + 1 < t1) {
            put((uint32_t)t + 2u);
            fetch((uint32_t)t + 3u);
            pair_x(oth + (8 * w + lo) * kPairRow, j, tw[0]);
            __syncthreads();
        }
    }

    if (!FR) {
        const int N = it.N;
        const int64_t plane = (int64_t)N * N;
        float *base = part ? part + slice * part_stride + it.part_off : acc + it.img_off;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int ky = 2 * (j + 8 * (s & 7)) + (s >> 3), kx = 2 * (8 * w + lo) + it.ox;
            float *dst = base + (int64_t)ky * N + kx;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if (part)
                    dst[p * plane] = av[s][p];
                else
                    dst[p * plane] += av[s][p];
            }
        }
    }
    if (own_autos) {
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A) {
                int32_t *d = autos + ((int64_t)it.c * A + a) * 4;
#pragma unroll
                for (int p = 0; p < 4; ++p) atomicAdd(d + p, sa[k][p]);
            }
        }
    }
}

// ------------------------------------------------- row-unfolded kernel
// Grids of side N = 3 M (96, 48) whose element rows span at most N / 2, two feeds.
// One class per item grids the channel nine times and transforms all M rows of
// every folded class.  Here an item is one class ox of the x axis (3 M columns
// folded modulo M) with its rows unfolded: it grids once into N / 2 rows,
// transforms them along x, and each of the three classes oy of the y axis folds the
// rows it needs in registers: row m = j + S q (S = M / RA) carries
// exp(+2 pi i oy m / N) = exp(2 pi i oy j / N) exp(2 pi i oy q / (3 RA)) and row m + M a
// further exp(2 pi i oy / 3), so class oy is the transform of
//   u_q = v_q + exp(2 pi i oy / 3) v_{q+RA}     (q < RA / 2, else u_q = v_q)
// with the constant input twiddles exp(2 pi i oy / (3 RA)), and the factor of j
// goes into the second step's twiddles, w = exp(2 pi i (3 p + oy) / N) on block p.
// Rows are counted from the first one an element touches (see k_fused_pair).
//
// Waves own rows in the x-pass (16 at a time, dealt to the waves from one that
// turns with the workgroup, since three groups on two waves leave half of the
// SIMDs with twice the work) and columns in the y-pass: three barriers a sample.
// Bound: vector issue and LDS latency at two waves per SIMD (the sums, the held
// rows and two classes in work take 250 registers).  256 elements, 512 samples:
// 81 channels of 96^2 1.22 ms against 1.98 with one class per item, 40 of 48^2 0.26
// against 0.66.  192^2 in this form (12 rows a lane, MX = 32) took 7.5 ms for 139
// channels against 7.3: two waves per SIMD instead of four cost it more than a
// third of the arithmetic.
template <int M_> struct RowsCfg {
    static constexpr int M = M_;
    static constexpr int RAX = M == 32 ? 8 : 4;        // x lines: RAX x 4
    static constexpr int RA = M == 16 ? 4 : 8;         // y lines: RA x S
    static constexpr int S = M / RA;
    static constexpr int T = M * S;                    // threads
    static constexpr int CW = 64 / S;                  // columns per wave
    static constexpr int NB = RA / S;                  // second-step blocks per lane
    static constexpr int QV = RA + RA / 2;             // rows per lane
    static constexpr int ROW = M + 1;
    static constexpr int H = QV * S;                   // rows in LDS: N / 2
    static constexpr int N = 3 * M;
    using Tw = Tw4;
    // LDS row of grid row j + S q (cf. pair_pos): rows of one j lie together
    static __host__ __device__ constexpr int row(int j, int q) {
        return q < RA ? RA * j + q : M + (RA / 2) * j + q - RA;
    }
    static constexpr size_t lds(int A) {
        return sizeof(float4) * ((size_t)H * ROW + A) + sizeof(Tw) * 3 * RA;
    }
};

// Class oy of the first y step: fold, then transform with constant twiddles.
template <int OY> __device__ __forceinline__ void rows_first(const float2 (&v)[12], float2 *u) {
    constexpr Root third = root_of(OY, 3);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        u[q] = v[q];
        if (q < 4) {
            const float2 b = v[q + 8];
            if (OY == 0)
                u[q] = cadd(v[q], b);
            else
                u[q] = make_float2(fmaf(third.c, fmaf(-third.t, b.y, b.x), v[q].x),
                                   fmaf(third.c, fmaf(third.t, b.x, b.y), v[q].y));
        }
    }
    if (OY == 0) {
        dft<8>(u);
    } else {
        constexpr Tw8 w = tw8_of(OY, 24);
        dft8_tw(u, w);
    }
}
template <int OY> __device__ __forceinline__ void rows_first(const float2 (&v)[6], float2 *u) {
    constexpr Root third = root_of(OY, 3);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        u[q] = v[q];
        if (q < 2) {
            const float2 b = v[q + 4];
            if (OY == 0)
                u[q] = cadd(v[q], b);
            else
                u[q] = make_float2(fmaf(third.c, fmaf(-third.t, b.y, b.x), v[q].x),
                                   fmaf(third.c, fmaf(third.t, b.x, b.y), v[q].y));
        }
    }
    if (OY == 0) {
        dft<4>(u);
    } else {
        constexpr Tw4 w = tw4_of(OY, 12);
        dft4_tw(u, w);
    }
}

// The gather (see gather_cells), with a batch's staged voltages read before its
// first sum: the registers of the y-pass are free here, so twelve entries and
// their voltages are in flight.  The first twelve are loaded by the caller.
constexpr int RG = 12;
template <int T>
__device__ __forceinline__ void rows_load(uint4 (&e)[RG], const uint4 *ent, int k0, int n_iter) {
    const uint4 *p = ent + opaque_zero();
#pragma unroll
    for (int k = 0; k < RG; ++k) e[k] = p[(int64_t)min(k0 + k, n_iter - 1) * T];
}
template <int T>
__device__ __forceinline__ void rows_gather(float4 *grid, const uint4 *ent, int n_iter,
                                            const float4 *stage, uint4 (&e)[RG]) {
    constexpr int B = 4;
    float2 sx = make_float2(0.f, 0.f), sy = make_float2(0.f, 0.f);
    for (int k0 = 0; k0 < n_iter; k0 += RG) {
        if (k0) rows_load<T>(e, ent, k0, n_iter);
#pragma unroll
        for (int h = 0; h < RG; h += B) {
            if (k0 + h >= n_iter) break;             // uniform: n_iter is per wave
            float4 v[B];
#pragma unroll
            for (int k = 0; k < B; ++k) v[k] = stage[e[h + k].x & 0xFFFFu];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                if (k0 + h + k >= n_iter) break;
                const float wr = __uint_as_float(e[h + k].z), wi = __uint_as_float(e[h + k].w);
                sx.x = fmaf(-wi, v[k].y, fmaf(wr, v[k].x, sx.x));
                sx.y = fmaf(wi, v[k].x, fmaf(wr, v[k].y, sx.y));
                sy.x = fmaf(-wi, v[k].w, fmaf(wr, v[k].z, sy.x));
                sy.y = fmaf(wi, v[k].z, fmaf(wr, v[k].w, sy.y));
                grid[e[h + k].y] = make_float4(sx.x, sx.y, sy.x, sy.y);
                const bool last = (e[h + k].x >> 31) != 0u;
                sx = last ? make_float2(0.f, 0.f) : sx;
                sy = last ? make_float2(0.f, 0.f) : sy;
            }
        }
    }
}

// x-pass of 16 rows; lane = row r + 16 j.
template <int M>
__device__ __forceinline__ void rows_x(float4 *grid, int row, int j, const Tw4 *tw) {
    using C = RowsCfg<M>;
    constexpr int RAX = C::RAX, NBX = RAX / 4;
    if (row >= C::H) return;
    Grid<2> g;
    g.g = grid + row * C::ROW;
    {
        float2 x[RAX], y[RAX];
#pragma unroll
        for (int q = 0; q < RAX; ++q) g.load(j + 4 * q, x[q], y[q]);
        dft<RAX>(x);
        dft<RAX>(y);
        wave_sync();
#pragma unroll
        for (int q = 0; q < RAX; ++q) g.store(j + 4 * q, x[q], y[q]);
    }
    wave_sync();
    float2 x[NBX][4], y[NBX][4];
#pragma unroll
    for (int k = 0; k < NBX; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) g.load(4 * (j + 4 * k) + q, x[k][q], y[k][q]);
    wave_sync();
#pragma unroll
    for (int k = 0; k < NBX; ++k) {
        dft4_tw(x[k], tw[k]);
        dft4_tw(y[k], tw[k]);
#pragma unroll
        for (int q = 0; q < 4; ++q) g.store(j + 4 * k + RAX * q, x[k][q], y[k][q]);
    }
}

// y-pass of the wave's columns and the products of all three classes; the
// column is left zeroed.  Sum slot (oy, k, q) holds frequency j + S k + RA q of
// class oy.
template <int M>
__device__ __forceinline__ void rows_y(float4 *col, int j, const typename RowsCfg<M>::Tw *tw,
                                       float (&av)[3][RowsCfg<M>::NB * RowsCfg<M>::S][4]) {
    using C = RowsCfg<M>;
    constexpr int RA = C::RA, S = C::S, NB = C::NB, QV = C::QV, ROW = C::ROW;
    Grid<2> g;
    g.g = col;
    float2 vx[QV], vy[QV];
#pragma unroll
    for (int q = 0; q < QV; ++q) g.load(C::row(j, q) * ROW, vx[q], vy[q]);
    wave_sync();
#pragma unroll
    for (int q = RA; q < QV; ++q) g.zero(C::row(j, q) * ROW);
    // first-step outputs p at rows j + S p, read back as blocks j + S k
    auto exchange = [&](float2 *x, float2 *y) {
        wave_sync();
#pragma unroll
        for (int p = 0; p < RA; ++p) g.store((j + S * p) * ROW, x[p], y[p]);
        wave_sync();
#pragma unroll
        for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int q = 0; q < S; ++q) g.load(((j + S * k) * S + q) * ROW, x[k * S + q], y[k * S + q]);
    };
    auto second = [&](float2 *x, float2 *y, int oy) {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const typename C::Tw w = tw[oy * RA + j + S * k];
            dft_tw(x + k * S, w);
            dft_tw(y + k * S, w);
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const float2 ex = x[k * S + q], ey = y[k * S + q];
                float *a = av[oy][k * S + q];
                a[0] = fmaf(ex.x, ex.x, fmaf(ex.y, ex.y, a[0]));
                a[1] = fmaf(ey.x, ey.x, fmaf(ey.y, ey.y, a[1]));
                a[2] = fmaf(ex.x, ey.x, fmaf(ex.y, ey.y, a[2]));
                a[3] = fmaf(ex.y, ey.x, fmaf(-ex.x, ey.y, a[3]));
            }
        }
    };
    // each exchange's LDS latency is covered by another class's arithmetic
    float2 ax[RA], ay[RA], bx[RA], by[RA];
    rows_first<0>(vx, ax);
    rows_first<0>(vy, ay);
    exchange(ax, ay);
    rows_first<1>(vx, bx);
    rows_first<1>(vy, by);
    exchange(bx, by);
    second(ax, ay, 0);
    rows_first<2>(vx, ax);
    rows_first<2>(vy, ay);
    exchange(ax, ay);
    second(bx, by, 1);
    wave_sync();
#pragma unroll
    for (int p = 0; p < RA; ++p) g.zero((j + S * p) * ROW);
    second(ax, ay, 2);
}

template <int M, int AR, bool FR>
__global__ __launch_bounds__((RowsCfg<M>::T))
__attribute__((amdgpu_waves_per_eu(M == 16 ? 3 : 2))) void k_fused_rows(
    const FusedItem *__restrict__ items, const uint4 *__restrict__ entries,
    const uint8_t *__restrict__ volt, int64_t volt_t_stride, int A, int n_time,
    float *__restrict__ acc, int32_t *__restrict__ autos, int frame_len,
    float *__restrict__ frames, int64_t fstride, int vb, int n_items, int tps,
    float *__restrict__ part, int64_t part_stride) {
    using C = RowsCfg<M>;
    constexpr int T = C::T, W = T / 64, NP = C::NB * C::S, N = C::N;
    extern __shared__ float4 smem[];
    float4 *stage = smem + C::H * C::ROW;
    typename C::Tw *twy = reinterpret_cast<typename C::Tw *>(stage + A);

    const int slice = blockIdx.x / n_items;
    const FusedItem &it = items[blockIdx.x % n_items];
    if (it.c < 0) return;
    // sample numbers that may pass n_time (up to 2^31 - 1 in frame mode) are unsigned
    const int t0 = slice * tps, t1 = (int)min((uint32_t)n_time, (uint32_t)t0 + (uint32_t)tps);
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    Grid<2> grid;
    grid.g = smem;
    for (int i = tid; i < C::H * C::ROW; i += T) grid.zero(i);
    if (tid < 3 * C::RA) {
        const int n = 3 * (tid % C::RA) + tid / C::RA;      // 3 p + oy
        if constexpr (M == 32) twy[tid] = kRoots.r96[n];
        if constexpr (M == 16) twy[tid] = kRoots.r48[n];
    }
    Tw4 twx[C::RAX / 4];
#pragma unroll
    for (int k = 0; k < C::RAX / 4; ++k) twx[k] = LineTw<M>::at((lane >> 4) + 4 * k);

    float av[3][NP][4];
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int k = 0; k < NP; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) av[o][k][q] = 0.f;

    const uint8_t *vbase = volt + (int64_t)it.c * 2 * A * vb;
    const uint4 *ent = entries + it.entry_off + tid;
    const int n_iter = it.wave_iter[w];
    // self terms here only with one element a thread (registers)
    const bool own_autos = AR == 1 && autos != nullptr && it.ox == 0;
    int sa[4] = {0, 0, 0, 0};
    uint32_t rx[AR], ry[AR];             // the next sample's voltages of elements tid + k T
    auto fetch = [&](uint32_t t) {
        const uint8_t *vt = vbase + (int64_t)t * volt_t_stride;
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A && t < (uint32_t)t1) {
                rx[k] = volt_raw(vt, a, vb);
                ry[k] = volt_raw(vt, A + a, vb);
            }
        }
    };
    auto put = [&](uint32_t t) {              // stage sample t, add its self terms
        if (t >= (uint32_t)t1) return;
#pragma unroll
        for (int k = 0; k < AR; ++k) {
            const int a = tid + k * T;
            if (a < A) {
                const int2 vx = volt_dec(rx[k], vb), vy = volt_dec(ry[k], vb);
                const int xr = vx.x, xi = vx.y, yr = vy.x, yi = vy.y;
                stage[a] = make_float4((float)xr, (float)xi, (float)yr, (float)yi);
                if (own_autos) {
                    sa[0] += xr * xr + xi * xi;
                    sa[1] += yr * yr + yi * yi;
                    sa[2] += xr * yr + xi * yi;
                    sa[3] += xi * yr - xr * yi;
                }
            }
        }
        const uint8_t *vt = vbase + (int64_t)t * volt_t_stride;
        for (int a = tid + AR * T; a < A; a += T) {
            const int2 vx = volt_at(vt, a, vb), vy = volt_at(vt, A + a, vb);
            stage[a] = make_float4((float)vx.x, (float)vx.y, (float)vy.x, (float)vy.y);
        }
    };
#pragma unroll
    for (int k = 0; k < AR; ++k) rx[k] = ry[k] = 0u;
    fetch((uint32_t)t0);
    put((uint32_t)t0);
    fetch((uint32_t)t0 + 1u);

    const int col = w * C::CW + lane % C::CW, jy = lane / C::CW;
    for (int t = t0; t < t1; ++t) {
        uint4 e[RG];
        rows_load<T>(e, ent, 0, n_iter);
        __syncthreads();                 // staged voltages, zeroed grid
        rows_gather<T>(smem, ent, n_iter, stage, e);
        __syncthreads();
        put((uint32_t)t + 1u);
        fetch((uint32_t)t + 2u);
        for (int g = (w + (int)blockIdx.x) % W; g < (C::H + 15) / 16; g += W)
            rows_x<M>(smem, 16 * g + (lane & 15), lane >> 4, twx);
        __syncthreads();
        rows_y<M>(smem + col, jy, twy, av);
        if (FR && (t + 1) % frame_len == 0) {
            float *fr = frames + (int64_t)(t / frame_len) * fstride + it.img_off;
#pragma unroll
            for (int o = 0; o < 3; ++o)
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const int ky = 3 * (jy + C::S * (k / C::S) + C::RA * (k % C::S)) + o;
                    float *dst = fr + (int64_t)ky * N + 3 * col + it.ox;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        dst[q * (int64_t)N * N] = av[o][k][q];
                        av[o][k][q] = 0.f;
                    }
                }
        }
    }

    if (!FR) {
        float *base = part ? part + slice * part_stride + it.part_off : acc + it.img_off;
#pragma unroll
        for (int o = 0; o < 3; ++o)
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int ky = 3 * (jy + C::S * (k / C::S) + C::RA * (k % C::S)) + o;
                float *dst = base + (int64_t)ky * N + 3 * col + it.ox;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (part)
                        dst[q * (int64_t)N * N] = av[o][k][q];
                    else
                        dst[q * (int64_t)N * N] += av[o][k][q];
                }
            }
    }
    if (own_autos && tid < A) {
        int32_t *d = autos + ((int64_t)it.c * A + tid) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) atomicAdd(d + q, sa[q]);
    }
}

// Sums += self products of the samples packed in words x and y (VB = 1: up to four
// samples of one byte, high nibble real; VB = 2: up to two of a real and an
// imaginary byte; zero: no sample): |x|^2, |y|^2, Re and Im of x y* by integer
// dot products.  Im = sum xi yr - sum xr yi is twice the first less both.
template <int P, int VB>
__device__ __forceinline__ void auto_dots(int (&sum)[P == 2 ? 4 : 1], uint32_t x, uint32_t y) {
    auto dot = [](uint32_t a, uint32_t b, int c) {
        if constexpr (VB == 1) return __builtin_amdgcn_sdot8((int)a, (int)b, c, false);
        else return __builtin_amdgcn_sdot4((int)a, (int)b, c, false);
    };
    sum[0] = dot(x, x, sum[0]);
    if constexpr (P == 2) {
        constexpr uint32_t LO = VB == 1 ? 0x0f0f0f0fu : 0x00ff00ffu;
        constexpr int H = 4 * VB;
        const uint32_t swapped = (y >> H & LO) | (y << H & ~LO);
        const uint32_t imag = x & (VB == 1 ? LO : ~LO);
        sum[1] = dot(y, y, sum[1]);
        sum[2] = dot(x, y, sum[2]);
        sum[3] += 2 * dot(imag, swapped, 0) - dot(x, swapped, 0);
    }
}

// Four words of four bytes transposed: byte i of word k to byte k of word i.
__device__ __forceinline__ void bytes4x4(uint32_t (&o)[4], uint32_t a, uint32_t b, uint32_t c,
                                         uint32_t d) {
    const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u);
    const uint32_t ab2 = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u);
    const uint32_t cd2 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(cd2, ab2, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(cd2, ab2, 0x07060302u);
}

// Per-element self-term sums S_a^{pq} = sum_t E_a^p conj(E_a^q), exact in
// int32 (|E|^2 <= 128 per sample).  Grid: (256 elements, channels, time chunks);
// a workgroup is blockDim.y groups of 256 / E lanes, E elements a lane, that take
// turns of eight samples, eight samples' loads in flight; VB bytes per voltage
// sample.  The groups' sums meet in LDS, so that a call of one time chunk adds
// them by plain loads and stores.  E = 4 (elements of one byte, whole aligned
// words) reads a word a lane and turns four samples' words into four elements'.
// 4096 elements x 2 feeds x 64 channels x 256 samples: 62 us with byte loads,
// products by multiplies and atomics, 36 us now (134 MB).
template <int P, int VB, int E>
__global__ __launch_bounds__(1024) void k_autos(const uint8_t *__restrict__ volt,
                                                int64_t volt_t_stride, int A, int n_time,
                                                int t_chunk, int32_t *__restrict__ autos) {
    static_assert(E == 1 || VB == 1, "words of four one-byte samples");
    constexpr int U = 8, NPROD = P == 2 ? 4 : 1;
    // sum k of lane l at PITCH k + l: both ways without bank conflicts
    constexpr int PITCH = 256 / E + 1, NK = E * NPROD;
    __shared__ int32_t s[PITCH * NK];
    const int tid = threadIdx.y * blockDim.x + threadIdx.x, T = blockDim.x * blockDim.y;
    for (int i = tid; i < PITCH * NK; i += T) s[i] = 0;
    const int a = blockIdx.x * 256 + E * threadIdx.x;
    const int c = blockIdx.y;
    const int t0 = blockIdx.z * t_chunk;
    const int t1 = min(n_time, t0 + t_chunk);
    int sum[E][NPROD] = {};
    const uint8_t *v = volt + (int64_t)c * P * A * VB;
    for (int tb = t0 + U * threadIdx.y; tb < t1 && a < A; tb += U * blockDim.y) {
        uint32_t rx[U], ry[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint8_t *vt = v + (int64_t)min(tb + k, t1 - 1) * volt_t_stride;
            if constexpr (E == 4) {
                rx[k] = *reinterpret_cast<const uint32_t *>(vt + a);
                ry[k] = P == 2 ? *reinterpret_cast<const uint32_t *>(vt + A + a) : 0u;
            } else {
                rx[k] = volt_raw(vt, a, VB);
                ry[k] = P == 2 ? volt_raw(vt, (int64_t)A + a, VB) : 0u;
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            // samples past the chunk (clamped loads) count as zero
            if (tb + k >= t1) rx[k] = ry[k] = 0u;
        if constexpr (E == 4) {
#pragma unroll
            for (int k = 0; k < U; k += 4) {
                uint32_t x[4], y[4] = {0u, 0u, 0u, 0u};
                bytes4x4(x, rx[k], rx[k + 1], rx[k + 2], rx[k + 3]);
                if (P == 2) bytes4x4(y, ry[k], ry[k + 1], ry[k + 2], ry[k + 3]);
#pragma unroll
                for (int i = 0; i < 4; ++i) auto_dots<P, VB>(sum[i], x[i], y[i]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < U; ++k) auto_dots<P, VB>(sum[0], rx[k], ry[k]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i)
#pragma unroll
        for (int q = 0; q < NPROD; ++q)
            atomicAdd(&s[PITCH * (i * NPROD + q) + threadIdx.x], sum[i][q]);
    __syncthreads();
    int32_t *dst = autos + ((int64_t)c * A + blockIdx.x * 256) * NPROD;
    const int n = min(256, A - (int)blockIdx.x * 256) * NPROD;
    for (int i = tid; i < n; i += T) {
        const int v = s[PITCH * (i % NK) + i / NK];
        if (gridDim.z == 1) dst[i] += v;
        else atomicAdd(dst + i, v);
    }
}

// acc[img_off + i] += sum over slices s = 0 .. S-1 of part[s part_stride +
// part_off + i], in a fixed order, for every channel of one fused group.  The
// slices are summed in FP64 and rounded once: with as many slices as samples a
// running FP32 sum would round at every one of them (16 elements, one 32^2 channel,
// 64 samples: error against 64 bits 1.6e-7 so, 7e-8 now, at no change in time).
// Grid: (float blocks, channels of the group).
__global__ __launch_bounds__(256) void k_fused_reduce(const GroupChan *__restrict__ chans, int S,
                                                      const float *__restrict__ part,
                                                      int64_t part_stride,
                                                      float *__restrict__ acc) {
    const GroupChan g = chans[blockIdx.y];
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < g.n_floats;
         i += (int64_t)gridDim.x * 256) {
        double s = 0.0;
        const float *q = part + g.part_off + i;
        int k = 0;
        for (; k + 8 <= S; k += 8) {           // eight loads in flight
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = (double)q[(k + u) * part_stride];
            s += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
        for (; k < S; ++k) s += (double)q[k * part_stride];
        acc[g.img_off + i] += (float)s;
    }
}

// ------------------------------------------------------------ host build
static int threads_of(int M) {
    return M == 64 ? FCfg<64>::T : M == 32 ? FCfg<32>::T : FCfg<16>::T;
}
static int threads_of(const FusedGroup *g) {
    if (g->kind == 2) return g->M == 32 ? RowsCfg<32>::T : RowsCfg<16>::T;
    return threads_of(g->M);
}
static int row_of(int M) {
    return M == 64 ? FCfg<64>::ROW : M == 32 ? FCfg<32>::ROW : FCfg<16>::ROW;
}

// Cells are dealt longest-first to the least-loaded of T lanes, so each cell
// is summed by one lane in a fixed order and written once.  Appends
// n_iter * T entries [iter][lane] (jones: n_iter * 3 * T, [iter][row][lane])
// to all (padding entries are zero) and returns n_iter.  wave_iter: the lanes
// are then sorted by the length of their lists, so that a few crowded cells
// lengthen one wave's gather and not all of them (an LWA channel at 40 MHz has
// cells of ten taps, but 4.5 taps a lane), and wave_iter[w] is the longest list
// of wave w.  Eight waves run in pairs (w, w + 4) on the four SIMDs: the longest
// and the shortest lists share one.
int lpt_pack(const std::vector<GatherTap> &taps, int T, std::vector<uint4> &all, bool jones,
             int32_t *wave_iter, bool banks) {
    const size_t n = taps.size();
    // taps by cell, cells by descending tap count: counting sorts, stable (a
    // band of hundreds of channels sorts millions of taps at plan time)
    int n_cells = 0;
    for (const GatherTap &t : taps) n_cells = std::max(n_cells, t.cell + 1);
    std::vector<int> at(n_cells + 1, 0), sorted_tap(n);
    for (const GatherTap &t : taps) ++at[t.cell + 1];
    for (int c = 0; c < n_cells; ++c) at[c + 1] += at[c];
    std::vector<std::pair<int, int>> runs;  // (start, count) per cell, into sorted_tap
    int longest = 0;
    for (int c = 0; c < n_cells; ++c)
        if (at[c + 1] > at[c]) {
            runs.push_back({at[c], at[c + 1] - at[c]});
            longest = std::max(longest, at[c + 1] - at[c]);
        }
    for (size_t i = 0; i < n; ++i) sorted_tap[at[taps[i].cell]++] = (int)i;
    std::vector<int> order(runs.size()), first(longest + 2, 0);
    for (const auto &r : runs) ++first[longest - r.second + 1];
    for (int k = 0; k <= longest; ++k) first[k + 1] += first[k];
    for (size_t i = 0; i < runs.size(); ++i) order[first[longest - runs[i].second]++] = (int)i;
    std::vector<std::vector<int>> lane_runs(T);
    std::vector<int> load(T, 0);
    using LP = std::pair<int, int>;
    // one heap, or (banks) one per cell index mod 8: lane l then owns cells = l mod
    // 8, so that eight neighbouring lanes' 16-byte stores meet distinct banks,
    // unless another lane's list is shorter by more than a tap
    const int nh = banks ? 8 : 1;
    std::vector<std::priority_queue<LP, std::vector<LP>, std::greater<LP>>> heap(nh);
    for (int l = 0; l < T; ++l) heap[l % nh].push({0, l});
    for (int r : order) {
        int own = taps[sorted_tap[runs[r].first]].cell % nh;
        for (int k = 0; k < nh; ++k)
            if (heap[k].top().first + 1 < heap[own].top().first) own = k;
        auto &h = heap[own];
        LP top = h.top();
        h.pop();
        lane_runs[top.second].push_back(r);
        load[top.second] += runs[r].second;
        h.push({load[top.second], top.second});
    }
    const int n_iter = *std::max_element(load.begin(), load.end());
    if (wave_iter) {
        const int W = T / 64;
        std::vector<std::vector<int>> sorted(T);
        for (int k = 0; k < W; ++k) wave_iter[k] = 0;
        for (int r = 0; r < nh; ++r) {           // within each residue, T / nh lanes
            std::vector<int> lanes;
            for (int l = r; l < T; l += nh) lanes.push_back(l);
            std::stable_sort(lanes.begin(), lanes.end(),
                             [&](int x, int y) { return load[x] > load[y]; });
            for (size_t i = 0; i < lanes.size(); ++i) {
                const int k = (int)i * nh / 64, w = W == 8 && k >= 4 ? 11 - k : k;
                wave_iter[w] = std::max(wave_iter[w], load[lanes[i]]);
                sorted[w * 64 + (int)i * nh % 64 + r].swap(lane_runs[lanes[i]]);
            }
        }
        lane_runs.swap(sorted);
    }
    const size_t off = all.size();
    const int rows = jones ? 3 : 1;
    all.resize(off + (size_t)n_iter * rows * T, make_uint4(0u, 0u, 0u, 0u));
    auto bits = [](float f) { return __builtin_bit_cast(uint32_t, f); };
    for (int l = 0; l < T; ++l) {
        int k = 0;
        for (int r : lane_runs[l])
            for (int i = 0; i < runs[r].second; ++i, ++k) {
                const GatherTap &tp = taps[sorted_tap[runs[r].first + i]];
                const bool last = (i == runs[r].second - 1);
                uint4 e;
                e.x = (uint32_t)tp.ant | (last ? 0x80000000u : 0u);
                e.y = (uint32_t)tp.cell;
                e.z = bits(tp.wr);
                e.w = bits(tp.wi);
                all[off + (size_t)k * rows * T + l] = e;
                if (jones) {
                    all[off + ((size_t)k * 3 + 1) * T + l] =
                        make_uint4(bits(tp.m[0]), bits(tp.m[1]), bits(tp.m[2]), bits(tp.m[3]));
                    all[off + ((size_t)k * 3 + 2) * T + l] =
                        make_uint4(bits(tp.m[4]), bits(tp.m[5]), 0u, 0u);
                }
            }
    }
    return n_iter;
}

// Gather entries of one item: the taps of class (ox, oy) folded modulo M
// (with Jones kernels all four weights of a tap carry the same fold factor).
static FusedItem build_item(epic_plan p, const std::vector<int> &j0, const std::vector<double> &w,
                            int c, int ox, int oy, int M, int T, std::vector<uint4> &all,
                            int ylo = 0, bool unfold = false, bool pair = false) {
    const int A = p->A, K = p->K, J = p->J;
    const int N = p->ch[c].N, R = p->ch[c].R, ROW = row_of(M);
    std::vector<GatherTap> taps;
    taps.reserve((size_t)A * K * K);
    // LDS cell of row y (from ylo) and folded column x
    auto place = [&](int y, int x) {
        if (pair) return pair_pos(y) * ROW + pair_pos(x);
        if (!unfold) return (y % M) * ROW + x;
        const int r = M == 32 ? RowsCfg<32>::row(y % 4, y / 4) : RowsCfg<16>::row(y % 4, y / 4);
        return r * ROW + x;
    };
    for (int a = 0; a < A; ++a) {
        const int jx0 = j0[((size_t)c * A + a) * 2];
        const int jy0 = j0[((size_t)c * A + a) * 2 + 1];
        for (int dy = 0; dy < K; ++dy)
            for (int dx = 0; dx < K; ++dx) {
                const int jx = jx0 + dx, jy = jy0 + dy;
                // conj(W) * (-1)^(jx+jy) * exp(+2 pi i (ox jx + oy jy) / N)
                const long ph = ((long)ox * jx + (long)oy * jy) % N;
                const double ang = 2.0 * M_PI * (double)ph / (double)N;
                const double sg = ((jx + jy) & 1) ? -1.0 : 1.0;
                const double cr = std::cos(ang) * sg, ci = std::sin(ang) * sg;
                float fw[8] = {};
                for (int m = 0; m < J; ++m) {
                    const size_t wi = ((((size_t)c * A + a) * J + m) * K * K + dy * K + dx) * 2;
                    const double wr0 = w[wi], wi0 = -w[wi + 1];
                    fw[2 * m] = (float)(wr0 * cr - wi0 * ci);
                    fw[2 * m + 1] = (float)(wr0 * ci + wi0 * cr);
                }
                GatherTap tp;
                tp.cell = place((jy - ylo), jx % M);
                tp.ant = a;
                tp.wr = fw[0];
                tp.wi = fw[1];
                for (int m = 0; m < 6; ++m) tp.m[m] = fw[2 + m];
                taps.push_back(tp);
            }
    }
    const size_t off = all.size();
    FusedItem fi{};
    int n_iter = lpt_pack(taps, T, all, J == 4, fi.wave_iter, (M == 64 || unfold) && p->P == 2);
    const int rows = J == 4 ? 3 : 1;
    // the kernels load the first entries of every list unconditionally: an
    // item always has at least one (padding) row
    if (n_iter == 0) {
        all.resize(off + (size_t)rows * T, make_uint4(0u, 0u, 0u, 0u));
        n_iter = 1;
    }
    for (int32_t &k : fi.wave_iter) k = std::max(k, 1);
    // The kernels store the running sum at every entry, so padding (all-zero)
    // entries point at a slot no pass reads: column M of row (lane mod M).
    for (int k = 0; k < n_iter; ++k)
        for (int l = 0; l < T; ++l) {
            uint4 &e = all[off + (size_t)k * rows * T + l];
            if (e.x == 0u && e.y == 0u && e.z == 0u && e.w == 0u)
                e.y = (uint32_t)((l % M) * ROW + M);
        }
    fi.c = c;
    fi.N = N;
    fi.R = R;
    fi.ox = ox;
    fi.oy = oy;
    fi.n_iter = n_iter;
    fi.entry_off = (int64_t)off;
    fi.img_off = p->ch[c].img_off;
    return fi;
}

// XCD-aware order.  Workgroups are dealt to the 8 XCDs round-robin by id, so
// items placed at ids x, x+8, x+16, ... share one XCD and its L2.  Channels go
// to XCD bins longest-first (a channel's items all read the same voltages);
// each bin lists its items channel by channel; the bins are then interleaved,
// padded with empty items (c = -1).
static void xcd_layout(std::vector<FusedItem> &items, int C) {
    constexpr int NX = 8;
    std::vector<int64_t> chan_cost(C, 0);
    std::vector<int> chans;
    for (const FusedItem &fi : items) {
        if (chan_cost[fi.c] == 0) chans.push_back(fi.c);
        chan_cost[fi.c] += 64 + fi.n_iter;
    }
    std::stable_sort(chans.begin(), chans.end(),
                     [&](int x, int y) { return chan_cost[x] > chan_cost[y]; });
    std::vector<int64_t> bin_cost(NX, 0);
    std::vector<std::vector<FusedItem>> bins(NX);
    for (int c : chans) {
        const int b = (int)(std::min_element(bin_cost.begin(), bin_cost.end()) - bin_cost.begin());
        bin_cost[b] += chan_cost[c];
        for (const FusedItem &fi : items)
            if (fi.c == c) bins[b].push_back(fi);
    }
    size_t depth = 0;
    for (auto &b : bins) depth = std::max(depth, b.size());
    FusedItem empty{};
    empty.c = -1;
    std::vector<FusedItem> laid(depth * NX, empty);
    for (int x = 0; x < NX; ++x)
        for (size_t i = 0; i < bins[x].size(); ++i) laid[i * NX + x] = bins[x][i];
    items.swap(laid);
}

// Workgroups of a kernel that the device runs at once (occupancy API over all
// CUs), or 0 if unknown.
static int64_t resident_slots(const void *k, int threads, size_t lds) {
    if (lds_ready(k, lds)) return 0;
    int dev = 0, n_cu = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, threads, lds) != hipSuccess)
        return 0;
    return (int64_t)n_cu * per_cu;
}

// The same for a one-class-per-item group.
template <int M, int P, bool JN>
static int64_t fused_slots_t(int A) {
    constexpr int T = FCfg<M>::T, GSZ = M * FCfg<M>::ROW;
    const size_t lds = sizeof(float2) * P * GSZ + sizeof(float4) * (size_t)A;
    const void *k = A <= T       ? reinterpret_cast<const void *>(k_fused<M, P, 1, false, JN>)
                    : A <= 2 * T ? reinterpret_cast<const void *>(k_fused<M, P, 2, false, JN>)
                                 : reinterpret_cast<const void *>(k_fused<M, P, 4, false, JN>);
    return resident_slots(k, T, lds);
}

static int64_t fused_slots(epic_plan p, int M) {
    const bool jn = p->J == 4;
    if (p->P == 1) {
        return M == 64 ? fused_slots_t<64, 1, false>(p->A)
               : M == 32 ? fused_slots_t<32, 1, false>(p->A) : fused_slots_t<16, 1, false>(p->A);
    }
    if (jn)
        return M == 64 ? fused_slots_t<64, 2, true>(p->A)
               : M == 32 ? fused_slots_t<32, 2, true>(p->A) : fused_slots_t<16, 2, true>(p->A);
    return M == 64 ? fused_slots_t<64, 2, false>(p->A)
           : M == 32 ? fused_slots_t<32, 2, false>(p->A) : fused_slots_t<16, 2, false>(p->A);
}

// The same for a row-unfolded group, by the element rounds that its launch takes.
template <int M>
static int64_t rows_slots(int A) {
    using C = RowsCfg<M>;
    const void *k = A <= C::T       ? reinterpret_cast<const void *>(k_fused_rows<M, 1, false>)
                    : A <= 2 * C::T ? reinterpret_cast<const void *>(k_fused_rows<M, 2, false>)
                                    : reinterpret_cast<const void *>(k_fused_rows<M, 4, false>);
    return resident_slots(k, C::T, C::lds(A));
}

static int cu_count() {
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 256;
    return n_cu;
}

// Time slices of a one-class-per-item group: at least enough workgroups for
// about four waves per SIMD (1024 SIMDs), then the fewest slices (at most 16)
// whose last round of resident workgroups is at least 90 % full; where one or a
// few small grids leave the chip idle, up to 64 slices (one 32 x 32 channel of 1000
// samples: 144 us with 16, 51 us with 64; not for 64 x 64 items, whose slices cost
// more than they save: two 128 x 128 channels of 250 samples 110 and 140 us); each
// channel's images get a place in the group's partial image set.
static epic_status slice_group(epic_plan p, FusedGroup *g, std::vector<FusedItem> &items,
                               hipStream_t s) {
    const int waves_per_wg = threads_of(g) / 64;
    int64_t real = 0;
    for (const FusedItem &fi : items) real += fi.c >= 0;
    const int64_t waves = real * waves_per_wg;
    const int cap = g->M == 64 ? 16 : 64;
    int S = (int)std::max<int64_t>(1, std::min<int64_t>(cap, (4096 + waves - 1) / std::max<int64_t>(1, waves)));
    const int64_t slots = g->kind == 0 ? fused_slots(p, g->M) : 0;
    if (slots > 0) {
        // workgroups launched = padded items x slices
        const int64_t wgs = (int64_t)items.size();
        // beyond 16 slices no more than one round of them (256 elements, 64 channels of
        // 32^2, 512 samples: 218 us with 32 slices, 184 with the 28 that fit).  Where many
        // elements leave room for fewer than 16, 16 x 16 items still gain by shorter turns
        // (2500 elements, 8 channels of 48^2, 50 samples: 666 us with 16, 509 with 57),
        // 32 x 32 ones, whose start costs more, do not (3000 elements, 8 channels of 96^2:
        // 508 with 16, 534 with 28).
        if (S > 16 && (slots >= 16 * wgs || g->M == 32))
            S = (int)std::max<int64_t>(16, std::min<int64_t>(S, slots / wgs));
        for (int s2 = S; s2 <= 16; ++s2) {
            const double rounds = (double)(wgs * s2) / (double)slots;
            if (rounds / std::ceil(rounds) >= 0.9 || s2 == 16) {
                S = s2;
                break;
            }
        }
    }
    if (p->time_slices > 0) S = p->time_slices;   // the caller's (autotuned) choice
    g->slices = g->kind == 0 || (g->kind == 2 && p->time_slices > 0) ? S : 1;
    // a paired workgroup fills a CU; of row-unfolded ones as many as registers and the
    // staged elements leave (M = 32: four a CU to about 950 elements, two with 2048)
    g->slots = cu_count();
    if (g->kind == 2)
        if (const int64_t n = g->M == 32 ? rows_slots<32>(p->A) : rows_slots<16>(p->A)) g->slots = n;
    std::vector<int64_t> off(p->C, -1);
    std::vector<GroupChan> chans;
    int64_t n = 0;
    for (FusedItem &fi : items) {
        if (fi.c < 0) continue;
        if (off[fi.c] < 0) {
            off[fi.c] = n;
            const int64_t nf = (int64_t)p->n_prod * fi.N * fi.N;
            chans.push_back(GroupChan{fi.img_off, n, nf});
            n += nf;
        }
        fi.part_off = off[fi.c];
    }
    g->part_floats = n;
    g->n_chans = (int)chans.size();
    if (g->kind != 0 && p->time_slices == 0)
        g->slices = reserved_slices((int64_t)items.size(), g->slots, n);
    epic_status st;
    if ((st = g->chans.alloc(sizeof(GroupChan) * std::max<size_t>(1, chans.size())))) return st;
    if (!chans.empty())
        EPIC_HIP(hipMemcpyAsync(g->chans.p, chans.data(), sizeof(GroupChan) * chans.size(),
                                hipMemcpyHostToDevice, s));
    return EPIC_OK;
}

// Place the sliced groups' partial image sets in the accumulator's working
// memory after what the plan already needs there.
void fused_assign_work(epic_plan p) {
    for (FusedGroup *g : p->groups) {
        if (g->slices <= 1) continue;
        g->work_off = (p->work_bytes + 255) / 256 * 256;
        p->work_bytes = g->work_off + (int64_t)sizeof(float) * g->slices * g->part_floats;
    }
    if (p->flags & EPIC_BATCH_QUEUE) {
        // the queue counter, one per accumulator (launches on different
        // accumulators may run at once)
        p->queue_off = (p->work_bytes + 255) / 256 * 256;
        p->work_bytes = p->queue_off + 256;
    }
}

static epic_status upload_group(epic_plan p, FusedGroup *g, std::vector<FusedItem> &items,
                                std::vector<uint4> &all, int C, hipStream_t s) {
    xcd_layout(items, C);
    epic_status st;
    if ((st = slice_group(p, g, items, s))) return st;
    g->n_items = (int)items.size();
    g->host_items = items;
    if ((st = g->items.alloc(sizeof(FusedItem) * items.size()))) return st;
    if ((st = g->entries.alloc(sizeof(uint4) * all.size()))) return st;
    EPIC_HIP(hipMemcpyAsync(g->items.p, items.data(), sizeof(FusedItem) * items.size(),
                            hipMemcpyHostToDevice, s));
    EPIC_HIP(hipMemcpyAsync(g->entries.p, all.data(), sizeof(uint4) * all.size(),
                            hipMemcpyHostToDevice, s));
    EPIC_HIP(hipStreamSynchronize(s));
    return EPIC_OK;
}

// The work queue of an EPIC_BATCH_QUEUE plan: every real item of the size
// groups, 64 x 64 items first, then same-channel bundles of 32 x 32 and
// 16 x 16 items, a unit per time slice of its size's group (longest processing
// time first).
static epic_status queue_build(epic_plan p, hipStream_t s) {
    // per size: units of one slice; a unit's cost ~ its transform's work x
    // the samples of a slice, so sort by M^2 log M / slices, largest first
    struct Keyed {
        double cost;
        QueueUnit u;
    };
    std::vector<Keyed> keyed;
    for (int M : {64, 32, 16}) {
        const int B = M == 64 ? 1 : M == 32 ? 4 : 8;
        for (FusedGroup *g : p->groups) {
            if (g->M != M || g->kind != 0) continue;
            std::vector<std::vector<int>> per(p->C);
            for (int i = 0; i < g->n_items; ++i)
                if (g->host_items[i].c >= 0) per[g->host_items[i].c].push_back(i);
            const double cost = (double)M * M * std::log2((double)M) / g->slices;
            // 16 x 16 bundles of any channels when eight stagings fit beside
            // the eight grids in the grid area: 8 A float4 <= P (kQueueGrid -
            // 8 x 16 x 17) float2
            const bool cross =
                M == 16 && (int64_t)8 * p->A * 16 <= (int64_t)p->P * (kQueueGrid - 8 * 16 * 17) * 8;
            std::vector<std::vector<int>> lists;
            if (cross) {
                lists.emplace_back();
                for (int c = 0; c < p->C; ++c)
                    lists.back().insert(lists.back().end(), per[c].begin(), per[c].end());
            } else {
                lists = per;
            }
            for (int sl = 0; sl < g->slices; ++sl)
                for (const std::vector<int> &li : lists)
                    for (size_t k = 0; k < li.size(); k += B) {
                        QueueUnit u{};
                        u.M = M;
                        u.n = (int)std::min<size_t>(B, li.size() - k);
                        u.slice = sl;
                        u.own_stage = cross ? 1 : 0;
                        for (int j = 0; j < 8; ++j) u.idx[j] = li[k + std::min(j, u.n - 1)];
                        keyed.push_back({cost, u});
                    }
        }
    }
    std::stable_sort(keyed.begin(), keyed.end(),
                     [](const Keyed &x, const Keyed &y) { return x.cost > y.cost; });
    std::vector<QueueUnit> units;
    for (const Keyed &k : keyed) units.push_back(k.u);
    p->n_units = (int)units.size();
    epic_status st = p->d_units.alloc(sizeof(QueueUnit) * std::max<size_t>(1, units.size()));
    if (st) return st;
    if (!units.empty())
        EPIC_HIP(hipMemcpyAsync(p->d_units.p, units.data(), sizeof(QueueUnit) * units.size(),
                                hipMemcpyHostToDevice, s));
    EPIC_HIP(hipStreamSynchronize(s));
    return EPIC_OK;
}

epic_status fused_build(epic_plan p, const std::vector<int> &j0, const std::vector<double> &w,
                        hipStream_t s) {
    const int A = p->A, K = p->K;
    // Paired items: two feeds, N = 2 * 64, every element row in a 64-row window, and
    // no more elements than the LDS beside two grids takes (one class per item, with
    // one grid, takes about 6000).
    std::vector<int> pair_ylo(p->C, -1);
    const bool queue = (p->flags & EPIC_BATCH_QUEUE) != 0;
    for (int c = 0; c < p->C; ++c) {
        // the queue takes single-class items only
        if (queue || A > kPairMaxAnt) break;
        if (p->banded[c] || p->P != 2 || p->ch[c].M != 64 || p->ch[c].R != 2) continue;
        int lo = 1 << 30, hi = -1;
        for (int a = 0; a < A; ++a) {
            const int jy = j0[((size_t)c * A + a) * 2 + 1];
            lo = std::min(lo, jy);
            hi = std::max(hi, jy + K - 1);
        }
        if (hi - lo < 64) pair_ylo[c] = lo;
    }
    {
        std::vector<FusedItem> items;
        std::vector<uint4> all;
        for (int c = 0; c < p->C; ++c) {
            if (pair_ylo[c] < 0) continue;
            for (int ox = 0; ox < 2; ++ox) {
                items.push_back(build_item(p, j0, w, c, ox, 0, 64, 512, all, pair_ylo[c], false, true));
            }
        }
        if (!items.empty()) {
            auto *g = new FusedGroup();
            g->M = 64;
            g->kind = 1;
            p->groups.push_back(g);
            epic_status st = upload_group(p, g, items, all, p->C, s);
            if (st) return st;
        }
    }
    // Row-unfolded items: sides 96 and 48 in sub-transforms of a third of the side
    // (the library's own choice), two feeds, one kernel per element, rows within
    // half the side, and elements that leave the LDS for it.
    std::vector<int> rows_ylo(p->C, -1);
    for (int c = 0; c < p->C; ++c) {
        const int N = p->ch[c].N;
        if (queue || p->banded[c] || p->P != 2 || p->J != 1 || A > 2048) continue;
        if ((N != 96 && N != 48) || p->ch[c].M != N / 3) continue;
        int lo = 1 << 30, hi = -1;
        for (int a = 0; a < A; ++a) {
            const int jy = j0[((size_t)c * A + a) * 2 + 1];
            lo = std::min(lo, jy);
            hi = std::max(hi, jy + K - 1);
        }
        if (hi - lo < N / 2) rows_ylo[c] = lo;
    }
    for (int M : {32, 16}) {
        std::vector<FusedItem> items;
        std::vector<uint4> all;
        auto *g = new FusedGroup();
        g->M = M;
        g->kind = 2;
        const int T = threads_of(g);
        for (int c = 0; c < p->C; ++c) {
            if (rows_ylo[c] < 0 || p->ch[c].N != 3 * M) continue;
            for (int ox = 0; ox < 3; ++ox)
                items.push_back(build_item(p, j0, w, c, ox, 0, M, T, all, rows_ylo[c], true));
        }
        if (items.empty()) {
            delete g;
            continue;
        }
        p->groups.push_back(g);
        epic_status st = upload_group(p, g, items, all, p->C, s);
        if (st) return st;
    }
    for (int M : {64, 32, 16}) {
        std::vector<FusedItem> items;
        std::vector<uint4> all;
        const int T = threads_of(M);
        for (int c = 0; c < p->C; ++c) {
            if (p->banded[c] || p->ch[c].M != M || pair_ylo[c] >= 0 || rows_ylo[c] >= 0) continue;
            const int R = p->ch[c].R;
            for (int oy = 0; oy < R; ++oy)
                for (int ox = 0; ox < R; ++ox) items.push_back(build_item(p, j0, w, c, ox, oy, M, T, all));
        }
        if (items.empty()) continue;
        auto *g = new FusedGroup();
        g->M = M;
        p->groups.push_back(g);
        epic_status st = upload_group(p, g, items, all, p->C, s);
        if (st) return st;
    }
    if (queue) return queue_build(p, s);
    return EPIC_OK;
}

epic_status lds_ready(const void *kern, size_t lds) {
    // first calls may come from several host threads at once
    static std::mutex mu;
    static int lds_max = -1;
    static std::vector<const void *> done;
    std::lock_guard<std::mutex> lock(mu);
    if (lds_max < 0) {
        int dev = 0, v = 0;
        EPIC_HIP(hipGetDevice(&dev));
        EPIC_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        lds_max = v;
    }
    if (std::find(done.begin(), done.end(), kern) == done.end()) {
        EPIC_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max));
        done.push_back(kern);
    }
    if ((int64_t)lds > lds_max)
        return fail(EPIC_ERR_UNSUPPORTED, "LDS need " + std::to_string(lds) +
                                              " B above the device limit");
    return EPIC_OK;
}

// `part`: the group's partial image sets (time slices), or nullptr.
template <int M, int P, int AR, bool FR, bool JN>
static epic_status launch_fused_fr(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                   int A, int vb, int n_time, float *acc, int32_t *autos,
                                   const FrameOut &fo, hipStream_t s, bool dry, float *part) {
    constexpr int T = FCfg<M>::T, GSZ = M * FCfg<M>::ROW;
    const size_t lds = sizeof(float2) * P * GSZ + sizeof(float4) * (size_t)A;
    auto kern = k_fused<M, P, AR, FR, JN>;
    epic_status st = lds_ready(reinterpret_cast<const void *>(kern), lds);
    if (st || dry) return st;
    // slices in use: at most one per sample
    const bool sliced = part && !FR && g->slices > 1 && acc;
    const int tps = sliced ? (n_time + g->slices - 1) / g->slices : n_time;
    const int used = sliced ? (n_time + tps - 1) / tps : 1;
    hipLaunchKernelGGL(kern, dim3(g->n_items * used), dim3(T), lds, s, g->items.as<FusedItem>(),
                       g->entries.as<uint4>(), d_volt, vstride, A, n_time, acc, autos, fo.len,
                       fo.out, fo.stride, vb, g->n_items, tps, sliced ? part : nullptr,
                       g->part_floats);
    EPIC_HIP(hipGetLastError());
    if (sliced) {
        hipLaunchKernelGGL(k_fused_reduce, dim3(64, g->n_chans), dim3(256), 0, s,
                           g->chans.as<GroupChan>(), used, part, g->part_floats, acc);
        EPIC_HIP(hipGetLastError());
    }
    return EPIC_OK;
}

template <int M, int P, int AR, bool JN>
static epic_status launch_fused_ar(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                   int A, int vb, int n_time, float *acc, int32_t *autos,
                                   const FrameOut &fo, hipStream_t s, bool dry, float *part) {
    return fo.len ? launch_fused_fr<M, P, AR, true, JN>(g, d_volt, vstride, A, vb, n_time, acc,
                                                        autos, fo, s, dry, nullptr)
                  : launch_fused_fr<M, P, AR, false, JN>(g, d_volt, vstride, A, vb, n_time, acc,
                                                         autos, fo, s, dry, part);
}

// Element rounds per thread: 1, 2 or 4; above 4 T the self terms come from a
// separate pass (autos == nullptr).
template <int M, int P, bool JN>
static epic_status launch_fused(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                int A, int vb, int n_time, float *acc, int32_t *autos,
                                const FrameOut &fo, hipStream_t s, bool dry, float *part) {
    constexpr int T = FCfg<M>::T;
    if (A <= T)
        return launch_fused_ar<M, P, 1, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s,
                                            dry, part);
    if (A <= 2 * T)
        return launch_fused_ar<M, P, 2, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s,
                                            dry, part);
    return launch_fused_ar<M, P, 4, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s, dry,
                                        part);
}

template <int AR, bool FR, bool JN>
static epic_status launch_pair_fr(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                  int A, int vb, int n_time, float *acc, int32_t *autos,
                                  const FrameOut &fo, hipStream_t s, bool dry, float *part) {
    const size_t lds = sizeof(float4) * (2 * (size_t)kPairGrid + (size_t)A);
    auto kern = k_fused_pair<AR, FR, JN>;
    epic_status st = lds_ready(reinterpret_cast<const void *>(kern), lds);
    if (st || dry) return st;
    const int unit = FR ? fo.len : 1;
    const int want = FR ? 64 : part && acc ? g->slices : 1;
    const SliceChoice sl = best_slices(g->n_items, g->slots, n_time, want, g->part_floats, unit, FR);
    const int S = sl.slices, tps = sl.len;
    float *sets = !FR && S > 1 ? part : nullptr;
    hipLaunchKernelGGL(kern, dim3(g->n_items * S), dim3(512), lds, s, g->items.as<FusedItem>(),
                       g->entries.as<uint4>(), d_volt, vstride, A, n_time, acc, autos, fo.len,
                       fo.out, fo.stride, vb, g->n_items, tps, sets, g->part_floats);
    EPIC_HIP(hipGetLastError());
    if (sets) {
        hipLaunchKernelGGL(k_fused_reduce, dim3(64, g->n_chans), dim3(256), 0, s,
                           g->chans.as<GroupChan>(), S, sets, g->part_floats, acc);
        EPIC_HIP(hipGetLastError());
    }
    return EPIC_OK;
}

template <int AR, bool JN>
static epic_status launch_pair_ar(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                  int A, int vb, int n_time, float *acc, int32_t *autos,
                                  const FrameOut &fo, hipStream_t s, bool dry, float *part) {
    return fo.len ? launch_pair_fr<AR, true, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos,
                                                 fo, s, dry, nullptr)
                  : launch_pair_fr<AR, false, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos,
                                                  fo, s, dry, part);
}

template <bool JN>
static epic_status launch_pair(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride, int A,
                               int vb, int n_time, float *acc, int32_t *autos, const FrameOut &fo,
                               hipStream_t s, bool dry, float *part) {
    static_assert(kPairMaxAnt <= 4 * 512, "four elements a thread cover every paired plan");
    if (A <= 512)
        return launch_pair_ar<1, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s, dry, part);
    if (A <= 1024)
        return launch_pair_ar<2, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s, dry, part);
    return launch_pair_ar<4, JN>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, s, dry, part);
}

template <int M, int AR, bool FR>
static epic_status launch_rows_fr(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride,
                                  int A, int vb, int n_time, float *acc, int32_t *autos,
                                  const FrameOut &fo, hipStream_t s, bool dry, float *part,
                                  bool fixed_slices) {
    using C = RowsCfg<M>;
    auto kern = k_fused_rows<M, AR, FR>;
    epic_status st = lds_ready(reinterpret_cast<const void *>(kern), C::lds(A));
    if (st || dry) return st;
    const int unit = FR ? fo.len : 1;
    const int want = FR ? 64 : part && acc ? g->slices : 1;
    const SliceChoice sl = best_slices(g->n_items, g->slots, n_time, want, g->part_floats, unit, FR);
    const int tps = fixed_slices && !FR ? slice_len(n_time, want, unit) : sl.len;
    const int S = (int)(((int64_t)n_time + tps - 1) / tps);
    float *sets = !FR && S > 1 ? part : nullptr;
    hipLaunchKernelGGL(kern, dim3(g->n_items * S), dim3(C::T), C::lds(A), s,
                       g->items.as<FusedItem>(), g->entries.as<uint4>(), d_volt, vstride, A,
                       n_time, acc, autos, fo.len, fo.out, fo.stride, vb, g->n_items, tps, sets,
                       g->part_floats);
    EPIC_HIP(hipGetLastError());
    if (sets) {
        hipLaunchKernelGGL(k_fused_reduce, dim3(64, g->n_chans), dim3(256), 0, s,
                           g->chans.as<GroupChan>(), S, sets, g->part_floats, acc);
        EPIC_HIP(hipGetLastError());
    }
    return EPIC_OK;
}

template <int M>
static epic_status launch_rows(const FusedGroup *g, const uint8_t *d_volt, int64_t vstride, int A,
                               int vb, int n_time, float *acc, int32_t *autos, const FrameOut &fo,
                               hipStream_t s, bool dry, float *part, bool fixed_slices) {
    constexpr int T = RowsCfg<M>::T;
#define EPIC_ROWS(AR)                                                                              \
    (fo.len ? launch_rows_fr<M, AR, true>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, \
                                               s, dry, nullptr, fixed_slices)                     \
            : launch_rows_fr<M, AR, false>(g, d_volt, vstride, A, vb, n_time, acc, autos, fo, \
                                                s, dry, part, fixed_slices))
    if (A <= T) return EPIC_ROWS(1);
    if (A <= 2 * T) return EPIC_ROWS(2);
    return EPIC_ROWS(4);
#undef EPIC_ROWS
}

// One persistent launch over the plan's work queue (EPIC_BATCH_QUEUE).
static epic_status queue_launch(epic_plan p, epic_acc acc, const uint8_t *d_volt, int n_time,
                                hipStream_t s, bool dry) {
    const void *kern = p->P == 2 ? reinterpret_cast<const void *>(k_fused_queue<2>)
                                 : reinterpret_cast<const void *>(k_fused_queue<1>);
    const size_t lds = sizeof(float2) * p->P * kQueueGrid + sizeof(float4) * ((size_t)p->A + 1);
    epic_status st = lds_ready(kern, lds);
    if (st || dry || p->n_units == 0) return st;
    QueueSizes qs{};
    const FusedGroup *grp[3] = {nullptr, nullptr, nullptr};
    for (const FusedGroup *g : p->groups) {
        if (g->kind != 0) continue;
        const int k = g->M == 64 ? 0 : g->M == 32 ? 1 : 2;
        grp[k] = g;
        qs.it[k] = g->items.as<FusedItem>();
        qs.e[k] = g->entries.as<uint4>();
        // slices in use for this call: at most one per sample
        qs.tps[k] = (n_time + g->slices - 1) / g->slices;
        qs.used[k] = (n_time + qs.tps[k] - 1) / qs.tps[k];
        qs.part[k] = qs.used[k] > 1 ? reinterpret_cast<float *>(acc->d_work.as<char>() + g->work_off)
                                    : nullptr;
        qs.pstride[k] = g->part_floats;
    }
    int dev = 0, n_cu = 0, per_cu = 0;
    EPIC_HIP(hipGetDevice(&dev));
    EPIC_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    EPIC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 512, lds));
    const int wgs = std::max(1, std::min(p->n_units, n_cu * std::max(1, per_cu)));
    unsigned int *head = reinterpret_cast<unsigned int *>(acc->d_work.as<char>() + p->queue_off);
    if (!acc->d_work.p || acc->d_work.bytes < (size_t)p->queue_off + 256)
        return fail(EPIC_ERR_ARG, "accumulator has no work-queue counter");
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(1), 0, s, head);
    EPIC_HIP(hipGetLastError());
    if (p->P == 2)
        hipLaunchKernelGGL(k_fused_queue<2>, dim3(wgs), dim3(512), lds, s,
                           p->d_units.as<QueueUnit>(), p->n_units, head, qs, d_volt,
                           p->vstride(), p->A, n_time, p->vb, acc->d_acc.as<float>());
    else
        hipLaunchKernelGGL(k_fused_queue<1>, dim3(wgs), dim3(512), lds, s,
                           p->d_units.as<QueueUnit>(), p->n_units, head, qs, d_volt,
                           p->vstride(), p->A, n_time, p->vb, acc->d_acc.as<float>());
    EPIC_HIP(hipGetLastError());
    // sliced sizes: add the partial image sets in slice order
    for (int k = 0; k < 3; ++k) {
        if (!grp[k] || !qs.part[k]) continue;
        hipLaunchKernelGGL(k_fused_reduce, dim3(64, grp[k]->n_chans), dim3(256), 0, s,
                           grp[k]->chans.as<GroupChan>(), qs.used[k], qs.part[k],
                           grp[k]->part_floats, acc->d_acc.as<float>());
        EPIC_HIP(hipGetLastError());
    }
    return EPIC_OK;
}

// Launches every size group; group i goes to branches[i] when given (graph
// capture with parallel branches), else to s.  dry: only set up the kernels'
// LDS allowance (done before a capture).  fo.len > 0: frame mode -- every
// fo.len samples the sums go to the next image set of fo.out, the
// accumulator's sums and self terms are left alone.
epic_status fused_accumulate(epic_plan p, epic_acc acc, const uint8_t *d_volt, int n_time,
                             hipStream_t s, const std::vector<hipStream_t> *branches, bool dry,
                             const FrameOut &fo) {
    const int64_t vstride = p->vstride();
    const bool frames = fo.len > 0;
    float *a = acc && !frames ? acc->d_acc.as<float>() : nullptr;
    // The fused kernels add the self-term sums when every group's threads
    // cover the elements in at most four rounds (one round in row-unfolded
    // groups, whose registers are full) and no channel is banded;
    // otherwise a separate pass does it for every channel.
    bool in_kernel = p->band.n == 0;
    for (const FusedGroup *g : p->groups)
        if (p->A > (g->kind == 2 ? 1 : 4) * threads_of(g)) in_kernel = false;
    int32_t *au = (in_kernel && acc && !frames) ? acc->d_autos.as<int32_t>() : nullptr;
    if (p->band.n) {
        // forks onto the accumulator's own queues; joined back into s below
        // (and here when it fails, so no queue is left forked)
        epic_status st = banded_accumulate(p, acc, d_volt, n_time, s, dry, fo);
        if (st) {
            if (!dry) (void)banded_join(p, acc, s);
            return st;
        }
    }
    if ((p->flags & EPIC_BATCH_QUEUE) && !frames) {
        epic_status st = queue_launch(p, acc, d_volt, n_time, s, dry);
        if (st) return st;
        if (dry) return EPIC_OK;
        st = autos_accumulate(p, acc, d_volt, n_time, s);
        if (st) return st;
        return p->band.n ? banded_join(p, acc, s) : EPIC_OK;
    }
    for (size_t gi = 0; gi < p->groups.size(); ++gi) {
        const FusedGroup *g = p->groups[gi];
        const hipStream_t gs = branches ? (*branches)[gi] : s;
        epic_status st = EPIC_OK;
        const int A = p->A;
        const int vb = p->vb;
        float *part = (acc && g->slices > 1)
                          ? reinterpret_cast<float *>(acc->d_work.as<char>() + g->work_off)
                          : nullptr;
        const bool fixed_slices = p->time_slices > 0;
        if (g->kind == 2) {
            if (g->M == 32) st = launch_rows<32>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part, fixed_slices);
            if (g->M == 16) st = launch_rows<16>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part, fixed_slices);
        } else if (g->kind == 1 && p->J == 4) {
            st = launch_pair<true>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
        } else if (g->kind == 1) {
            st = launch_pair<false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
        } else if (p->J == 4) {
            if (g->M == 64) st = launch_fused<64, 2, true>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 32) st = launch_fused<32, 2, true>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 16) st = launch_fused<16, 2, true>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
        } else if (p->P == 2) {
            if (g->M == 64) st = launch_fused<64, 2, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 32) st = launch_fused<32, 2, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 16) st = launch_fused<16, 2, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
        } else {
            if (g->M == 64) st = launch_fused<64, 1, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 32) st = launch_fused<32, 1, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
            if (g->M == 16) st = launch_fused<16, 1, false>(g, d_volt, vstride, A, vb, n_time, a, au, fo, gs, dry, part);
        }
        if (st) return st;
    }
    if (dry) return EPIC_OK;
    if (!in_kernel && !frames) {
        epic_status st = autos_accumulate(p, acc, d_volt, n_time, s);
        if (st) return st;
    }
    return p->band.n ? banded_join(p, acc, s) : EPIC_OK;
}

epic_status autos_accumulate(epic_plan p, epic_acc acc, const uint8_t *d_volt, int n_time,
                             hipStream_t s) {
    const int64_t vstride = p->vstride();
    if ((n_time + 63) / 64 > 65535) return fail(EPIC_ERR_ARG, "n_time too large for one call");
    // words of four elements where the element count, the samples' stride and the
    // input's address are multiples of four bytes
    const bool words = p->vb == 1 && p->A % 4 == 0 && vstride % 4 == 0 && (uintptr_t)d_volt % 4 == 0;
    // sample groups of a workgroup for about four thousand waves in all; further
    // time chunks (atomics) only where the chip is not full without, of eight samples
    // a group, all that it has in flight (20 elements x 10 channels x 900 samples: 30 us
    // with 64 samples a group, 4.9 with eight; 20000 x 1 x 781: 14.2 and 9.0)
    const int lanes = words ? 64 : 256;
    const int64_t blocks = (int64_t)((p->A + 255) / 256) * p->C;
    const int64_t want = std::max<int64_t>(1, 4096 * 64 / lanes / blocks);
    const int groups = (int)std::min<int64_t>({want, 1024 / lanes, (n_time + 7) / 8});
    const int64_t chunks = std::max<int64_t>(
        1, std::min<int64_t>(want / groups, ((int64_t)n_time + 8 * groups - 1) / (8 * groups)));
    const int t_chunk = (int)((n_time + chunks - 1) / chunks);
    dim3 grid((p->A + 255) / 256, p->C, (n_time + t_chunk - 1) / t_chunk);
    // at least 256 threads, also where some have no samples: they share the clearing
    // and the writing of the sums (5000 elements of one channel, 4 samples: 8.4 us on
    // one wave each, 4.0 us so)
    const int rows = std::max(groups, 256 / lanes);
#define EPIC_AUTOS(PP, VV, EE)                                                               \
    hipLaunchKernelGGL((k_autos<PP, VV, EE>), grid, dim3(lanes, rows), 0, s, d_volt,         \
                       vstride, p->A, n_time, t_chunk, acc->d_autos.as<int32_t>())
    if (p->P == 2) {
        if (p->vb == 2) EPIC_AUTOS(2, 2, 1);
        else if (words) EPIC_AUTOS(2, 1, 4);
        else EPIC_AUTOS(2, 1, 1);
    } else {
        if (p->vb == 2) EPIC_AUTOS(1, 2, 1);
        else if (words) EPIC_AUTOS(1, 1, 4);
        else EPIC_AUTOS(1, 1, 1);
    }
#undef EPIC_AUTOS
    EPIC_HIP(hipGetLastError());
    return EPIC_OK;
}

}  // namespace epic

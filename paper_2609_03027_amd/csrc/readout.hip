// Read-out of Eq. 2 (time average) with the per-element self terms removed.
//
// The image of element a's kernel footprint is
//   B_a[k] = sum_j conj(W_a(j)) exp(+2 pi i (k - N/2).(j - N/2) / N),
// and its power pattern expands over footprint displacements d = j - j':
//   |B_a[k]|^2 = sum_d R_a[d] exp(+2 pi i (k - N/2).d / N),
//   R_a[d]     = sum_j conj(W_a(j)) W_a(j - d),
// with d in [-(K-1), K-1]^2.  The self term of product pq is
// sum_a S_a^{pq} |B_a[k]|^2 = sum_d H^{pq}[d] exp(...), H^{pq}[d] =
// sum_a S_a^{pq} R_a[d], a (2K-1)^2-term sum per pixel.  H and the per-pixel sum are formed in FP64 from the exact int32
// self-term sums.  With Jones kernels (four per element) the same expansion
// holds per pair of kernels; see k_auto_h_jones.
#include <mutex>

#include "internal.h"

namespace epic {

// R_a[-d] = conj(R_a[d]), so R is kept for the displacements with linear index
// d >= D^2 / 2 only (the centre and everything after it, DH = D^2 / 2 + 1).
__host__ __device__ constexpr int half_disp(int K) { return (2 * K - 1) * (2 * K - 1) / 2 + 1; }

// Footprint self-correlation R_a[d] = sum_j conj(W_a(j)) W_a(j - d), one
// thread per (element, displacement, channel); layout double2 [C][DH][A].
__global__ void k_selfcorr(const double2 *__restrict__ w, int A, int K, double2 *__restrict__ R) {
    const int D = 2 * K - 1, DH = half_disp(K);
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int d = D * D / 2 + blockIdx.y, c = blockIdx.z;
    if (a >= A) return;
    const int dx = d % D - (K - 1), dy = d / D - (K - 1);
    const double2 *wa = w + ((size_t)c * A + a) * K * K;
    double rr = 0, ri = 0;
    for (int ty = 0; ty < K; ++ty) {
        const int uy = ty - dy;
        if (uy < 0 || uy >= K) continue;
        for (int tx = 0; tx < K; ++tx) {
            const int ux = tx - dx;
            if (ux < 0 || ux >= K) continue;
            const double2 p = wa[ty * K + tx], q = wa[uy * K + ux];
            rr += p.x * q.x + p.y * q.y;  // conj(p) * q
            ri += p.x * q.y - p.y * q.x;
        }
    }
    R[((size_t)c * DH + blockIdx.y) * A + a] = make_double2(rr, ri);
}

// Sums v[0 .. NV) over the 256 threads of a block (NV <= 8): 32 threads take
// one value each, reading eight threads' entries, and finish by shuffles.  The
// sum of value q is returned in thread 32 q.
template <int NV>
__device__ __forceinline__ double block_sum(const double (&v)[NV], double (*red)[256]) {
#pragma unroll
    for (int q = 0; q < NV; ++q) red[q][threadIdx.x] = v[q];
    __syncthreads();
    const int q = threadIdx.x >> 5, i = threadIdx.x & 31;
    double s = 0.0;
    if (q < NV) {
#pragma unroll
        for (int k = 0; k < 8; ++k) s += red[q][i + 32 * k];
    }
#pragma unroll
    for (int st = 16; st > 0; st >>= 1) s += __shfl_down(s, st, 32);
    return s;
}

// H^{pq}[d] = sum_a S_a^{pq} R_a[d]: one 256-thread block per (displacement
// d >= 0, channel) reducing over elements; the same sums give H[-d], since
// R_a[-d] = conj(R_a[d]).  H layout double2 [C][NH][D*D], NH = 1 (XX) or 3
// (XX, YY, XY).  Bound by latency: 128 channels of 256 elements (6.8 MB of R)
// take 5 us against 18 us over every displacement with a tree in LDS.
template <int P>
__global__ __launch_bounds__(256) void k_auto_h(const double2 *__restrict__ R,
                                                const int32_t *__restrict__ autos, int A, int K,
                                                double2 *__restrict__ H) {
    const int D2 = (2 * K - 1) * (2 * K - 1), DH = half_disp(K);
    const int d = D2 / 2 + blockIdx.x, c = blockIdx.y;
    constexpr int NPROD = P == 2 ? 4 : 1;
    constexpr int NV = P == 2 ? 8 : 2;
    double v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = 0.0;
    const double2 *r = R + ((size_t)c * DH + blockIdx.x) * A;
    for (int a = threadIdx.x; a < A; a += blockDim.x) {
        const double2 rv = r[a];
        const int32_t *s = autos + ((size_t)c * A + a) * NPROD;
        const double sxx = (double)s[0];
        v[0] += sxx * rv.x;
        v[1] += sxx * rv.y;
        if (P == 2) {
            const double syy = (double)s[1], sre = (double)s[2], sim = (double)s[3];
            v[2] += syy * rv.x;
            v[3] += syy * rv.y;
            v[4] += sre * rv.x;
            v[5] += sre * rv.y;
            v[6] += sim * rv.x;
            v[7] += sim * rv.y;
        }
    }
    __shared__ double red[NV][256];
    __shared__ double tot[8];
    const double s = block_sum<NV>(v, red);
    if ((threadIdx.x & 31) == 0) tot[threadIdx.x >> 5] = s;
    __syncthreads();
    // entry (product q, sign of d)
    constexpr int NH = P == 2 ? 3 : 1;
    const int q = threadIdx.x >> 1, neg = threadIdx.x & 1;
    if (q >= NH || (neg && 2 * d + 1 == D2)) return;   // the centre: one writer
    double2 o;
    if (q < 2)
        o = make_double2(tot[2 * q], neg ? -tot[2 * q + 1] : tot[2 * q + 1]);
    else
        o = neg ? make_double2(tot[4] + tot[7], tot[6] - tot[5])
                : make_double2(tot[4] - tot[7], tot[6] + tot[5]);
    H[((size_t)c * NH + q) * D2 + (neg ? D2 - 1 - d : d)] = o;
}

// Jones kernels: element a alone puts sum_p B_a^{alpha p} E_a^p on every
// pixel, so its self term of product alpha beta is
//   sum_{p,q} S_a^{pq} B_a^{alpha p} conj(B_a^{beta q})
//     = sum_d [sum_{p,q} S_a^{pq} R_a^{alpha p, beta q}[d]] exp(+2 pi i (k - N/2).d / N),
//   R_a^{alpha p, beta q}[d] = sum_j conj(W_a^{alpha p}(j)) W_a^{beta q}(j - d),
// with S_a^{yx} = conj(S_a^{xy}).  One block per (product, channel), one
// element a thread and step: V_p = sum_q S^{pq} W^{beta q} is formed once per
// footprint cell, each pair of cells then adds sum_p conj(W^{alpha p}) V_p to
// its displacement's register, and the block sums the 2 D^2 registers (a
// wave by shuffles, the waves through LDS).  H layout as for k_auto_h<2>:
// double2 [C][3][D*D] for XX, YY, XY.  LWA-like station (128 channels, 256
// elements, K = 3): 27 us against 181 us with one block per
// displacement, which read every weight 25 times and formed S W again for
// every pair.
template <int K>
__global__ __launch_bounds__(256) void k_auto_h_jones(const double2 *__restrict__ w,
                                                      const int32_t *__restrict__ autos, int A,
                                                      double2 *__restrict__ H) {
    constexpr int D = 2 * K - 1, D2 = D * D, KK = K * K;
    const int ab = blockIdx.x, c = blockIdx.y;
    const int al = ab == 1 ? 1 : 0, be = ab == 0 ? 0 : 1;
    double hr[D2], hi[D2];
#pragma unroll
    for (int d = 0; d < D2; ++d) hr[d] = hi[d] = 0.0;
    for (int a = threadIdx.x; a < A; a += 256) {
        const int32_t *s = autos + ((size_t)c * A + a) * 4;
        const double sxx = (double)s[0], syy = (double)s[1], sre = (double)s[2], sim = (double)s[3];
        const double2 *wa = w + ((size_t)c * A + a) * 4 * KK;
        const double2 *P0 = wa + al * 2 * KK, *Q0 = wa + be * 2 * KK;
#pragma unroll
        for (int u = 0; u < KK; ++u) {
            const double2 q0 = Q0[u], q1 = Q0[KK + u];
            // S[x][x] = sxx, S[x][y] = sre + i sim, S[y][x] its conjugate
            const double2 v0 = make_double2(sxx * q0.x + sre * q1.x - sim * q1.y,
                                            sxx * q0.y + sre * q1.y + sim * q1.x);
            const double2 v1 = make_double2(syy * q1.x + sre * q0.x + sim * q0.y,
                                            syy * q1.y + sre * q0.y - sim * q0.x);
            const int uy = u / K, ux = u % K;
#pragma unroll
            for (int t = 0; t < KK; ++t) {
                const double2 p0 = P0[t], p1 = P0[KK + t];
                const double rr = p0.x * v0.x + p0.y * v0.y + p1.x * v1.x + p1.y * v1.y;
                const double ri = p0.x * v0.y - p0.y * v0.x + p1.x * v1.y - p1.y * v1.x;
                const int d = (t / K - uy + K - 1) * D + (t % K - ux + K - 1);
                hr[d] += rr;
                hi[d] += ri;
            }
        }
    }
    __shared__ double2 part[4][D2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 0; d < D2; ++d) {
        double r = hr[d], i = hi[d];
#pragma unroll
        for (int st = 32; st > 0; st >>= 1) {
            r += __shfl_down(r, st);
            i += __shfl_down(i, st);
        }
        if (lane == 0) part[wave][d] = make_double2(r, i);
    }
    __syncthreads();
    if ((int)threadIdx.x < D2) {
        double2 o = make_double2(0.0, 0.0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o.x += part[k][threadIdx.x].x;
            o.y += part[k][threadIdx.x].y;
        }
        H[((size_t)c * 3 + ab) * D2 + threadIdx.x] = o;
    }
}

// img = (acc - remove * self) * scale.  One block per tile of 64 columns x
// 4 R rows of one channel; a thread keeps one column and takes R rows.  The
// self term sum_d H[d] exp(+2 pi i (k - N/2).d / N) is summed over dx once per
// column, F[dy] = sum_dx H[dy][dx] exp(.. kx dx), so that a pixel costs the
// 2 K - 1 terms over dy instead of (2 K - 1)^2; XX and YY are real (H[-d] =
// conj(H[d])), so they need dy >= 0 only.  All in FP64.  The kernel side K is
// a template argument so that the loops unroll and everything stays in
// registers.  Bound: HBM with R = 8 (16 B read and 16 written per pixel): 128
// channels of 128^2 take 17 us (3.9 TB/s), 43 us with every displacement summed
// per pixel.  R = 2 where R = 8 would make fewer than 1024 blocks, four per CU: a
// small read-out is bound by the latency of its rows.
template <int P, int K, int R>
__global__ __launch_bounds__(256) void k_readout(const float *__restrict__ acc,
                                                 const double2 *__restrict__ H,
                                                 const int4 *__restrict__ chan,
                                                 const int64_t *__restrict__ img_off, int remove,
                                                 int stokes, float scale, float *__restrict__ img) {
    constexpr int RB = 4 * R;
    const int c = blockIdx.y;
    const int N = chan[c].x;
    const int cols = (N + 63) / 64;
    const int ky0 = (int)(blockIdx.x / cols) * RB;
    if (ky0 >= N) return;
    const int kx = (int)(blockIdx.x % cols) * 64 + (threadIdx.x & 63);
    const int64_t plane = (int64_t)N * N;
    constexpr int NPROD = P == 2 ? 4 : 1;
    constexpr int D = 2 * K - 1;
    constexpr int KM = K > 1 ? K - 1 : 1;
    // exp(+2 pi i (k - N/2) / N) with the argument reduced exactly mod N
    auto phase = [&](int k) {
        double sn, cs;
        sincospi(2.0 * (double)(((k - N / 2) % N + N) % N) / (double)N, &sn, &cs);
        return make_double2(cs, sn);
    };
    auto cmul = [](double2 a, double2 b) {
        return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
    };
    __shared__ double2 ey[RB][KM];       // row phase to the powers 1 .. K - 1
    if (remove && K > 1) {
        if ((int)threadIdx.x < RB) {
            const double2 w = phase(ky0 + (int)threadIdx.x);
            double2 e = w;
#pragma unroll
            for (int m = 0; m < KM; ++m) {
                ey[threadIdx.x][m] = e;
                e = cmul(e, w);
            }
        }
        __syncthreads();
    }
    if (kx >= N) return;
    const int r0 = (int)(threadIdx.x >> 6) * R;
    const float *a = acc + img_off[c] + (int64_t)(ky0 + r0) * N + kx;
    float *o = img + img_off[c] + (int64_t)(ky0 + r0) * N + kx;
    const int rows = min(R, N - ky0 - r0);
    float v[R][NPROD];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < NPROD; ++q) v[r][q] = r < rows ? a[r * N + q * plane] : 0.f;
    // products (XX, YY, Re XY, Im XY) -> output planes: as they are, or the
    // pseudo-Stokes set I = XX + YY, Q = XX - YY, U = 2 Re XY, V = -2 Im XY
    auto put = [&](int r, double xx, double yy, double xr, double xi) {
        float *q = o + r * N;
        if (P == 2 && stokes) {
            q[0] = (float)((xx + yy) * scale);
            q[plane] = (float)((xx - yy) * scale);
            q[2 * plane] = (float)(2.0 * xr * scale);
            q[3 * plane] = (float)(-2.0 * xi * scale);
        } else {
            q[0] = (float)(xx * scale);
            if (P == 2) {
                q[plane] = (float)(yy * scale);
                q[2 * plane] = (float)(xr * scale);
                q[3 * plane] = (float)(xi * scale);
            }
        }
    };
    if (!remove) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r >= rows) break;
            if (P == 2 && stokes) {
                put(r, v[r][0], v[r][1], v[r][2], v[r][3]);
            } else {
#pragma unroll
                for (int q = 0; q < NPROD; ++q) o[r * N + q * plane] = v[r][q] * scale;
            }
        }
        return;
    }
    constexpr int NH = P == 2 ? 3 : 1;
    const double2 *h = H + (size_t)c * NH * D * D;
    // powers of the column phase, dx = -(K-1) .. K-1
    double2 px[D];
    px[K - 1] = make_double2(1.0, 0.0);
    if (K > 1) {
        const double2 wx = phase(kx);
#pragma unroll
        for (int m = 1; m < K; ++m) {
            px[K - 1 + m] = cmul(px[K - 2 + m], wx);
            px[K - 1 - m] = make_double2(px[K - 1 + m].x, -px[K - 1 + m].y);
        }
    }
    auto column = [&](int q, int iy) {        // F[dy = iy - (K - 1)] of product q
        double2 f = make_double2(0.0, 0.0);
#pragma unroll
        for (int ix = 0; ix < D; ++ix) {
            const double2 t = h[(q * D + iy) * D + ix];
            f.x += t.x * px[ix].x - t.y * px[ix].y;
            f.y += t.x * px[ix].y + t.y * px[ix].x;
        }
        return f;
    };
    // XX, YY: F0 + sum_m 2 (Re F_m c_m - Im F_m s_m); XY: the real part is
    // F0.x + sum_m (p_m c_m - q_m s_m), the imaginary F0.y + sum_m (u_m c_m + w_m s_m)
    double f0[4];
    double2 fc[4][KM];
#pragma unroll
    for (int q = 0; q < (P == 2 ? 2 : 1); ++q) {
        f0[q] = column(q, K - 1).x;
#pragma unroll
        for (int m = 1; m < K; ++m) {
            const double2 f = column(q, K - 1 + m);
            fc[q][m - 1] = make_double2(2.0 * f.x, -2.0 * f.y);
        }
    }
    if (P == 2) {
        const double2 f = column(2, K - 1);
        f0[2] = f.x;
        f0[3] = f.y;
#pragma unroll
        for (int m = 1; m < K; ++m) {
            const double2 fp = column(2, K - 1 + m), fn = column(2, K - 1 - m);
            fc[2][m - 1] = make_double2(fp.x + fn.x, fn.y - fp.y);
            fc[3][m - 1] = make_double2(fp.y + fn.y, fp.x - fn.x);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= rows) break;
        double self[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < NPROD; ++q) {
            self[q] = f0[q];
#pragma unroll
            for (int m = 1; m < K; ++m) {
                const double2 e = ey[r0 + r][m - 1];
                self[q] += fc[q][m - 1].x * e.x + fc[q][m - 1].y * e.y;
            }
        }
        if (P == 2)
            put(r, (double)v[r][0] - self[0], (double)v[r][1] - self[1], (double)v[r][2] - self[2],
                (double)v[r][3] - self[3]);
        else
            put(r, (double)v[r][0] - self[0], 0.0, 0.0, 0.0);
    }
}

epic_status selfcorr_build(epic_plan p, hipStream_t s) {
    const int DH = half_disp(p->K);
    epic_status st = p->d_selfcorr.alloc(sizeof(double2) * (size_t)p->C * DH * p->A);
    if (st) return st;
    dim3 g((p->A + 255) / 256, DH, p->C);
    hipLaunchKernelGGL(k_selfcorr, g, dim3(256), 0, s, p->d_w.as<double2>(), p->A, p->K,
                       p->d_selfcorr.as<double2>());
    EPIC_HIP(hipGetLastError());
    return EPIC_OK;
}

// The read-out proper: sums `a`, self-term sums `autos` (read only when
// removing), sample count, and `H` the [C][NH][D*D] FP64 table k_auto_h fills.
static epic_status readout_core(epic_plan p, const float *a, const int32_t *autos, int64_t count,
                                double2 *H, float *d_img, uint32_t flags, hipStream_t s) {
    const bool remove = (flags & EPIC_REMOVE_AUTOS) != 0;
    const bool norm = (flags & EPIC_NORMALISE) != 0;
    const int stokes = (flags & EPIC_STOKES) ? 1 : 0;
    if (stokes && p->P != 2) return fail(EPIC_ERR_ARG, "pseudo-Stokes needs two feeds");
    if (norm && count <= 0) return fail(EPIC_ERR_ARG, "normalise requested with no samples");
    const float scale = norm ? (float)(1.0 / (double)count) : 1.0f;
    const double2 *w = p->d_w.as<double2>();
    if (remove && p->J == 4) {
        dim3 g(3, p->C);
        if (p->K == 1)
            hipLaunchKernelGGL(k_auto_h_jones<1>, g, dim3(256), 0, s, w, autos, p->A, H);
        else if (p->K == 2)
            hipLaunchKernelGGL(k_auto_h_jones<2>, g, dim3(256), 0, s, w, autos, p->A, H);
        else
            hipLaunchKernelGGL(k_auto_h_jones<3>, g, dim3(256), 0, s, w, autos, p->A, H);
        EPIC_HIP(hipGetLastError());
    } else if (remove) {
        dim3 g(half_disp(p->K), p->C);
        const double2 *R = p->d_selfcorr.as<double2>();
        if (p->P == 2)
            hipLaunchKernelGGL(k_auto_h<2>, g, dim3(256), 0, s, R, autos, p->A, p->K, H);
        else
            hipLaunchKernelGGL(k_auto_h<1>, g, dim3(256), 0, s, R, autos, p->A, p->K, H);
        EPIC_HIP(hipGetLastError());
    }
    // tiles of the largest side: blocks past a smaller channel's end return
    const int cols = (p->max_n + 63) / 64;
    const int tiles8 = cols * ((p->max_n + 31) / 32), tiles2 = cols * ((p->max_n + 7) / 8);
    const bool wide = (int64_t)tiles8 * p->C >= 1024;
    dim3 g(wide ? tiles8 : tiles2, p->C);
    const double2 *h = H;
    const int4 *ch = p->d_chan.as<int4>();
    const int64_t *off = p->d_img_off.as<int64_t>();
    const int rm = remove ? 1 : 0;
#define EPIC_READOUT(PP, KK)                                                                      \
    do {                                                                                          \
        auto kern = wide ? k_readout<PP, KK, 8> : k_readout<PP, KK, 2>;                           \
        hipLaunchKernelGGL(kern, g, dim3(256), 0, s, a, h, ch, off, rm, stokes, scale, d_img);    \
    } while (0)
    switch (p->P * 4 + p->K) {
        case 9: EPIC_READOUT(2, 1); break;
        case 10: EPIC_READOUT(2, 2); break;
        case 11: EPIC_READOUT(2, 3); break;
        case 5: EPIC_READOUT(1, 1); break;
        case 6: EPIC_READOUT(1, 2); break;
        case 7: EPIC_READOUT(1, 3); break;
        default: return fail(EPIC_ERR_UNSUPPORTED, "read-out: feeds or kernel size");
    }
#undef EPIC_READOUT
    EPIC_HIP(hipGetLastError());
    return EPIC_OK;
}

epic_status readout(epic_plan p, epic_acc acc, float *d_img, uint32_t flags, hipStream_t s) {
    return readout_core(p, acc->d_acc.as<float>(), acc->d_autos.as<int32_t>(), acc->count,
                        acc->d_h.as<double2>(), d_img, flags, s);
}

// Read-out without allocation: the self-term table H lives in this
// file-scope device array (one copy per GPU, held until the process ends).
// In host code `scratch` names a host-side stand-in, never the device copy;
// the device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kNoAllocH = 65536;   // double2 entries: 1 MiB
static __device__ __align__(256) double2 scratch[kNoAllocH];

static std::mutex g_scratch_mu;
static double2 *g_scratch_ptr[64] = {};

static epic_status scratch_ptr(double2 **out) {
    int dev = 0;
    EPIC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(EPIC_ERR_UNSUPPORTED, "device index above 63");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[dev] = static_cast<double2 *>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return EPIC_OK;
}

int64_t readout_noalloc_max_channels(epic_plan p) {
    const int D = 2 * p->K - 1;
    return (int64_t)(kNoAllocH / (size_t)((p->P == 2 ? 3 : 1) * D * D));
}

epic_status readout_noalloc(epic_plan p, const float *d_acc, const int32_t *d_autos,
                            int64_t count, float *d_img, uint32_t flags, hipStream_t s) {
    const int D = 2 * p->K - 1;
    const size_t need = (size_t)p->C * (p->P == 2 ? 3 : 1) * D * D;
    if (need > kNoAllocH)
        return fail(EPIC_ERR_BUDGET, "read-out without allocation: the self-term table needs " +
                                         std::to_string(need * sizeof(double2)) +
                                         " bytes, above the library's 1 MiB scratch (at most " +
                                         std::to_string(readout_noalloc_max_channels(p)) +
                                         " channels for this plan)");
    double2 *h = nullptr;
    epic_status st = scratch_ptr(&h);
    if (st) return st;
    return readout_core(p, d_acc, d_autos, count, h, d_img, flags, s);
}

}  // namespace epic

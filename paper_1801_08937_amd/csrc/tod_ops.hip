// Time-domain operators: P (map -> TOD gather), P^T (pixel-sorted segmented
// reduction, no float atomics), the banded-Toeplitz N^-1 applied directly,
// and the flag mask applied to the data.  The FFT form of N^-1 lives in
// noise_fft.hip.
//
// Layouts: map x[(3 j + a) R + r] (FP64); TOD y[t R + r] (T = float or double).
// With several columns a lane holds two of them (P, P^T from 8 columns) or one (P^T of
// 2 and 4, the direct band), and a wave's lanes are split into sample groups of R
// columns, so one wave step touches consecutive samples x R columns: contiguous TOD
// rows.  Each column is computed with the same arithmetic and order whatever the other
// columns hold.
#include <algorithm>
#include <functional>
#include <type_traits>

#include "mm_internal.h"
#include "pointing_gather.h"
#include "xcd.h"

namespace mm {

namespace {

constexpr int BS = 256;

template <typename T>
__global__ void __launch_bounds__(BS) k_zero(int64_t n, T *__restrict__ y) {
    for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < n; e += (int64_t)gridDim.x * BS)
        y[e] = (T)0;
}

template <typename E> struct Pair {  // two neighbours at any alignment
    typedef E type __attribute__((ext_vector_type(2), aligned(sizeof(E))));
};

// Columns r and r + 1 of P x at U samples (pixels j, weights ww), maps
// x[(NC j + a) R + r], NC = 3: weights 1, cos, sin; 2: cos, sin; 1: 1.  Branch-free,
// so that the U x NC gathers are in flight together: an unobserved sample (j < 0)
// reads pixel 0 and yields 0 (the map is never empty here).
template <typename T, int R, int NC, int U>
__device__ __forceinline__ void p_rows(const int32_t (&j)[U],
                                       const typename Vec2<T>::type (&ww)[U],
                                       const double *__restrict__ x, int r,
                                       typename Pair<T>::type (&o)[U]) {
    typedef typename Pair<double>::type d2;
    d2 m[U][NC];
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
        for (int a = 0; a < NC; ++a)
            m[q][a] = *reinterpret_cast<const d2 *>(
                x + ((int64_t)NC * (j[q] < 0 ? 0 : j[q]) + a) * R + r);
#pragma unroll
    for (int q = 0; q < U; ++q) {
        auto at = [&](auto v) {
            if constexpr (NC == 1) return (T)v(0);
            else if constexpr (NC == 2) return ww[q].x * (T)v(0) + ww[q].y * (T)v(1);
            else return (T)v(0) + ww[q].x * (T)v(1) + ww[q].y * (T)v(2);
        };
        o[q].x = at([&](int a) { return m[q][a].x; });
        o[q].y = at([&](int a) { return m[q][a].y; });
        if (j[q] < 0) o[q] = (T)0;
    }
}

// y = P x for R > 1 columns of IQU, QU or I maps.  A lane holds two columns of a sample, and a wave takes `per`
// consecutive samples, PR_U x 128 / R at a time: PR_U pixel indices and weights, then
// the PR_U x NC map gathers, are in flight together.  The output is interleaved, or
// planar with the columns `plane` apart (plane > 0).  Bound by HBM at 20 + 8 R bytes
// per sample (IQU, FP64).  One column per lane, samples a grid's stride apart, took
// (us, before and after): 8.4M samples x 4 columns 175 -> 62 (7.0 TB/s, part of it
// from the Infinity Cache); 1M x 16 44 -> 24, x 64 230 -> 97; 65,536 x 64 14 -> 9;
// I, 1M x 64 179 -> 92.  PR_U = 4 takes 70 us where 2 takes 62.
constexpr int PR_U = 2;
constexpr int P_PLANAR_COLS = 16;  // most columns of a planar output
template <typename T, int R, int NC>
__global__ void __launch_bounds__(BS) k_apply_P(const int32_t *__restrict__ jpix,
                                                const typename Vec2<T>::type *__restrict__ w,
                                                int64_t n, int64_t per, int64_t plane,
                                                const double *__restrict__ x,
                                                T *__restrict__ y) {
    typedef typename Pair<T>::type t2;
    constexpr int LPS = R / 2, SPW = 64 / LPS;
    const int lane = threadIdx.x & 63, sub = lane / LPS, r = 2 * (lane % LPS);
    const int64_t t0 = (((int64_t)blockIdx.x * BS + threadIdx.x) >> 6) * per;
    const int64_t t1 = t0 + per < n ? t0 + per : n;
    for (int64_t t = t0 + sub; t - sub < t1; t += PR_U * SPW) {
        int32_t j[PR_U];
        typename Vec2<T>::type ww[PR_U];
#pragma unroll
        for (int q = 0; q < PR_U; ++q) {
            const int64_t tq = t + q * SPW < t1 ? t + q * SPW : t1 - 1;
            j[q] = jpix[tq];
            if constexpr (NC > 1) ww[q] = w[tq];
        }
        t2 o[PR_U];
        p_rows<T, R, NC, PR_U>(j, ww, x, r, o);
#pragma unroll
        for (int q = 0; q < PR_U; ++q) {
            const int64_t tq = t + q * SPW;
            if (tq < t1) {
                if (R > P_PLANAR_COLS || plane == 0) {
                    __builtin_nontemporal_store(o[q], reinterpret_cast<t2 *>(y + tq * R + r));
                } else {
                    __builtin_nontemporal_store((T)o[q].x, y + r * plane + tq);
                    __builtin_nontemporal_store((T)o[q].y, y + (r + 1) * plane + tq);
                }
            }
        }
    }
}

// The copies of an IQU map for the FP32 P of one column: 32-byte records (I, Q, U, 0)
// at each of the n_copies slots of every pixel, so that a sample's gather is two aligned
// 16-byte loads instead of three 8-byte ones.
__global__ void __launch_bounds__(BS) k_pack_map(const double *__restrict__ x, int32_t n_obs,
                                                 int n_copies, const int32_t *__restrict__ slot,
                                                 double2 *__restrict__ x4) {
    for (int64_t j = (int64_t)blockIdx.x * BS + threadIdx.x; j < n_obs;
         j += (int64_t)gridDim.x * BS) {
        const double2 iq = make_double2(x[3 * j], x[3 * j + 1]);
        const double2 u0 = make_double2(x[3 * j + 2], 0.0);
        for (int g = 0; g < n_copies; ++g) {
            const int64_t s = slot[(int64_t)g * n_obs + j];
            x4[2 * s] = iq;
            x4[2 * s + 1] = u0;
        }
    }
}

// The copies for the FP64 P: I in xi, (Q, U) in xqu, at each of the n_copies slots of
// every pixel.
__global__ void __launch_bounds__(BS) k_pack_map_split(const double *__restrict__ x,
                                                       int32_t n_obs, int n_copies,
                                                       const int32_t *__restrict__ slot,
                                                       double *__restrict__ xi,
                                                       double2 *__restrict__ xqu) {
    for (int64_t c = (int64_t)blockIdx.x * BS + threadIdx.x; c < n_obs;
         c += (int64_t)gridDim.x * BS) {
        const double vi = x[3 * c];
        const double2 vqu = make_double2(x[3 * c + 1], x[3 * c + 2]);
        for (int g = 0; g < n_copies; ++g) {
            const int64_t s = slot[(int64_t)g * n_obs + c];
            xi[s] = vi;
            xqu[s] = vqu;
        }
    }
}

// y = P x, one column: a thread forms two neighbouring samples, read and
// written in one access per stream, and blocks take consecutive samples, so the
// blocks resident together gather from neighbouring pixels.  FP64 forms the
// weights from the stored angles (12 bytes per sample with the slot, against 20
// with stored weights).  Bound by HBM: 2^27 samples with three map copies (IQU
// FP64) 595 -> 537 us, 5.0 TB/s of its 20 bytes per sample, the rate of a copy; 2^25
// 240 -> 142 us, 2^23 54 -> 39 us.  Eight samples per thread a grid's stride apart
// (150 VGPRs, three waves per SIMD, and only one sample per thread below 2^26)
// was the earlier form; four neighbours per thread take 595 us, one 684 us, and
// contiguous runs of blocks per XCD 603 us.
template <typename T, typename S>
__global__ void __launch_bounds__(BS) k_apply_P1(S src, int64_t n, T *__restrict__ y) {
    const int64_t t = 2 * ((int64_t)blockIdx.x * BS + threadIdx.x);
    if (t + 1 < n) {
        typedef T t2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));
        T v[2];
        src.get_pair(t, v);
        const t2 o = {v[0], v[1]};
        // written once, read by the next kernel from beyond the L2
        __builtin_nontemporal_store(o, reinterpret_cast<t2 *>(y + t));
    } else if (t < n) {
        const int64_t t1[1] = {t};
        T v[1];
        src.get(t1, v);
        y[t] = v[0];
    }
}

// Pixels are visited in the order `order` (NULL = ascending), e.g. square
// tiles of the map, and each XCD takes a contiguous range of that order: the
// pixels one XCD reduces together are neighbours, hit by the same stretches of
// the scan, so their gathers of z share cache lines in that XCD's L2.
template <typename T, int R, int NC>
__global__ void __launch_bounds__(BS) k_apply_PT(const int32_t *__restrict__ off,
                                                 const int32_t *__restrict__ perm,
                                                 const typename Vec2<T>::type *__restrict__ ws,
                                                 int32_t n_obs, const int32_t *__restrict__ order,
                                                 const T *__restrict__ z,
                                                 double *__restrict__ x) {
    constexpr int G = 64 / R;
    const int lane = threadIdx.x & 63;
    const int sub = lane / R, r = lane % R;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t s = blk * (BS / 64) + (threadIdx.x >> 6);
    if (s >= n_obs) return;
    const int64_t j = order ? order[s] : s;
    const int32_t a = off[j], b = off[j + 1];
    T acc[NC] = {};
    auto add = [&](T zq, typename Vec2<T>::type wq) {
        if constexpr (NC != 2) acc[0] += zq;
        if constexpr (NC > 1) {
            acc[NC - 2] += wq.x * zq;
            acc[NC - 1] += wq.y * zq;
        }
    };
    int32_t i = a + sub;
    // IQU: four entries in flight per lane, accumulated in segment order (I and QU, whose
    // loop the compiler unrolls further: 3M samples on 77 x 77 pixels, QU FP64 21 us, and
    // 25 with four; I 16 and 18; 8.4M x 2 columns, I 41 and 66)
    for (; NC == 3 && i + 3 * G < b; i += 4 * G) {
        int32_t tt[4];
        T zz[4];
        typename Vec2<T>::type ww[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) tt[q] = perm[i + q * G];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            zz[q] = z[(int64_t)tt[q] * R + r];
            if constexpr (NC > 1) ww[q] = ws[i + q * G];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) add(zz[q], ww[q]);
    }
    for (; i < b; i += G) {
        typename Vec2<T>::type wq{};
        if constexpr (NC > 1) wq = ws[i];
        add(z[(int64_t)perm[i] * R + r], wq);
    }
#pragma unroll
    for (int m = 32; m >= R; m >>= 1)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] += __shfl_xor(acc[c], m);
    if (sub == 0)
#pragma unroll
        for (int c = 0; c < NC; ++c) x[((int64_t)NC * j + c) * R + r] = (double)acc[c];
}

// Sliced single-column P^T.  Wave w = s G + g (remapped so that each XCD takes
// a contiguous range of w) owns 64 pixels (one per lane) and time segment s;
// every lane walks its pixel's entries of that segment in time order and
// accumulates in registers.  Lanes hold neighbouring pixels, and all waves
// are resident together, so the whole grid advances through the TOD at a
// similar pace and the lines of z it gathers are shared in L2 and the
// Infinity Cache instead of re-read from HBM.  Partial maps per segment go to
// part[s][3 c + a] (or straight to x when S = 1).
// FP32 I and QU sums are kept in FP64: a lane's chain of hits / (S directions) samples
// is longer than the 64-way split of the one-wave-per-pixel form (512 samples in 8
// segments: rounding 3.5e-6 of a sample against 2.0e-6).
template <typename T, int NC>
__global__ void __launch_bounds__(BS) k_apply_PT_sl(const int64_t *__restrict__ base,
                                                    const int32_t *__restrict__ sl_perm,
                                                    const typename SlRec<T>::type *__restrict__ sl_w,
                                                    const int32_t *__restrict__ sl_pix, int32_t G,
                                                    int32_t S, int32_t n_obs,
                                                    const T *__restrict__ z,
                                                    double *__restrict__ out) {
    using A = std::conditional_t<NC == 3, T, double>;
    const int lane = threadIdx.x & 63;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t w = blk * (BS / 64) + (threadIdx.x >> 6);
    if (w >= (int64_t)G * S) return;
    const int32_t sg = (int32_t)(w / G), g = (int32_t)(w % G);
    const int64_t b0 = base[w];
    const int64_t W = (base[w + 1] - b0) >> 6;
    const int32_t *pp = sl_perm + b0 + lane;
    const auto *wp = NC > 1 ? sl_w + b0 + lane : nullptr;
    A s0 = 0, s1 = 0, s2 = 0;
    int64_t k = 0;
    // eight entries in flight per lane, accumulated in entry order
    for (; k + 7 < W; k += 8) {
        int32_t tt[8];
        typename SlRec<T>::type ww[8];
        T zz[8];
        // the sample indices and weights are read once: non-temporal, so
        // that they do not push the gathered z lines out of the L2
#pragma unroll
        for (int q = 0; q < 8; ++q) tt[q] = __builtin_nontemporal_load(pp + 64 * (k + q));
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if constexpr (NC > 1) ww[q] = nt_load_w(wp + 64 * (k + q));
            // a padding entry (-1) reads sample 0 and adds 0: no branch
            // between the eight gathers
            const T zq = z[tt[q] < 0 ? 0 : tt[q]];
            zz[q] = tt[q] >= 0 ? zq : (T)0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if constexpr (NC != 2) s0 += (A)zz[q];
            if constexpr (NC > 1) {
                T c, sn;
                SlRec<T>::weights(ww[q], c, sn);
                s1 += (A)c * (A)zz[q];
                s2 += (A)sn * (A)zz[q];
            }
        }
    }
    for (; k < W; ++k) {
        const int32_t tq = pp[64 * k];
        const T zq = tq >= 0 ? z[tq] : (T)0;
        if constexpr (NC != 2) s0 += (A)zq;
        if constexpr (NC > 1) {
            T c, sn;
            SlRec<T>::weights(wp[64 * k], c, sn);
            s1 += (A)c * (A)zq;
            s2 += (A)sn * (A)zq;
        }
    }
    const int32_t c = sl_pix[(int64_t)g * 64 + lane];
    if (c < 0) return;
    double *o = out + ((int64_t)sg * n_obs + c) * NC;
    if constexpr (NC != 2) *o++ = (double)s0;
    if constexpr (NC > 1) {
        o[0] = (double)s1;
        o[1] = (double)s2;
    }
}

// x[e] = part[0][e] + part[1][e] + ... in segment order; the partials' loads
// are issued eight at a time (a runtime-length loop would wait for each).
__global__ void __launch_bounds__(BS) k_pt_sum_parts(const double *__restrict__ part, int32_t S,
                                                     int64_t n3, double *__restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < n3;
         e += (int64_t)gridDim.x * BS) {
        double acc = part[e];
        int32_t sg = 1;
        for (; sg + 7 < S; sg += 8) {
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = part[(sg + q) * n3 + e];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc += v[q];
        }
        for (; sg < S; ++sg) acc += part[sg * n3 + e];
        x[e] = acc;
    }
}

// The copies of an I or QU map, NC values per slot.
template <int NC>
__global__ void __launch_bounds__(BS) k_pack_map_nc(const double *__restrict__ x, int32_t n_obs,
                                                    int n_copies,
                                                    const int32_t *__restrict__ slot,
                                                    double *__restrict__ xm) {
    for (int64_t c = (int64_t)blockIdx.x * BS + threadIdx.x; c < n_obs;
         c += (int64_t)gridDim.x * BS) {
        double v[NC];
#pragma unroll
        for (int a = 0; a < NC; ++a) v[a] = x[NC * c + a];
        for (int g = 0; g < n_copies; ++g) {
            const int64_t s = slot[(int64_t)g * n_obs + c];
#pragma unroll
            for (int a = 0; a < NC; ++a) xm[NC * s + a] = v[a];
        }
    }
}

// P^T of several columns: a lane holds two columns of an entry, 128 / R entries per
// wave side by side and PT_U of those steps in flight.  A pixel is a wave's (S = 1),
// or a block's (S = 4, each wave a quarter of its entries, added in order) where a wave
// per pixel leaves most of the chip idle.  Bound by HBM and the gathers of z.  Which
// kernel, by the pixels and by hits per pixel times R, h R (pt_form), us, IQU FP64, one
// column per lane (k_apply_PT) / S = 1 / S = 4:
//   h R = 128: 65,536 samples on 4,096 pixels x 8 3.9 / 4.9 / 12.6; 1M on 65,536 x 8
//     28 / 38 / 158; 256: 65,536 on 4,096 x 16 4.5 / 4.5 / 10.7, 262,144 on 16,384 x 16
//     12.1 / 10.5 / 34;
//   2,048: 65,536 on 1,024 x 32 5.8 / 5.1 / 4.8, 262,144 on 1,024 x 8 7.2 / 5.6 / 6.0;
//     4,096: 65,536 on 1,024 x 64 14 / 10.6 / 6.8, 262,144 on 1,024 x 16 15 / 9.3 / 6.8;
//   4,096 pixels: 1M x 64 123 / 95 / 99, 262,144 x 64 24 / 21 / 21; 256 pixels: 1M x 64
//     903 / 596 / 169.
// With four columns one column per lane is the faster form (96 against 104 us).
constexpr int PT_U = 4;
constexpr int PT_MIN_COLS = 8;
template <typename T, int R, int NC, int S>
__global__ void __launch_bounds__(BS) k_apply_PT_cols(
    const int32_t *__restrict__ off, const int32_t *__restrict__ perm,
    const typename Vec2<T>::type *__restrict__ ws, int32_t n_obs,
    const int32_t *__restrict__ order, const T *__restrict__ z, double *__restrict__ x) {
    typedef typename Pair<double>::type d2;
    typedef typename Pair<T>::type t2;
    constexpr int LPS = R / 2, G = 64 / LPS;
    const int lane = threadIdx.x & 63, sub = lane / LPS, r = 2 * (lane % LPS);
    const int wv = threadIdx.x >> 6;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t s = S == 1 ? blk * (BS / 64) + wv : blk;
    if (s >= n_obs) return;
    const int64_t j = order ? order[s] : s;
    int32_t a = off[j], b = off[j + 1];
    if constexpr (S > 1) {
        const int32_t len = b - a, q = len / S, e = len % S;
        a += wv * q + (wv < e ? wv : e);
        b = a + q + (wv < e ? 1 : 0);
    }
    t2 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = (T)0;
    for (int32_t i = a + sub; i < b; i += PT_U * G) {
        int32_t tt[PT_U];
        t2 zz[PT_U];
        typename Vec2<T>::type ww[PT_U];
#pragma unroll
        for (int q = 0; q < PT_U; ++q) {
            const int32_t iq = i + q * G < b ? i + q * G : b - 1;
            tt[q] = perm[iq];
            if constexpr (NC > 1) ww[q] = ws[iq];
        }
#pragma unroll
        for (int q = 0; q < PT_U; ++q) {
            zz[q] = *reinterpret_cast<const t2 *>(z + (int64_t)tt[q] * R + r);
            if (i + q * G >= b) zz[q] = (T)0;  // past the end: the last entry, as 0
        }
#pragma unroll
        for (int q = 0; q < PT_U; ++q) {
            if constexpr (NC != 2) acc[0] += zz[q];
            if constexpr (NC > 1) {
                acc[NC - 2] += ww[q].x * zz[q];
                acc[NC - 1] += ww[q].y * zz[q];
            }
        }
    }
#pragma unroll
    for (int m = 32; m >= LPS; m >>= 1)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            acc[c].x += __shfl_xor(acc[c].x, m);
            acc[c].y += __shfl_xor(acc[c].y, m);
        }
    if constexpr (S > 1) {
        __shared__ t2 part[S][NC][LPS];
        if (sub == 0)
#pragma unroll
            for (int c = 0; c < NC; ++c) part[wv][c][lane] = acc[c];
        __syncthreads();
        if (wv != 0) return;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 1; k < S; ++k) acc[c] += part[k][c][lane % LPS];
    }
    if (sub == 0)
#pragma unroll
        for (int c = 0; c < NC; ++c)
            *reinterpret_cast<d2 *>(x + ((int64_t)NC * j + c) * R + r) =
                d2{(double)acc[c].x, (double)acc[c].y};
}

// plus = (a + b) / 2, minus = (a - b) / 2 (either output may be null; an
// output may be one of the inputs, as each element is read before it is
// written).
template <typename T>
__global__ void __launch_bounds__(BS) k_sum_diff(int64_t n, const T *a, const T *b, T *plus,
                                                 T *minus) {
    for (int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * BS) {
        const T u = a[t], v = b[t];
        if (plus) plus[t] = (u + v) * (T)0.5;
        if (minus) minus[t] = (u - v) * (T)0.5;
    }
}

// Direct band, register-tiled.  A block owns TL = (BS / R) * BT_OPT
// consecutive outputs of one interval for all R columns; thread (g, r) =
// (threadIdx / R, threadIdx mod R) keeps outputs g*BT_OPT .. g*BT_OPT + 7 of
// column r in registers (O = BT_OPT).  The filter is taken as the full symmetric one,
// f[d] = c_|d - lambda|, d = 0 .. 2 lambda, and walked in chunks of at most
// CL taps; for each chunk the taps and the input window [t0 - lambda + d0,
// t0 + TL - lambda + d0 + CL - 1) (zero outside the interval, R values per
// row, so a wave's reads are consecutive) are staged in LDS.  Per block of
// BT_OPT taps a thread loads 15 inputs and 8 taps and does 64 FMAs from
// registers.  Every output sums its taps in ascending offset, chunk after
// chunk, so its value does not depend on R, TL or CL; zero-padded terms add
// exactly +0.
constexpr int BT_OPT = 8;
constexpr int BT_LDS = 65536;  // bytes of LDS per block
// One column on a short stream (nz->band_small): tiles of 512 outputs, so that the few
// tiles of such a stream still spread over the CUs (131,072 samples: 256 blocks
// instead of 64), in blocks of 128 threads with 4 outputs each: 64 threads of 8 took,
// for A of 2^17 samples at lambda 32, 12.2 us where these take 11.3 (lambda 300: 26.8
// and 19.6); 256 of 2 gain on at most 2^17 samples and lose beyond.
constexpr int BAND_SMALL_NT = 128, BAND_SMALL_OPT = 4;

// Stages rows w0 .. w0 + rows - 1 of the R columns (0 outside [a, b)) in sy.
template <typename T> struct TodRows {
    const T *__restrict__ y;
    template <int R, int NT>
    __device__ __forceinline__ void stage(T *__restrict__ sy, int64_t w0, int rows, int64_t a,
                                          int64_t b) const {
        int e = threadIdx.x;
        for (; e + 7 * NT < rows * R; e += 8 * NT) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int eu = e + u * NT;
                const int64_t t = w0 + eu / R;
                const bool in = t >= a && t < b;
                v[u] = y[(in ? t : a) * R + eu % R];
                v[u] = in ? v[u] : (T)0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) sy[e + u * NT] = v[u];
        }
        for (; e < rows * R; e += NT) {
            const int64_t t = w0 + e / R;
            sy[e] = (t >= a && t < b) ? y[t * R + e % R] : (T)0;
        }
    }
};
// One column of P x, gathered here (A = P^T N^-1 P): the window is staged once, for
// all taps, and its 2 lambda halo rows are gathered by the neighbouring tiles too.  A
// in all, P and band apart or in one launch, FP64, lambda 32, us: 2^17 samples
// 11.3 -> 9.0, 2^20 28.3 -> 24.2, 2^25 459 -> 402.  On short streams latency bounds it.
template <typename T, typename S> struct PRows {
    S src;
    template <int R, int NT>
    __device__ __forceinline__ void stage(T *__restrict__ sy, int64_t w0, int rows, int64_t a,
                                          int64_t b) const {
        static_assert(R == 1, "");
        constexpr int U = 5;
        for (int e = threadIdx.x; e < rows; e += U * NT) {
            int64_t t[U];
            T v[U];
            bool in[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t[u] = w0 + e + u * NT;
                in[u] = t[u] >= a && t[u] < b;
                t[u] = in[u] ? t[u] : a;
            }
            src.get(t, v);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e + u * NT < rows) sy[e + u * NT] = in[u] ? v[u] : (T)0;
        }
    }
};

template <typename T, int R, int NT, int O, typename Rows>
__global__ void __launch_bounds__(NT) k_band_tiled(const int64_t *__restrict__ pref, int n_int,
                                                   const int64_t *__restrict__ istart,
                                                   const int32_t *__restrict__ fid,
                                                   const T *__restrict__ band, int lam, int CL,
                                                   Rows src, T *__restrict__ z) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int TL = (NT / R) * O;
    const int nf = 2 * lam + 1;
    const int nf_pad = (nf + BT_OPT - 1) / BT_OPT * BT_OPT;
    // CL is a multiple of BT_OPT; rounding it here lets the compiler see
    // that the window is 16-byte aligned and read it with 128-bit LDS loads
    const int CLa = CL / BT_OPT * BT_OPT;
    T *sf = reinterpret_cast<T *>(smem_raw);  // CL taps
    T *sy = sf + CLa;                          // (TL + CL - 1) rows of R
    // tile -> interval: pref[i] counts the tiles of intervals before i
    const int64_t bt = blockIdx.x;
    int lo = 0, hi = n_int;  // pref[lo] <= bt < pref[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pref[mid] <= bt) lo = mid; else hi = mid;
    }
    const int64_t iv = lo;
    const int64_t a = istart[iv], b = istart[iv + 1];
    const int64_t t0 = a + (bt - pref[iv]) * TL;
    const T *c = band + (int64_t)fid[iv] * (lam + 1);
    const int r = threadIdx.x % R;
    const int m0 = (threadIdx.x / R) * O;
    T acc[O];
#pragma unroll
    for (int m = 0; m < O; ++m) acc[m] = 0;
    for (int d0 = 0; d0 < nf_pad; d0 += CLa) {
        const int cl = nf_pad - d0 < CLa ? nf_pad - d0 : CLa;
        __syncthreads();  // the previous chunk's reads are done
        // The staging loads are issued eight per thread at a time: each
        // address is clamped to a valid element (tap 0, or the interval's
        // first sample) and the value zeroed where it falls outside, so no
        // load waits behind a branch.  The staged values are the same.
        int k = threadIdx.x;
        for (; k + 7 * NT < cl; k += 8 * NT) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int ku = k + u * NT;
                const int d = d0 + ku - lam;
                const bool in = d0 + ku < nf;
                v[u] = c[in ? (d < 0 ? -d : d) : 0];
                v[u] = in ? v[u] : (T)0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) sf[k + u * NT] = v[u];
        }
        for (; k < cl; k += NT) {
            const int d = d0 + k - lam;
            sf[k] = d0 + k < nf ? c[d < 0 ? -d : d] : (T)0;
        }
        const int rows = TL + cl - 1;
        src.template stage<R, NT>(sy, t0 - lam + d0, rows, a, b);
        __syncthreads();
        for (int db = 0; db < cl; db += O) {
            T w[2 * O - 1], cf[O];
#pragma unroll
            for (int q = 0; q < 2 * O - 1; ++q) w[q] = sy[(m0 + db + q) * R + r];
#pragma unroll
            for (int q = 0; q < O; ++q) cf[q] = sf[db + q];
#pragma unroll
            for (int q = 0; q < O; ++q)
#pragma unroll
                for (int m = 0; m < O; ++m) acc[m] += cf[q] * w[m + q];
        }
    }
    const int64_t t1 = t0 + TL < b ? t0 + TL : b;
#pragma unroll
    for (int m = 0; m < O; ++m) {
        const int64_t t = t0 + m0 + m;
        if (t < t1) z[t * R + r] = acc[m];
    }
}

// Direct band for several columns (8 and more), without LDS: thread (g, r) of
// a wave keeps BC_OPT consecutive outputs of column r in registers and walks
// the BC_OPT + 2 lambda input rows they need once, in ascending order, eight
// loads in flight.  Every lane of the wave uses the same tap at the same time,
// so the taps (the full symmetric filter, 2 lambda + 1 per filter) come through
// scalar loads and each row feeds BC_OPT FMAs from registers: 1 + 2 lambda /
// BC_OPT row loads per output, from the L1 and L2, against the tiled kernel's
// 23 LDS reads per 64 FMAs.  Rows whose taps do not cover all BC_OPT outputs
// (the first and last BC_OPT - 1) are unrolled on their own, so only true taps
// are used.  Every output sums its taps in ascending offset, as in
// k_band_tiled: the same bits.  Bound by FP64 FMA issue and the traffic of the
// rows, which add up: 64 columns of 131,072 samples, lambda 32, 65.5 -> 44.2 us
// (FMAs 14, reading and writing the columns once 27), lambda 100 175 -> 78 us; 8
// columns of 2^20 samples, lambda 100, 110 -> 80 us.  8 outputs per thread took
// 48.5 us, 24 and 32 the same as 16 but longer with fewer columns; holding the
// kernel to 8 waves per SIMD spills (62 us).
constexpr int BC_OPT = 16;
constexpr int BC_MIN_R = 8;       // fewer columns: a wave's row loads fall in 16 or more lines
constexpr int BC_MIN_LAMBDA = 8;  // 2 lambda + 1 >= BC_OPT

// row(u) is input row t0 - lam + u of the column; EDGE: outputs from b on are not written.
template <typename T, int R, bool EDGE, typename F>
__device__ __forceinline__ void band_rows(const T *__restrict__ f, int lam, int64_t t0, int64_t b,
                                          int r, const F &row, T *__restrict__ z) {
    constexpr int O = BC_OPT;
    T acc[O];
#pragma unroll
    for (int m = 0; m < O; ++m) acc[m] = 0;
    T w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) w[q] = row(q);
    // rows 0 .. O - 1: outputs m <= u
#pragma unroll
    for (int ub = 0; ub < O; ub += 8) {
        if (ub > 0) {
#pragma unroll
            for (int q = 0; q < 8; ++q) w[q] = row(ub + q);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int m = 0; m < O; ++m)
                if (m <= ub + q) acc[m] += f[ub + q - m] * w[q];
    }
    // rows O .. 2 lam: all outputs (w holds rows u .. u + 7)
    const int last = 2 * lam;
    int u = O;
    for (; u + 7 <= last; u += 8) {
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = row(u + q);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int m = 0; m < O; ++m) acc[m] += f[u + q - m] * w[q];
    }
    for (; u <= last; ++u) {
        const T v = row(u);
#pragma unroll
        for (int m = 0; m < O; ++m) acc[m] += f[u - m] * v;
    }
    // rows 2 lam + 1 .. 2 lam + O - 1: outputs m >= u - 2 lam
    const T *fe = f + last;
#pragma unroll
    for (int db = 1; db < O; db += 8) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (db + q < O) w[q] = row(last + db + q);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int m = 0; m < O; ++m)
                if (m >= db + q) acc[m] += fe[db + q - m] * w[q];
    }
#pragma unroll
    for (int m = 0; m < O; ++m)
        if (!EDGE || t0 + m < b) z[(t0 + m) * R + r] = acc[m];
}

template <typename T, int R>
__global__ void __launch_bounds__(BS) k_band_cols(const int64_t *__restrict__ pref, int n_int,
                                                  const int64_t *__restrict__ istart,
                                                  const int32_t *__restrict__ fid,
                                                  const T *__restrict__ full, int lam,
                                                  int64_t n_tiles, const T *__restrict__ y,
                                                  T *__restrict__ z) {
    constexpr int GW = 64 / R, TL = (BS / R) * BC_OPT;
    // neighbouring tiles share 2 lambda rows: contiguous runs per XCD
    const int64_t bt = xcd_block(blockIdx.x, gridDim.x);
    if (bt >= n_tiles) return;
    int lo = 0, hi = n_int;  // pref[lo] <= bt < pref[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pref[mid] <= bt) lo = mid; else hi = mid;
    }
    const int64_t a = istart[lo], b = istart[lo + 1];
    const T *f = full + (int64_t)fid[lo] * (2 * lam + 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t tw = a + (bt - pref[lo]) * TL + wave * GW * BC_OPT;  // the wave's first output
    if (tw >= b) return;
    const int64_t t0 = tw + lane / R * BC_OPT;
    const int r = lane % R;
    const T *yr = y + r;
    // rows read ahead past the last needed one by at most 8
    if (tw - lam >= a && tw + GW * BC_OPT + lam + 8 <= b)
        band_rows<T, R, false>(f, lam, t0, b, r, [&](int u) { return yr[(t0 - lam + u) * R]; }, z);
    else
        band_rows<T, R, true>(
            f, lam, t0, b, r,
            [&](int u) {  // 0 outside the interval
                const int64_t t = t0 - lam + u;
                const bool in = t >= a && t < b;
                const T v = yr[(in ? t : a) * R];
                return in ? v : (T)0;
            },
            z);
}

// z = N^-1 P x of many columns in one pass: a block gathers the rows of P x that its
// outputs, CB columns of a tile, need into LDS (as k_apply_P does), and walks them from
// there as k_band_cols does.  The tile's halo, 2 lambda rows, is gathered by its
// neighbours too, but P x is neither written nor read back.  The same bits as the two
// launches.  Bound by the gathers, from the L2, and the FMAs of the band.  A of 64
// columns, FP64, P and band apart or in one pass, us: 131,072 samples, lambda 32
// 73 -> 48, lambda 80 103 -> 81; 524,288 299 -> 174; 8 columns of 2^20 samples, lambda
// 32, 80 -> 53.  64-column blocks, whose halo is twice the share, took 56 us where
// 32 take 48.  From halos of 2.5 tiles on the gathers outweigh (FP32, 32 columns of
// 2^20, lambda 120 338 -> 305, 200 494 -> 513).
constexpr int BP_MIN_R = 8;
constexpr int BP_LDS = 80 * 1024;  // two blocks per CU
template <int R> constexpr int bp_cols() { return R < 32 ? R : 32; }
// Row stride in LDS: the rows of two neighbouring threads of a column, BC_OPT apart,
// on different banks.
template <int R> constexpr int bp_stride() { return bp_cols<R>() < 32 ? bp_cols<R>() + 1 : 32; }
template <typename T, int R> size_t bp_lds(int lam) {
    return sizeof(T) * bp_stride<R>() *
           (size_t)((BS / bp_cols<R>()) * BC_OPT + 2 * lam + 8);  // 8 are read ahead
}

template <typename T, int R, int NC>
__global__ void __launch_bounds__(BS) k_band_P(const int64_t *__restrict__ pref, int n_int,
                                               const int64_t *__restrict__ istart,
                                               const int32_t *__restrict__ fid,
                                               const T *__restrict__ full, int lam,
                                               int64_t n_tiles, const int32_t *__restrict__ jpix,
                                               const typename Vec2<T>::type *__restrict__ w,
                                               const double *__restrict__ x, T *__restrict__ z) {
    extern __shared__ char smem[];
    T *const sy = reinterpret_cast<T *>(smem);
    constexpr int CB = bp_cols<R>(), SR = bp_stride<R>(), K = R / CB, TL = (BS / CB) * BC_OPT;
    // the K column groups of a tile are neighbours; pref counts tiles of CB columns
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x), bt = blk / K;
    if (bt >= n_tiles) return;
    const int c0 = (int)(blk % K) * CB;
    int lo = 0, hi = n_int;  // pref[lo] <= bt < pref[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pref[mid] <= bt) lo = mid; else hi = mid;
    }
    const int64_t a = istart[lo], b = istart[lo + 1];
    const int64_t ta = a + (bt - pref[lo]) * TL;  // the tile's first output
    const T *f = full + (int64_t)fid[lo] * (2 * lam + 1);
    {
        // two columns per lane, BP_U steps of the block's rows in flight
        constexpr int LPS = CB / 2, RPB = BS / LPS, BP_U = 4;
        const int sub = threadIdx.x / LPS, r = 2 * (threadIdx.x % LPS);
        const int rows = TL + 2 * lam;
        for (int i = sub; i < rows; i += BP_U * RPB) {
            int32_t j[BP_U];
            typename Vec2<T>::type ww[BP_U];
            bool in[BP_U];
#pragma unroll
            for (int q = 0; q < BP_U; ++q) {
                const int64_t t = ta - lam + i + q * RPB;
                in[q] = t >= a && t < b;
                const int64_t tq = in[q] ? t : a;
                j[q] = jpix[tq];
                if constexpr (NC > 1) ww[q] = w[tq];
            }
            typename Pair<T>::type v[BP_U];
            p_rows<T, R, NC, BP_U>(j, ww, x, c0 + r, v);
#pragma unroll
            for (int q = 0; q < BP_U; ++q) {
                const int row = i + q * RPB;
                if (row >= rows) break;
                if (!in[q]) v[q] = (T)0;
                sy[row * SR + r] = v[q].x;
                sy[row * SR + r + 1] = v[q].y;
            }
        }
    }
    __syncthreads();
    const int m0 = threadIdx.x / CB * BC_OPT, r = threadIdx.x % CB;
    if (ta + m0 >= b) return;
    const T *const yr = sy + m0 * SR + r;
    band_rows<T, R, true>(f, lam, ta + m0, b, c0 + r, [&](int u) { return yr[u * SR]; }, z);
}

// y[t R + r] = mask_t * tod[r * n + t]; flags non-finite data on kept samples.
template <typename T, int R>
__global__ void __launch_bounds__(BS) k_mask(const int32_t *__restrict__ jpix, int64_t n,
                                             const T *__restrict__ tod, T *__restrict__ y,
                                             int *__restrict__ flag) {
    int bad = 0;
    for (int64_t e = (int64_t)blockIdx.x * BS + threadIdx.x; e < n * R;
         e += (int64_t)gridDim.x * BS) {
        const int64_t t = e / R;
        const int r = (int)(e % R);
        T v = tod[(int64_t)r * n + t];
        if (jpix[t] >= 0) {
            bad |= !isfinite(v);
        } else {
            v = (T)0;
        }
        y[e] = v;
    }
    if (bad) atomicOr(flag, 1);
}

int grid_for(int64_t n, int max_blocks = 16384) {
    int64_t g = (n + BS - 1) / BS;
    if (g > max_blocks) g = max_blocks;
    return (int)(g < 1 ? 1 : g);
}

template <typename F> void dispatch_r(int nrhs, F &&f) {
    switch (nrhs) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 8: f(std::integral_constant<int, 8>()); break;
        case 16: f(std::integral_constant<int, 16>()); break;
        case 32: f(std::integral_constant<int, 32>()); break;
        case 64: f(std::integral_constant<int, 64>()); break;
        default: throw Error(MM_E_INVALID, "nrhs must be a power of two <= 64");
    }
}

// f(time-domain type, component count 1 or 2) of an I or QU pointing.
template <typename F> void dispatch_t_nc(const mm_pointing *p, F &&f) {
    auto nc = [&](auto TT) {
        if (p->nc == 1) f(TT, std::integral_constant<int, 1>());
        else if (p->nc == 2) f(TT, std::integral_constant<int, 2>());
        else f(TT, std::integral_constant<int, 3>());
    };
    if (p->prec == MM_F32) nc(0.f);
    else nc(0.0);
}

}  // namespace

PMap p_map_dev(mm_ctx *ctx, const mm_pointing *p, const double *x, char *scratch) {
    const bool f32 = p->prec == MM_F32;
    PMap m{};
    m.w = p->nc == 1 ? nullptr : (f32 ? p->w.ptr : p->psi.ptr);
    if (p->p_j.ptr == nullptr) {
        m.kind = p->nc;
        m.slot = p->j.as<int32_t>();
        m.xm = x;
        return m;
    }
    if (!scratch) {
        ws_alloc(ctx, ctx->xpack, apply_P_scratch_bytes(p, 1));
        scratch = static_cast<char *>(ctx->xpack.ptr);
    }
    const int copies = p->p_copies, grid = grid_for(p->n_obs, 1024);
    const int32_t *slot = p->p_slot.as<int32_t>();
    m.slot = p->p_j.as<int32_t>();
    double *pk = reinterpret_cast<double *>(scratch);
    if (p->nc != 3) {
        m.kind = p->nc;
        m.xm = pk;
        if (p->nc == 1)
            k_pack_map_nc<1><<<grid, BS, 0, ctx->stream>>>(x, p->n_obs, copies, slot, pk);
        else
            k_pack_map_nc<2><<<grid, BS, 0, ctx->stream>>>(x, p->n_obs, copies, slot, pk);
    } else if (f32) {
        m.kind = PK_PACKED;
        m.xq = reinterpret_cast<double2 *>(scratch);
        k_pack_map<<<grid, BS, 0, ctx->stream>>>(x, p->n_obs, copies, slot,
                                                 reinterpret_cast<double2 *>(scratch));
    } else {
        // I of all slots, then (Q, U) of all slots, 16-byte aligned
        m.kind = PK_PACKED;
        const size_t no = (size_t)p->n_obs * copies;
        m.xm = pk;
        double2 *xqu = reinterpret_cast<double2 *>(pk + 2 * ((no + 1) / 2));
        m.xq = xqu;
        k_pack_map_split<<<grid, BS, 0, ctx->stream>>>(x, p->n_obs, copies, slot, pk, xqu);
    }
    MM_HIP(hipGetLastError());
    return m;
}

// planar: several columns one after the other, [R][n], instead of interleaved.
void apply_P_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const double *x, void *y,
                 char *scratch, bool planar) {
    Scope sc(ctx->prof, ctx->stream, "P");
    const int64_t n = p->n_samp;
    if (p->n_obs == 0) {  // no observed pixel: y = 0 (the gathers assume a pixel 0)
        const int64_t ne = n * nrhs;
        if (ne > 0) {
            if (p->prec == MM_F32)
                k_zero<float><<<grid_for(ne), BS, 0, ctx->stream>>>(ne, static_cast<float *>(y));
            else
                k_zero<double><<<grid_for(ne), BS, 0, ctx->stream>>>(ne, static_cast<double *>(y));
            MM_HIP(hipGetLastError());
        }
        return;
    }
    if (nrhs == 1) {
        const PMap m = p_map_dev(ctx, p, x, scratch);
        const unsigned grid = (unsigned)((n + 2 * BS - 1) / (2 * BS));
        auto go = [&](auto TT) {
            using T = decltype(TT);
            dispatch_src<T>(m, [&](auto src) {
                k_apply_P1<T><<<grid, BS, 0, ctx->stream>>>(src, n, static_cast<T *>(y));
            });
        };
        if (p->prec == MM_F32) go(0.f);
        else go(0.0);
        MM_HIP(hipGetLastError());
        return;
    }
    dispatch_r(nrhs, [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        if constexpr (R > 1) {
            constexpr int step = PR_U * 128 / R;  // samples of a wave at a time
            const int64_t per =
                p_wave_samples(n, step, p->p_blocks[log2i(R)], (int64_t)sizeof(double) * p->n() * R);
            const unsigned grid = (unsigned)((n + 4 * per - 1) / (4 * per));
            auto go = [&](auto TT, auto NN) {
                using T = decltype(TT);
                constexpr int NC = decltype(NN)::value;
                k_apply_P<T, R, NC><<<grid, BS, 0, ctx->stream>>>(
                    p->j.as<int32_t>(),
                    NC > 1 ? static_cast<const typename Vec2<T>::type *>(p->w.ptr) : nullptr, n,
                    per, planar ? n : 0, x, static_cast<T *>(y));
            };
            dispatch_t_nc(p, go);
        }
    });
    MM_HIP(hipGetLastError());
}

size_t apply_P_scratch_bytes(const mm_pointing *p, int nrhs) {
    if (nrhs != 1) return 0;
    // I and QU gather from x itself without a grid, else from NC-value copies
    if (p->nc != 3)
        return p->p_j.ptr ? sizeof(double) * (size_t)(p->nc * (int64_t)p->n_obs * p->p_copies) : 0;
    const int copies = p->p_copies > 0 ? p->p_copies : 1;
    return sizeof(double2) * 2 * (size_t)(p->n_obs > 0 ? p->n_obs : 1) * copies;
}

size_t apply_PT_scratch_bytes(const mm_pointing *p, int nrhs) {
    if (nrhs != 1 || !p->sl_perm.ptr || p->n_obs == 0) return 0;
    const int64_t parts = (int64_t)p->sl_S * p->sl_D;
    return parts > 1 ? sizeof(double) * (size_t)(p->n() * parts) : 0;
}

void apply_PT_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const void *z, double *x,
                  char *scratch) {
    Scope sc(ctx->prof, ctx->stream, "PT");
    if (p->n_obs == 0) return;
    if (nrhs == 1 && p->sl_perm.ptr) {
        // lane pixels are virtual ids d n_obs + c (sl_D scan directions), so
        // wave (s, g) writes partial map s D + d; the partials are then
        // added in that fixed order
        const int32_t G = p->sl_G, S = p->sl_S, D = p->sl_D;
        const int64_t n3 = p->n();
        const int32_t parts = S * D;
        double *out = x;
        if (parts > 1) {
            if (!scratch) {
                ws_alloc(ctx, ctx->pt_part, apply_PT_scratch_bytes(p, nrhs));
                scratch = static_cast<char *>(ctx->pt_part.ptr);
            }
            out = reinterpret_cast<double *>(scratch);
        }
        const int32_t nv = D * p->n_obs;
        int64_t nb = ((int64_t)G * S + 3) / 4;
        if (nb >= 64) nb = (nb + 7) & ~(int64_t)7;
        auto go = [&](auto TT, auto NN) {
            using T = decltype(TT);
            k_apply_PT_sl<T, decltype(NN)::value><<<(unsigned)nb, BS, 0, ctx->stream>>>(
                p->sl_base.as<int64_t>(), p->sl_perm.as<int32_t>(),
                p->sl_w.as<typename SlRec<T>::type>(), p->sl_pix.as<int32_t>(), G, S, nv,
                static_cast<const T *>(z), out);
        };
        dispatch_t_nc(p, go);
        if (parts > 1)
            k_pt_sum_parts<<<grid_for(n3, 2048), BS, 0, ctx->stream>>>(out, parts, n3, x);
        MM_HIP(hipGetLastError());
        return;
    }
    const int po = p->pt_order[log2i(nrhs)];
    const bool tiled = p->seg_order.ptr && (nrhs == 1 || p->nc != 3 || po != 0);
    const int32_t *order = tiled ? p->seg_order.as<int32_t>() : nullptr;
    const PtForm form = pt_form(p->n_obs, p->n_valid, nrhs, ctx->n_cu);
    int64_t nb = form == PtForm::BLOCK ? p->n_obs : (p->n_obs + 3) / 4;
    if (nb >= 64) nb = (nb + 7) & ~(int64_t)7;
    dispatch_r(nrhs, [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        auto go = [&](auto TT, auto NN) {
            using T = decltype(TT);
            constexpr int NC = decltype(NN)::value;
            const auto *ws =
                NC > 1 ? static_cast<const typename Vec2<T>::type *>(p->ws.ptr) : nullptr;
            auto run = [&](auto k) {
                k<<<(unsigned)nb, BS, 0, ctx->stream>>>(p->off.as<int32_t>(),
                                                        p->perm.as<int32_t>(), ws, p->n_obs,
                                                        order, static_cast<const T *>(z), x);
            };
            if constexpr (R >= PT_MIN_COLS) {
                if (form == PtForm::BLOCK) return run(k_apply_PT_cols<T, R, NC, 4>);
                if (form == PtForm::COLUMNS) return run(k_apply_PT_cols<T, R, NC, 1>);
            }
            run(k_apply_PT<T, R, NC>);
        };
        dispatch_t_nc(p, go);
    });
    MM_HIP(hipGetLastError());
}

void noise_fft_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z);
void noise_fft_planar_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z);

// Whether R columns take the register kernel without LDS: from 8 columns on,
// where a row load of a wave falls in at most 8 runs of cache lines, and from
// 2^21 values on, 8 waves per CU: with fewer its longer threads (16 outputs
// each, against 8) leave the chip idle (us, register / tiled kernel, 8 columns,
// lambda 64: 2^19 values 12.8 / 10.1, 2^20 14.0 / 15.7, 2^21 19.9 / 26.4; 16
// columns: 12.4 / 8.8, 13.6 / 11.4, 20.8 / 20.4, 2^22 32.5 / 34.7; 64 columns:
// 14.1 / 11.6, 15.3 / 18.7, 19.6 / 33.9).
static bool band_by_rows(int nrhs, int lam, int64_t n_samp) {
    return nrhs >= BC_MIN_R && lam >= BC_MIN_LAMBDA && n_samp * nrhs >= ((int64_t)1 << 21);
}

// The same for N^-1 alone.  8 columns in FP64 with short filters on long streams are
// bound by the rows' traffic, which the tiled kernel's LDS saves (us, register / tiled,
// 2^25 values: lambda 8 114 / 106, 16 135 / 130, 24 156 / 148, 32 175 / 177; 24M values,
// lambda 16 103 / 91; 2^23, lambda 16 34 / 37).  16 and 32 columns in FP32 with longer
// filters fill the chip sooner in the tiled kernel (2^21 values x 32 columns, lambda 24 9.0 / 8.6, 48
// 13.0 / 10.9, 80 18.3 / 14.9; 2^23 values 34 / 36, 51 / 48 at 48 and 80).  With P inside, the
// rows win there too.
static bool band_rows_alone(int nrhs, int lam, int64_t n_samp, mm_precision prec) {
    if (!band_by_rows(nrhs, lam, n_samp)) return false;
    if (prec == MM_F64) return !(nrhs == 8 && lam < 32 && n_samp >= ((int64_t)1 << 21));
    return !((nrhs == 16 || nrhs == 32) && lam >= 32 && n_samp * nrhs < ((int64_t)1 << 22));
}

// Tile length of N^-1 by the direct band for R columns.
static int band_rows_tile(int nrhs) { return (BS / nrhs) * BC_OPT; }
static int band_tile_len(int nrhs, bool small, int lam, int64_t n_samp, mm_precision prec) {
    if (band_rows_alone(nrhs, lam, n_samp, prec)) return band_rows_tile(nrhs);
    return nrhs == 1 && small ? BAND_SMALL_NT * BAND_SMALL_OPT : (BS / nrhs) * BT_OPT;
}

// Taps per LDS chunk of the direct band: taps + window rows of R values fit
// in BT_LDS bytes; a multiple of BT_OPT, at most the padded filter length.
static int band_chunk(int lam, int R, mm_precision prec, bool small, int64_t n_samp) {
    const size_t te = prec == MM_F32 ? sizeof(float) : sizeof(double);
    const int tl = band_tile_len(R, small, lam, n_samp, prec);
    const int nf_pad = (2 * lam + 1 + BT_OPT - 1) / BT_OPT * BT_OPT;
    int cl = (int)(((int64_t)(BT_LDS / te) - (int64_t)(tl - 1) * R) / (R + 1));
    cl = cl / BT_OPT * BT_OPT;
    return cl < nf_pad ? cl : nf_pad;
}

size_t noise_scratch_bytes(const mm_noise *nz, int nrhs) {
    return nz->method == MM_NOISE_POLY ? polyfilter_scratch_bytes(nz, nrhs) : 0;
}

// Tile counts for every column count are built with the noise handle, so an apply
// never modifies it (handles may be shared across contexts): of N^-1 alone, then of the
// rows with P inside.
constexpr int BAND_TABLES = 14;
static const int64_t *band_tiles(const mm_noise *nz, int nrhs, int64_t *n_tiles,
                                 bool with_P = false) {
    const size_t li = (size_t)(log2i(nrhs) + (with_P ? 7 : 0)) * (nz->n_int + 1);
    *n_tiles = nz->h_tile_pref[li + nz->n_int];
    return nz->tile_pref.as<int64_t>() + li;
}

static int band_chunk_used(const mm_noise *nz, int nrhs) {
    const int tuned = nz->band_cl[log2i(nrhs)];
    return tuned > 0 ? tuned
                     : band_chunk(nz->half_bw, nrhs, nz->prec, nz->band_small, nz->n_samp);
}

template <typename T, int R, typename Rows>
static void band_tiled_launch(mm_ctx *ctx, const mm_noise *nz, const Rows &rows, T *z, int cl) {
    const int lam = nz->half_bw;
    const int tl = band_tile_len(R, nz->band_small, lam, nz->n_samp, nz->prec);
    int64_t n_tiles;
    const int64_t *pref = band_tiles(nz, R, &n_tiles);
    const size_t sm = sizeof(T) * ((size_t)cl + (size_t)(tl + cl - 1) * R);
    auto run = [&](auto k, int nt) {
        k<<<(unsigned)n_tiles, nt, sm, ctx->stream>>>(pref, nz->n_int, nz->istart.as<int64_t>(),
                                                      nz->fid.as<int32_t>(), nz->band.as<T>(),
                                                      lam, cl, rows, z);
    };
    if constexpr (R == 1)
        if (nz->band_small)  // short single streams
            return run(k_band_tiled<T, R, BAND_SMALL_NT, BAND_SMALL_OPT, Rows>, BAND_SMALL_NT);
    run(k_band_tiled<T, R, BS, BT_OPT, Rows>, BS);
}

// z = N^-1 P x in one launch; false where that does not apply.  One column: all taps in
// one LDS chunk.  More: the direct band runs by rows, two blocks' rows fit in a CU's LDS
// and the halo is at most 2.5 tiles.
static bool band_P_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, int nrhs,
                       const double *x, void *z, char *scratch) {
    const int lam = nz->half_bw;
    if (nz->method != MM_NOISE_DIRECT || p->n_obs == 0) return false;
    if (nrhs == 1) {
        // the window is gathered once, for all taps: whatever chunk N^-1 alone is tuned to
        const int cl = band_chunk(lam, 1, nz->prec, nz->band_small, nz->n_samp);
        if (cl < 2 * lam + 1) return false;  // several windows per tile
        Scope sc(ctx->prof, ctx->stream, "Ninv_band");
        const PMap m = p_map_dev(ctx, p, x, scratch);
        auto go = [&](auto TT) {
            using T = decltype(TT);
            dispatch_src<T>(m, [&](auto src) {
                band_tiled_launch<T, 1>(ctx, nz, PRows<T, decltype(src)>{src},
                                        static_cast<T *>(z), cl);
            });
        };
        if (nz->prec == MM_F32) go(0.f);
        else go(0.0);
        MM_HIP(hipGetLastError());
        return true;
    }
    bool done = false;
    dispatch_r(nrhs, [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        if constexpr (R >= BP_MIN_R) {
            auto go = [&](auto TT, auto NN) {
                using T = decltype(TT);
                constexpr int NC = decltype(NN)::value, K = R / bp_cols<R>();
                constexpr int CB = bp_cols<R>();
                const size_t lds = bp_lds<T, R>(lam);
                if (lds > BP_LDS || 4 * lam > 5 * (BS / CB) * BC_OPT ||
                    !band_by_rows(CB, lam, nz->n_samp))
                    return;
                Scope sc(ctx->prof, ctx->stream, "Ninv_band");
                int64_t n_tiles;
                const int64_t *pref = band_tiles(nz, CB, &n_tiles, true);
                k_band_P<T, R, NC><<<(unsigned)((n_tiles * K + 7) / 8 * 8), BS, lds,
                                     ctx->stream>>>(
                    pref, nz->n_int, nz->istart.as<int64_t>(),
                    nz->fid.as<int32_t>(), nz->band_full.as<T>(), lam, n_tiles,
                    p->j.as<int32_t>(),
                    NC > 1 ? static_cast<const typename Vec2<T>::type *>(p->w.ptr) : nullptr, x,
                    static_cast<T *>(z));
                done = true;
            };
            dispatch_t_nc(p, go);
        }
    });
    MM_HIP(hipGetLastError());
    return done;
}

void noise_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z) {
    if (nz->method == MM_NOISE_FFT) {
        noise_fft_apply_dev(ctx, nz, nrhs, y, z);
        return;
    }
    if (nz->method == MM_NOISE_POLY) {
        polyfilter_apply_dev(ctx, nz, nrhs, y, z);
        return;
    }
    Scope sc(ctx->prof, ctx->stream, "Ninv_band");
    const int lam = nz->half_bw;
    if (band_rows_alone(nrhs, lam, nz->n_samp, nz->prec)) {
        dispatch_r(nrhs, [&](auto RR) {
            constexpr int R = decltype(RR)::value;
            if constexpr (R >= BC_MIN_R) {
                int64_t n_tiles;
                const int64_t *pref = band_tiles(nz, R, &n_tiles);
                const unsigned grid = (unsigned)((n_tiles + 7) / 8 * 8);
                auto go = [&](auto TT) {
                    using T = decltype(TT);
                    k_band_cols<T, R><<<grid, BS, 0, ctx->stream>>>(
                        pref, nz->n_int, nz->istart.as<int64_t>(), nz->fid.as<int32_t>(),
                        nz->band_full.as<T>(), lam, n_tiles, static_cast<const T *>(y),
                        static_cast<T *>(z));
                };
                if (nz->prec == MM_F32) go(0.f);
                else go(0.0);
            }
        });
        MM_HIP(hipGetLastError());
        return;
    }
    dispatch_r(nrhs, [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        auto go = [&](auto TT) {
            using T = decltype(TT);
            band_tiled_launch<T, R>(ctx, nz, TodRows<T>{static_cast<const T *>(y)},
                                    static_cast<T *>(z), band_chunk_used(nz, R));
        };
        if (nz->prec == MM_F32) go(0.f);
        else go(0.0);
    });
    MM_HIP(hipGetLastError());
}

// I and QU: P's map copies and P^T's partial maps lie in whichever TOD vector is
// not in use then; both fit there (checked when they are laid out).
size_t apply_A_scratch_bytes(const mm_pointing *p, const mm_noise *nz, int nrhs) {
    size_t b = noise_scratch_bytes(nz, nrhs);
    if (p->nc == 3)
        b = std::max(b, std::max(apply_P_scratch_bytes(p, nrhs), apply_PT_scratch_bytes(p, nrhs)));
    return b;
}

void apply_A_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, int nrhs,
                 const double *x, double *y, void *ta, void *tb, char *scratch) {
    const bool in_tod = scratch && p->nc != 3;
    const void *z = tb;
    if (nz->method == MM_NOISE_POLY) {
        // the filter's first pass reads the copies while it writes tb
        z = polyfilter_apply_P_dev(ctx, p, nz, nrhs, x, ta, tb, scratch,
                                   in_tod ? static_cast<char *>(ta) : scratch);
    } else if (!band_P_dev(ctx, p, nz, nrhs, x, tb,
                           in_tod ? static_cast<char *>(ta) : scratch)) {
        // up to 16 columns, A's own TOD between P and the FFT is planar: the FFT then
        // reads runs of 16 bytes per lane, which saves more than P's shorter runs cost.
        // Interleaved and planar, us (FP64): 8.4M samples x 4 columns 491 and 477, x 8
        // 974 and 848; 1M x 8 118 and 107, x 16 248 and 218, x 32 469 and 657
        const bool planar = nrhs > 1 && nrhs <= P_PLANAR_COLS && nz->method == MM_NOISE_FFT;
        apply_P_dev(ctx, p, nrhs, x, ta, in_tod ? static_cast<char *>(tb) : scratch, planar);
        if (planar) noise_fft_planar_dev(ctx, nz, nrhs, ta, tb);
        else noise_apply_dev(ctx, nz, nrhs, ta, tb);
    }
    apply_PT_dev(ctx, p, nrhs, z, y,
                 in_tod ? static_cast<char *>(z == tb ? ta : tb) : scratch);
}

void pair_sum_diff_dev(mm_ctx *ctx, int64_t n, mm_precision prec, const void *a, const void *b,
                       void *plus, void *minus) {
    const int grid = grid_for(n);
    if (prec == MM_F32)
        k_sum_diff<float><<<grid, BS, 0, ctx->stream>>>(
            n, static_cast<const float *>(a), static_cast<const float *>(b),
            static_cast<float *>(plus), static_cast<float *>(minus));
    else
        k_sum_diff<double><<<grid, BS, 0, ctx->stream>>>(
            n, static_cast<const double *>(a), static_cast<const double *>(b),
            static_cast<double *>(plus), static_cast<double *>(minus));
    MM_HIP(hipGetLastError());
}

void mask_tod_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const void *tod, void *y,
                  int *flag) {
    const int64_t n = p->n_samp;
    dispatch_r(nrhs, [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        const int grid = grid_for(n * R);
        if (p->prec == MM_F32)
            k_mask<float, R><<<grid, BS, 0, ctx->stream>>>(p->j.as<int32_t>(), n,
                                                           static_cast<const float *>(tod),
                                                           static_cast<float *>(y), flag);
        else
            k_mask<double, R><<<grid, BS, 0, ctx->stream>>>(p->j.as<int32_t>(), n,
                                                            static_cast<const double *>(tod),
                                                            static_cast<double *>(y), flag);
    });
    MM_HIP(hipGetLastError());
}

}  // namespace mm

namespace mm {

// Tile counts of the direct band for every column count R = 2^li (tile lengths above, of
// N^-1 alone and with P inside): pref[li][i] = tiles in the intervals before i; and the
// full symmetric filters f[d] = c_|d - lambda| of the register kernel where 64
// columns would take it.
void build_band_tiles(mm_ctx *ctx, mm_noise *nz) {
    std::vector<char> full;  // in use until the copies are done
    if (band_by_rows(64, nz->half_bw, nz->n_samp)) {
        const size_t lam = (size_t)nz->half_bw, nf = 2 * lam + 1, n = nf * nz->n_filters;
        auto fill = [&](auto TT) {
            using T = decltype(TT);
            full.resize(sizeof(T) * n);
            T *out = reinterpret_cast<T *>(full.data());
            for (size_t f = 0; f < (size_t)nz->n_filters; ++f)
                for (size_t d = 0; d < nf; ++d)
                    out[f * nf + d] = (T)nz->h_band[f * (lam + 1) + (d < lam ? lam - d : d - lam)];
            nz->band_full.alloc(sizeof(T) * n);
            MM_HIP(hipMemcpyAsync(nz->band_full.ptr, out, sizeof(T) * n, hipMemcpyHostToDevice,
                                  ctx->stream));
        };
        if (nz->prec == MM_F32) fill(0.f);
        else fill(0.0);
    }
    const size_t np = (size_t)nz->n_int + 1;
    nz->h_tile_pref.assign(BAND_TABLES * np, 0);
    for (int li = 0; li < BAND_TABLES; ++li) {
        const int64_t tl = li < 7 ? band_tile_len(1 << li, nz->band_small, nz->half_bw,
                                                  nz->n_samp, nz->prec)
                                  : band_rows_tile(1 << (li - 7));
        int64_t *pr = nz->h_tile_pref.data() + li * np;
        for (int i = 0; i < nz->n_int; ++i)
            pr[i + 1] = pr[i] + (nz->h_istart[i + 1] - nz->h_istart[i] + tl - 1) / tl;
    }
    nz->tile_pref.alloc(sizeof(int64_t) * nz->h_tile_pref.size());
    MM_HIP(hipMemcpyAsync(nz->tile_pref.ptr, nz->h_tile_pref.data(),
                          sizeof(int64_t) * nz->h_tile_pref.size(), hipMemcpyHostToDevice,
                          ctx->stream));
    MM_HIP(hipStreamSynchronize(ctx->stream));
}

// Measure candidates for each stage with HIP events and keep the fastest:
//   stage 0, P of several columns: the grid size, i.e. the samples per wave (the P of
//     one column has no such choice: it is timed once);
//   stage 1, direct band: the taps per LDS chunk (smaller chunks need less
//     LDS per block, so more blocks share a CU); the kernel by rows has none and is
//     timed once, and so is untouched an A that forms P inside the band;
//   stage 2, P^T with several columns: visiting the pixels in the tiled
//     order or ascending;
//   stage 3 (flag MM_TUNE_FFT_BLOCK only), FFT: the overlap-save block length.
// Stages 0-2 change speed only: every output sums its terms in a fixed order
// that no candidate changes, so results are bitwise the same.  Stage 3 moves
// results at the rounding level.  report: (stage, candidate, ms) triples.
void autotune(mm_ctx *ctx, mm_pointing *p, mm_noise *nz, int nrhs, int flags, double *report,
              int *n_report, int max_report) {
    const int li = log2i(nrhs);
    const size_t te = p->prec == MM_F32 ? sizeof(float) : sizeof(double);
    DBuf x, y, z;
    x.alloc(sizeof(double) * (size_t)p->n() * nrhs);
    y.alloc(te * (size_t)p->n_samp * nrhs);
    z.alloc(te * (size_t)p->n_samp * nrhs);
    MM_HIP(hipMemsetAsync(x.ptr, 0, x.bytes, ctx->stream));
    MM_HIP(hipMemsetAsync(y.ptr, 0, y.bytes, ctx->stream));
    hipEvent_t e0, e1;
    MM_HIP(hipEventCreate(&e0));
    MM_HIP(hipEventCreate(&e1));
    int nr = 0;
    auto time_it = [&](const std::function<void()> &f) {
        f();
        MM_HIP(hipEventRecord(e0, ctx->stream));
        for (int i = 0; i < 5; ++i) f();
        MM_HIP(hipEventRecord(e1, ctx->stream));
        MM_HIP(hipEventSynchronize(e1));
        float ms = 0;
        MM_HIP(hipEventElapsedTime(&ms, e0, e1));
        return ms / 5.0;
    };
    auto note = [&](int stage, double cand, double ms) {
        if (report && nr < max_report) {
            report[3 * nr] = stage;
            report[3 * nr + 1] = cand;
            report[3 * nr + 2] = ms;
        }
        ++nr;
    };
    const bool prof = ctx->prof.on;
    ctx->prof.on = false;
    try {
        // stage 0: P grid size
        {
            double best = 1e30;
            int best_g = 0;
            for (int mult : {0, 2, 4, 8, 16, 32}) {  // 0: the default
                if (nrhs == 1 && mult > 0) break;
                const int g = ctx->n_cu * mult;
                p->p_blocks[li] = g;
                const double ms =
                    time_it([&]() { apply_P_dev(ctx, p, nrhs, x.as<double>(), y.ptr); });
                note(0, g, ms);
                if (ms < best) { best = ms; best_g = g; }
            }
            p->p_blocks[li] = best_g;
        }
        // stage 1: taps per LDS chunk of the direct band
        if (nz->method == MM_NOISE_DIRECT) {
            const int def = band_chunk(nz->half_bw, nrhs, nz->prec, nz->band_small, nz->n_samp);
            double best = 1e30;
            int best_c = 0;
            const bool rows = band_rows_alone(nrhs, nz->half_bw, nz->n_samp, nz->prec);
            for (int div : {1, 2, 4, 8}) {
                const int c = def / div / BT_OPT * BT_OPT;
                if (c < BT_OPT || (div > 1 && (c == def || rows))) continue;
                nz->band_cl[li] = c;
                const double ms = time_it([&]() { noise_apply_dev(ctx, nz, nrhs, y.ptr, z.ptr); });
                note(1, c, ms);
                if (ms < best) { best = ms; best_c = c; }
            }
            nz->band_cl[li] = best_c == def ? 0 : best_c;
        }
        // stage 2: visiting order of the one-wave-per-pixel P^T
        if (nrhs > 1 && p->seg_order.ptr) {
            double best = 1e30;
            int best_o = -1;
            for (int o : {1, 0}) {
                p->pt_order[li] = o;
                const double ms = time_it([&]() { apply_PT_dev(ctx, p, nrhs, z.ptr, x.as<double>()); });
                note(2, o, ms);
                if (ms < best) { best = ms; best_o = o; }
            }
            p->pt_order[li] = best_o;
        }
        // stage 3: FFT block length (results move at the rounding level)
        if ((flags & MM_TUNE_FFT_BLOCK) && nz->method == MM_NOISE_FFT) {
            // the state as it is first, then the lengths that it does not run already;
            // the state stays, a pick at build as such, unless one of them is faster
            const int run = nz->fft.n, keep = nz->fft_auto ? 0 : nz->fft_n;
            auto prep = [&](int n) {
                MM_HIP(hipStreamSynchronize(ctx->stream));
                noise_fft_prepare(ctx, nz, n);
            };
            auto time_apply = [&]() {
                return time_it([&]() { noise_apply_dev(ctx, nz, nrhs, y.ptr, z.ptr); });
            };
            const double now = time_apply();
            double best = now;
            int best_n = keep, is = keep;
            for (int n_fft : {16384, 32768}) {
                if (n_fft == 16384 && nz->half_bw > 6144) continue;
                double ms = now;
                if (n_fft != run) {
                    prep(n_fft);
                    is = n_fft;
                    ms = time_apply();
                }
                note(3, n_fft, ms);
                if (ms < best) { best = ms; best_n = n_fft; }
            }
            if (is != best_n) prep(best_n);
        }
    } catch (...) {
        ctx->prof.on = prof;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        throw;
    }
    MM_HIP(hipStreamSynchronize(ctx->stream));
    ctx->prof.on = prof;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (n_report) *n_report = nr < max_report ? nr : max_report;
}

}  // namespace mm

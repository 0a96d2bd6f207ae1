// Device helpers shared by the FFT kernels of N^-1: 64th roots of unity and
// in-register DFTs of 4, 8, 16 and 32 points.
#pragma once

#include "mm_internal.h"

namespace mm {
namespace fft {

// cos(2 pi m / 64)
__device__ constexpr double C64[64] = {
    1.0, 0.9951847266721969, 0.9807852804032304, 0.9569403357322088,
    0.9238795325112867, 0.881921264348355, 0.8314696123025452, 0.773010453362737,
    0.7071067811865476, 0.6343932841636455, 0.5555702330196022, 0.47139673682599764,
    0.3826834323650898, 0.2902846772544624, 0.19509032201612828, 0.0980171403295606,
    0.0, -0.0980171403295606, -0.19509032201612828, -0.2902846772544624,
    -0.3826834323650898, -0.47139673682599764, -0.5555702330196022, -0.6343932841636455,
    -0.7071067811865476, -0.773010453362737, -0.8314696123025452, -0.881921264348355,
    -0.9238795325112867, -0.9569403357322088, -0.9807852804032304, -0.9951847266721969,
    -1.0, -0.9951847266721969, -0.9807852804032304, -0.9569403357322088,
    -0.9238795325112867, -0.881921264348355, -0.8314696123025452, -0.773010453362737,
    -0.7071067811865476, -0.6343932841636455, -0.5555702330196022, -0.47139673682599764,
    -0.3826834323650898, -0.2902846772544624, -0.19509032201612828, -0.0980171403295606,
    0.0, 0.0980171403295606, 0.19509032201612828, 0.2902846772544624,
    0.3826834323650898, 0.47139673682599764, 0.5555702330196022, 0.6343932841636455,
    0.7071067811865476, 0.773010453362737, 0.8314696123025452, 0.881921264348355,
    0.9238795325112867, 0.9569403357322088, 0.9807852804032304, 0.9951847266721969};
__device__ constexpr double cos64(int m) { return C64[m & 63]; }
__device__ constexpr double sin64(int m) { return C64[(m + 48) & 63]; }  // cos(x - pi/2)

// (r, i) *= e^(DIR 2 pi i m / 32), without the products by 0 and 1.
template <typename T, int DIR>
__device__ __forceinline__ void mul_w32(T &r, T &i, int m) {
    if (m == 0) return;
    if (m == 8) {
        const T t = r;
        r = DIR * -i;
        i = DIR * t;
        return;
    }
    const T wr = (T)cos64(2 * m), wi = (T)(DIR * sin64(2 * m));
    const T xr = r, xi = i;
    r = wr * xr - wi * xi;
    i = wr * xi + wi * xr;
}

// 4-point DFT in place, DIR = -1 forward (W4 = -i), +1 inverse.
template <typename T, int DIR>
__device__ __forceinline__ void dft4(T &r0, T &i0, T &r1, T &i1, T &r2, T &i2, T &r3, T &i3) {
    const T ar = r0 + r2, ai = i0 + i2, br = r0 - r2, bi = i0 - i2;
    const T cr = r1 + r3, ci = i1 + i3, dr = r1 - r3, di = i1 - i3;
    // (DIR i) (dr + i di) = DIR (-di + i dr)
    const T er = DIR * -di, ei = DIR * dr;
    r0 = ar + cr; i0 = ai + ci;
    r2 = ar - cr; i2 = ai - ci;
    r1 = br + er; i1 = bi + ei;
    r3 = br - er; i3 = bi - ei;
}

// 8-point DFT of elements B .. B + 7 in place, natural order out: 4-point
// DFTs of the even and the odd elements, then radix 2.
template <typename T, int DIR, int B, int N>
__device__ __forceinline__ void dft8_at(T (&re)[N], T (&im)[N]) {
    dft4<T, DIR>(re[B], im[B], re[B + 2], im[B + 2], re[B + 4], im[B + 4], re[B + 6], im[B + 6]);
    dft4<T, DIR>(re[B + 1], im[B + 1], re[B + 3], im[B + 3], re[B + 5], im[B + 5], re[B + 7],
                 im[B + 7]);
    T er[4], ei[4], dr[4], di[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        er[k] = re[B + 2 * k];
        ei[k] = im[B + 2 * k];
        dr[k] = re[B + 2 * k + 1];
        di[k] = im[B + 2 * k + 1];
        mul_w32<T, DIR>(dr[k], di[k], 4 * k);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        re[B + k] = er[k] + dr[k];
        im[B + k] = ei[k] + di[k];
        re[B + k + 4] = er[k] - dr[k];
        im[B + k + 4] = ei[k] - di[k];
    }
}

// 16-point DFT of elements B .. B + 15 in place, natural order out: 4 x 4,
// n = n1 + 4 n2, k = 4 k1 + k2.  Radix 4 over n2, twiddle W16^(n1 k2), radix
// 4 over n1; X[4 k1 + k2] lands in slot k1 + 4 k2 and is renamed.
template <typename T, int DIR, int B, int N>
__device__ __forceinline__ void dft16_at(T (&re)[N], T (&im)[N]) {
#pragma unroll
    for (int n1 = 0; n1 < 4; ++n1)
        dft4<T, DIR>(re[B + n1], im[B + n1], re[B + n1 + 4], im[B + n1 + 4], re[B + n1 + 8],
                     im[B + n1 + 8], re[B + n1 + 12], im[B + n1 + 12]);
#pragma unroll
    for (int n1 = 1; n1 < 4; ++n1)
#pragma unroll
        for (int k2 = 1; k2 < 4; ++k2)
            mul_w32<T, DIR>(re[B + n1 + 4 * k2], im[B + n1 + 4 * k2], 2 * n1 * k2);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2)
        dft4<T, DIR>(re[B + 4 * k2], im[B + 4 * k2], re[B + 4 * k2 + 1], im[B + 4 * k2 + 1],
                     re[B + 4 * k2 + 2], im[B + 4 * k2 + 2], re[B + 4 * k2 + 3],
                     im[B + 4 * k2 + 3]);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = a + 1; b < 4; ++b) {
            T t = re[B + a + 4 * b]; re[B + a + 4 * b] = re[B + b + 4 * a]; re[B + b + 4 * a] = t;
            t = im[B + a + 4 * b]; im[B + a + 4 * b] = im[B + b + 4 * a]; im[B + b + 4 * a] = t;
        }
}

// 32-point DFT as 4 x 8: n = n1 + 8 n2, k = k2 + 4 k1.  Radix 4 over n2,
// twiddle W32^(n1 k2), radix 8 over n1.  X[k] is left in slot out32(k).
__device__ constexpr int out32(int k) { return (k >> 2) + 8 * (k & 3); }
template <typename T, int DIR>
__device__ __forceinline__ void dft32(T (&re)[32], T (&im)[32]) {
#pragma unroll
    for (int n1 = 0; n1 < 8; ++n1)
        dft4<T, DIR>(re[n1], im[n1], re[n1 + 8], im[n1 + 8], re[n1 + 16], im[n1 + 16],
                     re[n1 + 24], im[n1 + 24]);
#pragma unroll
    for (int n1 = 1; n1 < 8; ++n1)
#pragma unroll
        for (int k2 = 1; k2 < 4; ++k2)
            mul_w32<T, DIR>(re[n1 + 8 * k2], im[n1 + 8 * k2], n1 * k2);
    dft8_at<T, DIR, 0>(re, im);
    dft8_at<T, DIR, 8>(re, im);
    dft8_at<T, DIR, 16>(re, im);
    dft8_at<T, DIR, 24>(re, im);
}

}  // namespace fft
}  // namespace mm

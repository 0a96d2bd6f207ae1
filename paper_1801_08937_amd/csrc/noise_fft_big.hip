// N^-1 by FFT with register-resident overlap-save blocks of N = 2 NC real
// samples, packed as NC complex points (the packed-real scheme of
// noise_fft.hip), V = N - 2 lambda valid outputs.
//
// A block has TH = NC / X threads of X complex values each and a transform is
// NC = X x X x L:
//   pass 1  thread j holds x[j + TH r], r < X: DFT over r, giving k1, times
//           W_NC^(j k1);
//   pass 2  per k1 a TH-point transform on L lanes of one wave: lane l holds
//           j = l + L q, q < X; DFT over q, giving k2a, times W_TH^(l k2a);
//   pass 3  L-point DFTs over l, giving k2b.  L <= X: lane l takes k2a = l + L p,
//           p < X / L, for all values of l, and register p L + k2b then holds
//           X[k1 + X (k2a + X k2b)].  L = 2 X: two lanes share each k2a
//           (dft_lanes); register i of lane k2a + X h holds k2b = 2 i + h.
// and the inverse transform runs the passes backwards.  Only the exchange
// between passes 1 and 2 crosses waves: it goes through LDS one component at
// a time, with three barriers.  A wave owns the values k1 of a contiguous
// stretch of LDS rows, so the exchange between passes 2 and 3 and the spectrum
// step stay inside the wave's own rows and need no barrier: 6 barriers per
// block, and the waves of a block drift apart, so that one wave's LDS accesses
// overlap another's arithmetic.
//
// The spectrum step pairs Z_k with Z_{NC-k}.  A wave's k1 come as pairs (a,
// X - a) (wave 0 has 0 and X / 2, each its own partner), so the partner of
// (k1, lane l, register i) is (X - k1, lane L-1-l, register X-1-i) of the same
// wave; for k1 = 0 it is lane L-l, and lane 0 there pairs its own registers.
//
// Three geometries (X, L), and the bandwidths they serve:
//   Short (16, 16): NC =  4,096, 256 threads, FP64 four blocks per CU; 3,072;
//   Mid   (16, 32): NC =  8,192, 512 threads, two per CU;            6,144;
//   Big   (32, 16): NC = 16,384, 512 threads, one per CU;           12,288.
// 16 points are 64 VGPRs of FP64 data, so that four waves share a SIMD; with 32
// (Big) two do.
//
// What bounds it.  Short blocks, 2^26 samples, FP64, lambda 200: memory (238 us,
// 4.5 TB/s of samples read and written); at lambda 2,048, and Mid ones, VALU
// issue (70 % of the cycles at lambda 6,000; LDS 53 %).  Big blocks: one per
// CU, whose waves start in step, so that loads, VALU (42 %) and LDS (27 %) take
// turns; without global traffic they take 0.55 ms of 0.73 ms at 2^27 samples,
// lambda 4,096, the loads and stores alone 0.40 ms.
// Measured, before and after:
//   Big against 1,024 threads of 16 points (radices 16 x 16 x 16 x 4, three
//     exchanges across the block per direction, 25 barriers), 2^27 samples:
//     FP64 0.910 -> 0.738 ms, FP32 0.611 -> 0.368 ms;
//   Mid against 256 threads of 32 points (32 x 32 x 8), FP64: 2^26 samples,
//     lambda 2,048 363 -> 338 us, 2^20 samples 18.8 -> 15.9 us;
//   Short against that, lambda 1,024: 2^26 samples 329 -> 273 us, 2^20 samples
//     18.8 -> 11.4 us.
// Big blocks of 1,024 threads with 16 points (16 x 16 x 64, four lanes per
// transform of pass 3, one row per wave and so two more barriers) took 748 us
// where 32 points take 728 (FP32 448 against 382).
#include <cmath>
#include <vector>

#include "fft_common.h"
#include "xcd.h"

namespace mm {
namespace {

using fft::dft16_at;
using fft::dft32;
using fft::mul_w32;

// Transform geometry (see the top of the file).
template <int X_, int L_> struct Geo {
    static constexpr int X = X_;                // points per thread (radix of passes 1 and 2)
    static constexpr int L = L_;                // lanes per sub-transform
    static constexpr int NC = X * X * L;        // complex points
    static constexpr int TH = X * L;            // threads; points per sub-transform
    static constexpr bool SPLIT = L > X;        // two lanes share a transform of pass 3
    static constexpr int W = 64 / L;            // sub-transforms (rows) per wave
    static constexpr int LX = L < X ? L : X;
    // LDS row of one k1: holds TH values (exchange of passes 1 and 2), or X
    // groups of L values spaced Q apart (passes 2 and 3).  Q and RS put the lanes
    // of every access on distinct bank pairs (RS = L mod 32); with two lanes per
    // transform, the pairs of neighbours that 16 lanes load, 34 apart.
    static constexpr int Q = SPLIT ? L + 2 : L + 1;
    static constexpr int RS = X * Q + (X == 32 ? L : 0);
    static_assert((X == 32 && L == 16) || (X == 16 && (L == 16 || L == 32)), "");
    static_assert(W * RS >= X * 64, "a wave's rows hold its half spectrum, two components");
};
using Big = Geo<32, 16>;
using Mid = Geo<16, 32>;
using Short = Geo<16, 16>;
constexpr int BIG_MAX_LAMBDA = 12288;   // 32,768-sample blocks: V = N - 2 lambda >= 8,192
constexpr int MID_MAX_LAMBDA = 6144;    // 16,384-sample blocks: V >= 4,096
constexpr int SHORT_MAX_LAMBDA = 3072;  // 8,192-sample blocks: V >= 2,048

// Slot of output k of the DFT of X points.
template <int X> __host__ __device__ constexpr int outx(int k) {
    return X == 32 ? fft::out32(k) : k;
}
template <typename T, int DIR> __device__ __forceinline__ void dftx(T (&re)[32], T (&im)[32]) {
    dft32<T, DIR>(re, im);
}
template <typename T, int DIR> __device__ __forceinline__ void dftx(T (&re)[16], T (&im)[16]) {
    dft16_at<T, DIR, 0>(re, im);
}

// Rows are numbered wave by wave, a wave's first W / 2 rows holding k1 = a and
// the next their partners X - a (X / 2 for a = 0).
template <typename G> __host__ __device__ constexpr int row_k1(int row) {
    constexpr int H = G::W / 2;
    const int w = row / G::W, s = row % G::W, a = H * w + s % H;
    return s < H ? a : (a == 0 ? G::X / 2 : G::X - a);
}
template <typename G> __host__ __device__ constexpr int k1_row(int k1) {
    constexpr int H = G::W / 2;
    const int a = k1 == G::X / 2 ? 0 : (k1 > G::X / 2 ? G::X - k1 : k1);
    return (a / H) * G::W + a % H + (k1 >= G::X / 2 ? H : 0);
}
// Partner, among its own registers, of register e of the lane that pairs itself
// (k1 = 0, lane 0).
template <typename G> __host__ __device__ constexpr int self_partner(int e) {
    if (G::L >= G::X) return (G::X - e) % G::X;
    const int p = e / G::L, k = e % G::L;
    return p == 0 ? (G::L - k) % G::L : (G::X / G::L - p) * G::L + G::L - 1 - k;
}
// That lane's table entries are numbered in order of the pairs' lower
// register; the last register paired with itself (k = NC / 2) is entry X / 2.
template <typename G> __host__ __device__ constexpr int self_entry(int e) {
    int n = 0;
    for (int f = 0; f < e; ++f) n += f != G::LX / 2 && self_partner<G>(f) >= f;
    return e == G::LX / 2 ? G::X / 2 : n;
}
// Frequency held by register i of lane l of sub-transform k1.
template <typename G> __host__ __device__ constexpr int reg_k(int k1, int l, int i) {
    return k1 + G::X * l + (G::L >= G::X ? G::X * G::L * i
                                         : G::X * G::L * (i / G::L) + G::X * G::X * (i % G::L));
}
// Frequency of table entry (i, tid) of a filter's spectrum table, i < X / 2 (the
// owner's register), and of the one entry past them (i = X / 2, tid = 0).
template <typename G> __device__ int spec_k(int i, int tid) {
    if (tid == 0) {
        for (int e = 0; e < G::X; ++e)
            if ((e == G::LX / 2 || self_partner<G>(e) >= e) && self_entry<G>(e) == i)
                return reg_k<G>(0, 0, e);
        return 0;
    }
    return reg_k<G>(row_k1<G>(tid / G::L), tid % G::L, i);
}

// Raw buffer accesses (resource word of the gfx9 family, stride 0): a load
// whose offset (VGPR part plus instruction offset) falls outside
// [0, num_records) bytes returns 0 and such a store is dropped.  A block's
// input resource covers its window clipped to the interval and its output
// resource the block's valid outputs, which gives the overlap-save block its
// zero padding and discards its edges with 32-bit offsets and no compares.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
}
template <typename T> __device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t r, int off);
template <> __device__ __forceinline__ double buf_ld<double>(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <> __device__ __forceinline__ float buf_ld<float>(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, int off, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
}
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, int off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 0);
}
// Two consecutive elements in one access (16 bytes FP64, 8 bytes FP32).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void buf_ld2(__amdgpu_buffer_rsrc_t r, int off, double &a, double &b) {
    const double2 v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    a = v.x;
    b = v.y;
}
__device__ __forceinline__ void buf_ld2(__amdgpu_buffer_rsrc_t r, int off, float &a, float &b) {
    const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    a = v.x;
    b = v.y;
}
__device__ __forceinline__ void buf_st2(__amdgpu_buffer_rsrc_t r, int off, double a, double b) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_double2(a, b)), r, off,
                                           0, 0);
}
__device__ __forceinline__ void buf_st2(__amdgpu_buffer_rsrc_t r, int off, float a, float b) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, make_float2(a, b)), r, off, 0,
                                          0);
}

// Orders a wave's own LDS accesses across its lanes: the hardware runs one
// wave's LDS instructions in order, so only the compiler has to be held.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Twiddles w^k, 1 <= k < X, from w, w^2, w^4, w^8 (and w^16) (each a rounded
// table value, S apart at t): w^k is a product of at most five of them, so its
// error does not grow with k as it does for powers of one rounded w.
// f(k, w^k) is called for every k.
constexpr int n_powers(int X) { return X == 32 ? 5 : 4; }
template <typename T> struct Cx { T r, i; };
template <typename T> __device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b) {
    return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r};
}
template <int X, int DIR, int S, typename T2, typename F>
__device__ __forceinline__ void powers(const T2 *__restrict__ t, const F &f) {
    using T = decltype(T2::x);
    Cx<T> w[n_powers(X)];
#pragma unroll
    for (int c = 0; c < n_powers(X); ++c) {
        const auto v = t[c * S];
        w[c] = {v.x, DIR < 0 ? v.y : -v.y};
    }
    const Cx<T> w3 = cmul(w[1], w[0]);
    f(1, w[0]);
    f(2, w[1]);
    f(3, w3);
    auto four = [&](int k, Cx<T> a) {  // w^k .. w^(k+3) from a = w^k
        f(k, a);
        f(k + 1, cmul(a, w[0]));
        f(k + 2, cmul(a, w[1]));
        f(k + 3, cmul(a, w3));
    };
    four(4, w[2]);
    four(8, w[3]);
    four(12, cmul(w[3], w[2]));
    if constexpr (X == 32) {
        four(16, w[4]);
        four(20, cmul(w[4], w[2]));
        const Cx<T> w24 = cmul(w[4], w[3]);
        four(24, w24);
        four(28, cmul(w24, w[2]));
    }
}

// Swap between lanes 16 apart: a of the upper lane <-> b of the lower.
__device__ __forceinline__ void lane_swap(unsigned &a, unsigned &b) {
    const auto v = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = v[0];
    b = v[1];
}
__device__ __forceinline__ void lane_swap(float &a, float &b) {
    unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    lane_swap(x, y);
    a = __builtin_bit_cast(float, x);
    b = __builtin_bit_cast(float, y);
}
__device__ __forceinline__ void lane_swap(double &a, double &b) {
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    lane_swap(x.x, y.x);
    lane_swap(x.y, y.y);
    a = __builtin_bit_cast(double, x);
    b = __builtin_bit_cast(double, y);
}

// The L-point DFTs of pass 3.  SPLIT (L = 32 on 16 registers): lanes h = 0 and 1,
// 16 apart, share a transform.  Forward: registers i and i + 8 hold elements
// 8 h + i and 8 h + i + 16; radix 2 and its twiddle W32^(8 h + i) in the lane, then
// lane 0 takes the sums and lane 1 the differences, in order, and register i of
// lane h ends with output 2 i + h.
template <typename G, typename T, int DIR>
__device__ __forceinline__ void dft_lanes(T (&re)[G::X], T (&im)[G::X], int l) {
    auto radix2 = [&](int i) {
        const T r = re[i] - re[i + 8], m = im[i] - im[i + 8];
        re[i] += re[i + 8];
        im[i] += im[i + 8];
        re[i + 8] = r;
        im[i + 8] = m;
    };
    auto twiddle = [&](int i) {
        mul_w32<T, DIR>(re[i + 8], im[i + 8], i);
        const T r = re[i + 8], m = im[i + 8];
        re[i + 8] = l >= 16 ? -DIR * m : r;
        im[i + 8] = l >= 16 ? DIR * r : m;
    };
    if constexpr (G::SPLIT && DIR < 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            radix2(i);
            twiddle(i);
            lane_swap(re[i], re[i + 8]);
            lane_swap(im[i], im[i + 8]);
        }
    }
    dft16_at<T, DIR, 0>(re, im);
    if constexpr (G::X == 32) dft16_at<T, DIR, 16>(re, im);
    if constexpr (G::SPLIT && DIR > 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            lane_swap(re[i], re[i + 8]);
            lane_swap(im[i], im[i + 8]);
            twiddle(i);
            radix2(i);
        }
    }
}

// Forward exchange of passes 1 and 2, one component: thread j stores its X
// outputs (k1 in slot outx(k1)) in column j of the rows k1, then loads its own
// row's elements l + L q.
template <typename G, typename T>
__device__ __forceinline__ void put_cols(T *__restrict__ sh, const T (&v)[G::X], int tid) {
#pragma unroll
    for (int k = 0; k < G::X; ++k) sh[k1_row<G>(k) * G::RS + tid] = v[outx<G::X>(k)];
}
template <typename G, typename T>
__device__ __forceinline__ void get_row(const T *__restrict__ row, T (&v)[G::X], int l) {
#pragma unroll
    for (int q = 0; q < G::X; ++q) v[q] = row[l + G::L * q];
}
// Inverse: a lane stores y[l + L q] (slot outx(q)) in its row, then thread j
// loads column j of all rows.
template <typename G, typename T>
__device__ __forceinline__ void put_row(T *__restrict__ row, const T (&v)[G::X], int l) {
#pragma unroll
    for (int q = 0; q < G::X; ++q) row[l + G::L * q] = v[outx<G::X>(q)];
}
template <typename G, typename T>
__device__ __forceinline__ void get_cols(const T *__restrict__ sh, T (&v)[G::X], int tid) {
#pragma unroll
    for (int k = 0; k < G::X; ++k) v[k] = sh[k1_row<G>(k) * G::RS + tid];
}
// Exchange of passes 2 and 3 within a row: [k2a][l] groups, Q apart.  Forward:
// store k2a (slot outx(k2a)) for the own l, load k2a = l + L p for all l.  SPLIT:
// lane k2a + 16 h loads elements 8 h + i and 8 h + i + 16, i < 8, which are kept
// side by side, at 16 h.
template <typename G> __device__ __forceinline__ int row_pos(int l) {
    return G::SPLIT ? (l & 7) | ((l & 16) >> 1) | ((l & 8) << 1) : l;
}
template <typename G> __device__ __forceinline__ int row_at(int l, int i) {
    return G::SPLIT ? (l & 15) * G::Q + (l & 16) + i
                    : (l + G::L * (i / G::LX)) * G::Q + i % G::LX;
}
template <typename G, typename T>
__device__ __forceinline__ void row_fwd(T *__restrict__ row, T (&v)[G::X], int l) {
    wave_sync();
#pragma unroll
    for (int k = 0; k < G::X; ++k) row[k * G::Q + row_pos<G>(l)] = v[outx<G::X>(k)];
    wave_sync();
#pragma unroll
    for (int i = 0; i < G::X; ++i) v[i] = row[row_at<G>(l, i)];
}
template <typename G, typename T>
__device__ __forceinline__ void row_inv(T *__restrict__ row, T (&v)[G::X], int l) {
    wave_sync();
#pragma unroll
    for (int i = 0; i < G::X; ++i) row[row_at<G>(l, i)] = v[i];
    wave_sync();
#pragma unroll
    for (int k = 0; k < G::X; ++k) v[k] = row[k * G::Q + row_pos<G>(l)];
}

// Z'_k and Z'_{NC-k} of a pair in place.  With E = z1 + conj z2 and O = (z1 -
// conj z2) / i (twice E_k and O_k of noise_fft.hip), w = W^k B_k / 2, and A, B
// even and odd under k -> NC - k, W^(NC-k) = -W^-k:
//   P = w O, Q = conj(w) E:  Z'_k = A z1 + P + iQ,
//   Z'_{NC-k} = A z2 + (P_r + Q_i) + i (Q_r - P_i).
template <typename T>
__device__ __forceinline__ void spectrum_pair(T &z1r, T &z1i, T &z2r, T &z2i, T A, Cx<T> w) {
    const T er = z1r + z2r, ei = z1i - z2i;
    const T orr = z1i + z2i, oi = z2r - z1r;
    const T pr = w.r * orr - w.i * oi, pi = w.r * oi + w.i * orr;
    const T qr = w.r * er + w.i * ei, qi = w.r * ei - w.i * er;
    z1r = (A * z1r + pr) - qi;
    z1i = (A * z1i + pi) + qr;
    z2r = (A * z2r + pr) + qi;
    z2i = (A * z2i - pi) + qr;
}

// Entries of a filter's spectrum table: A_k and W^k B_k / 2, each rounded once,
// at k = spec_k(i, tid), entry i TH + tid for i < X / 2 and one entry past them:
// the A of all filters' entries first, then the W^k B_k / 2.
template <typename G> __host__ __device__ constexpr int spec_len() {
    return G::X / 2 * G::TH + 16;
}

// Spectrum step.  A lane owns the pairs of its registers i < X / 2; the partners
// (registers X - 1 - i of the partner lane) go through the wave's own LDS rows
// and back.
template <typename G, typename T>
__device__ __forceinline__ void spectrum_step(T *__restrict__ wsh, T (&re)[G::X], T (&im)[G::X],
                                              const T *__restrict__ sa,
                                              const typename Vec2T<T>::type *__restrict__ sw,
                                              int tid) {
    constexpr int HX = G::X / 2;
    const int lane = tid & 63, l = tid % G::L;
    const int k1 = row_k1<G>(tid / G::L);
    wave_sync();
#pragma unroll
    for (int i = HX; i < G::X; ++i) {
        wsh[((i - HX) * 2) * 64 + lane] = re[i];
        wsh[((i - HX) * 2 + 1) * 64 + lane] = im[i];
    }
    wave_sync();
    if (tid != 0) {
        // partner lane: rows k1 and X - k1 are W / 2 rows apart
        const int s = lane / G::L;
        const int pl = k1 == 0 ? G::L - l
                               : ((k1 == HX ? s : s ^ (G::W / 2)) * G::L + G::L - 1 - l);
        T *ps = wsh + pl;
#pragma unroll
        for (int i = 0; i < HX; ++i) {
            const auto w = sw[i * G::TH + tid];
            T z2r = ps[(HX - 1 - i) * 128], z2i = ps[(HX - 1 - i) * 128 + 64];
            spectrum_pair<T>(re[i], im[i], z2r, z2i, sa[i * G::TH + tid], {w.x, w.y});
            ps[(HX - 1 - i) * 128] = z2r;
            ps[(HX - 1 - i) * 128 + 64] = z2i;
        }
    } else {
#pragma unroll
        for (int e = 0; e < G::X; ++e) {
            const int f = self_partner<G>(e);
            if (f < e) continue;
            const auto w = sw[self_entry<G>(e) * G::TH];
            const T A = sa[self_entry<G>(e) * G::TH];
            if (f == e) {
                T z2r = re[e], z2i = im[e];
                spectrum_pair<T>(re[e], im[e], z2r, z2i, A, {w.x, w.y});
            } else {
                spectrum_pair<T>(re[e], im[e], re[f], im[f], A, {w.x, w.y});
            }
        }
        // its upper half comes back from LDS with the others'
#pragma unroll
        for (int i = HX; i < G::X; ++i) {
            wsh[((i - HX) * 2) * 64] = re[i];
            wsh[((i - HX) * 2 + 1) * 64] = im[i];
        }
    }
    wave_sync();
#pragma unroll
    for (int i = HX; i < G::X; ++i) {
        re[i] = wsh[((i - HX) * 2) * 64 + lane];
        im[i] = wsh[((i - HX) * 2 + 1) * 64 + lane];
    }
}

// qtab[m] = cos(2 pi m / N), m <= N / 4 = NC / 2.
template <typename G, typename T>
__global__ void k_fft_spec(const double *__restrict__ H, int n_filters,
                           const double *__restrict__ qtab, T *__restrict__ sa,
                           typename Vec2T<T>::type *__restrict__ sw) {
    constexpr int NE = spec_len<G>(), HF = G::NC / 2;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)n_filters * NE) return;
    const int64_t f = e / NE;
    const int s = (int)(e % NE);
    // the entries after the X / 2 TH + 1 used ones only pad the table
    const int k = s <= G::X / 2 * G::TH ? spec_k<G>(s / G::TH, s % G::TH) : 0;
    const double hk = H[f * (G::NC + 1) + k];
    const double hc = H[f * (G::NC + 1) + (G::NC - k)];  // H_{k+NC} = H_{NC-k}
    // W^k = e^(-2 pi i k / N), 0 <= k <= NC = N / 2
    const double c = k <= HF ? qtab[k] : -qtab[G::NC - k];
    const double sn = k <= HF ? qtab[HF - k] : qtab[k - HF];
    const double b = (hk - hc) / (4.0 * G::NC);
    typename Vec2T<T>::type v;
    v.x = (T)(b * c);
    v.y = (T)(-b * sn);
    sa[e] = (T)((hk + hc) / (2.0 * G::NC));
    sw[e] = v;
}

// RC = the column count when it is known at compile time (1), else 0 and the
// column count is R.  IN_PLANAR: y holds column after column ([R][n], contiguous
// reads; 8.4M samples x 4 columns, FP64, 16,384-sample blocks: 295 -> 273 us).  IN_MASKED: the data
// as given, [R][n]; flagged samples (jpix < 0) are read as 0 and a non-finite
// value on any other sample sets *bad, so that b = P^T N^-1 (mask . d) needs no
// masked copy of d (2^26 samples, FP64: a pass of 231 us less).
enum { IN_INTERLEAVED, IN_PLANAR, IN_MASKED };
template <typename G, typename T, int RC, int IN>
__global__ void __launch_bounds__(G::TH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 || G::X == 16 ? 4 : 2)))
    k_noise_fft_reg(const int64_t *__restrict__ blocks, const int64_t *__restrict__ istart,
                    const int32_t *__restrict__ fid,
                    const T *__restrict__ sa, const typename Vec2T<T>::type *__restrict__ sw,
                    const typename Vec2T<T>::type *__restrict__ tw, int lam, int V, int R_,
                    int64_t n_blk, const T *__restrict__ y, T *__restrict__ z,
                    const int32_t *__restrict__ jpix, int64_t n, int *__restrict__ bad) {
    __shared__ T sh[G::X * G::RS];
    const int R = RC > 0 ? RC : R_;
    const int tid = threadIdx.x;
    // One flat grid of (block, column) pairs, padded to a multiple of 8 and
    // remapped so that each XCD takes a contiguous run of them.  Neighbouring
    // blocks of an interval then share their 2 lambda-sample halos, and the
    // blocks of one filter its spectrum table, in that XCD's L2; the R columns
    // of a block are neighbours too, and read and write the same interleaved
    // cache lines.  Padding blocks leave before any barrier.
    int64_t bx = blockIdx.x;
    int rr = 0;
    {
        const int64_t l = xcd_block(blockIdx.x, gridDim.x);
        if (l >= n_blk * R) return;
        bx = l / R;
        rr = (int)(l % R);
    }
    const int64_t t0 = blocks[2 * bx];
    const int64_t iv = blocks[2 * bx + 1];
    const int64_t a = istart[iv], e = istart[iv + 1];
    const int64_t base = t0 - lam;
    T re[G::X], im[G::X];
    // pass 1 reads global memory: z_m = y_{base+2m} + i y_{base+2m+1}, m = tid + TH r.
    // The resource spans the window [base, base + 2 NC) clipped to the
    // interval [a, e): samples outside it read as 0.
    const int64_t w0 = base > a ? base : a;
    const int64_t w1 = base + 2 * G::NC < e ? base + 2 * G::NC : e;
    constexpr bool MASK = IN == IN_MASKED, PLANAR = IN != IN_INTERLEAVED;
    const int RI = PLANAR ? 1 : R;  // distance of a column's samples in the input
    const auto ry = raw_rsrc(PLANAR ? y + rr * n + w0 : y + w0 * R,
                             (w1 - w0) * RI * (int64_t)sizeof(T));
    const int off0 = ((int)(base - w0) * RI + (PLANAR ? 0 : rr)) * (int)sizeof(T);
    const bool pairs = (RC == 1 || PLANAR) && (((w0 - base) | (w1 - base)) & 1) == 0;
    // One column: each thread's pair (y_{2m}, y_{2m+1}) is one access when
    // the window's ends fall on even offsets from base, so that no pair
    // straddles them (block-uniform; false only for odd lambda or an odd
    // interval end).  Otherwise, and for several columns, every access moves
    // one element, wholly inside or outside the resource; the second
    // element's offset is hidden from the optimiser there so that the two
    // are never merged into one access across a resource end.
    // MASK: out-of-window pixels read as 0, and the samples there too
    const auto rj = raw_rsrc(MASK ? jpix + w0 : nullptr, MASK ? (w1 - w0) * 4 : 0);
    const int offj = (int)(base - w0) * 4;
    int nf = 0;
    auto keep = [&](unsigned j, T &v) {
        const bool on = (int)j >= 0;
        nf |= on && !isfinite(v);
        v = on ? v : (T)0;
    };
    if (pairs) {
#pragma unroll
        for (int r = 0; r < G::X; ++r)
            buf_ld2(ry, off0 + 2 * (tid + G::TH * r) * (int)sizeof(T), re[r], im[r]);
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < G::X; ++r) {
                const u32x2 j = __builtin_bit_cast(
                    u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                               rj, offj + 8 * (tid + G::TH * r), 0, 0));
                keep(j.x, re[r]);
                keep(j.y, im[r]);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < G::X; ++r) {
            const int off = off0 + 2 * (tid + G::TH * r) * RI * (int)sizeof(T);
            int off1 = off + RI * (int)sizeof(T);
            asm volatile("" : "+v"(off1));
            re[r] = buf_ld<T>(ry, off);
            im[r] = buf_ld<T>(ry, off1);
        }
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < G::X; ++r) {
                const int off = offj + 8 * (tid + G::TH * r);
                int off1 = off + 4;
                asm volatile("" : "+v"(off1));
                keep(__builtin_amdgcn_raw_buffer_load_b32(rj, off, 0, 0), re[r]);
                keep(__builtin_amdgcn_raw_buffer_load_b32(rj, off1, 0, 0), im[r]);
            }
        }
    }
    if (MASK && nf) atomicOr(bad, 1);
    constexpr int NW = n_powers(G::X);
    const int l = tid % G::L;
    T *const row = sh + (tid / G::L) * G::RS;                      // the lane's k1
    T *const wsh = sh + (tid >> 6) * G::W * G::RS;                 // the wave's rows
    // pass 1
    dftx<T, -1>(re, im);
    {
        powers<G::X, -1, G::TH>(tw + tid, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[outx<G::X>(k)], im[outx<G::X>(k)]}, v);
            re[outx<G::X>(k)] = x.r;
            im[outx<G::X>(k)] = x.i;
        });
    }
    put_cols<G>(sh, re, tid);
    __syncthreads();
    get_row<G>(row, re, l);
    __syncthreads();
    put_cols<G>(sh, im, tid);
    __syncthreads();
    get_row<G>(row, im, l);
    // pass 2
    dftx<T, -1>(re, im);
    {
        powers<G::X, -1, G::L>(tw + NW * G::TH + l, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[outx<G::X>(k)], im[outx<G::X>(k)]}, v);
            re[outx<G::X>(k)] = x.r;
            im[outx<G::X>(k)] = x.i;
        });
    }
    row_fwd<G>(row, re, l);
    row_fwd<G>(row, im, l);
    // pass 3, the spectrum, and back
    dft_lanes<G, T, -1>(re, im, l);
    spectrum_step<G, T>(wsh, re, im, sa + (int64_t)fid[iv] * spec_len<G>(),
                        sw + (int64_t)fid[iv] * spec_len<G>(), tid);
    dft_lanes<G, T, 1>(re, im, l);
    row_inv<G>(row, re, l);
    row_inv<G>(row, im, l);
    {
        powers<G::X, 1, G::L>(tw + NW * G::TH + l, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[k], im[k]}, v);
            re[k] = x.r;
            im[k] = x.i;
        });
    }
    dftx<T, 1>(re, im);
    // the wave's rows are its own until the first barrier
    wave_sync();
    put_row<G>(row, re, l);
    __syncthreads();
    get_cols<G>(sh, re, tid);
    __syncthreads();
    put_row<G>(row, im, l);
    __syncthreads();
    get_cols<G>(sh, im, tid);
    {
        powers<G::X, 1, G::TH>(tw + tid, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[k], im[k]}, v);
            re[k] = x.r;
            im[k] = x.i;
        });
    }
    dftx<T, 1>(re, im);
    // slot outx(r) holds z'_m, m = tid + TH r: outputs 2m and 2m + 1 of the
    // block.  Output 2m - lam is valid in [0, nvalid): the resource spans
    // exactly those outputs, the stores of the others are dropped.
    const int64_t nvalid = e - t0 < V ? e - t0 : V;
    const auto rz = raw_rsrc(z + t0 * R, nvalid * R * (int64_t)sizeof(T));
    // pairs as for the loads: the valid range [0, nvalid) starts lam before
    // each pair's even offset 2m, so pairs are whole when lam and nvalid are even
    if (RC == 1 && ((lam | (int)nvalid) & 1) == 0) {
#pragma unroll
        for (int r = 0; r < G::X; ++r)
            buf_st2(rz, (2 * (tid + G::TH * r) - lam) * (int)sizeof(T), re[outx<G::X>(r)],
                    im[outx<G::X>(r)]);
    } else {
#pragma unroll
        for (int r = 0; r < G::X; ++r) {
            const int off = ((2 * (tid + G::TH * r) - lam) * R + rr) * (int)sizeof(T);
            int off1 = off + R * (int)sizeof(T);
            asm volatile("" : "+v"(off1));
            buf_st(rz, off, re[outx<G::X>(r)]);
            buf_st(rz, off1, im[outx<G::X>(r)]);
        }
    }
}

}  // namespace

bool noise_fft_big_supported(int half_bw) { return half_bw >= 1 && half_bw <= BIG_MAX_LAMBDA; }
bool noise_fft_mid_supported(int half_bw) { return half_bw >= 1 && half_bw <= MID_MAX_LAMBDA; }
int noise_fft_big_nc() { return Big::NC; }
int noise_fft_mid_nc() { return Mid::NC; }
int noise_fft_short_nc() { return Short::NC; }
bool noise_fft_short_supported(int half_bw) {
    return half_bw >= 1 && half_bw <= SHORT_MAX_LAMBDA;
}

// The block lengths.
template <typename F> static void pick_geo(int n, const F &f) {
    if (n == 2 * Big::NC) f(Big());
    else if (n == 2 * Mid::NC) f(Mid());
    else f(Short());
}

// Spectrum and twiddle tables for blocks of tb.n = 2 nc real samples, from H_k,
// k <= nc, per filter and cos(2 pi m / 2nc), m <= nc / 2.
void noise_fft_tables_dev(mm_ctx *ctx, const mm_noise *nz, FftTables &tb, const double *H,
                          const double *qtab) {
    auto go = [&](auto GG, auto TT) {
        using G = decltype(GG);
        using T = decltype(TT);
        using T2 = typename Vec2T<T>::type;
        const int64_t tot = (int64_t)nz->n_filters * spec_len<G>();
        tb.spec.alloc(sizeof(T) * 3 * (size_t)tot);
        T *sa = tb.spec.as<T>();
        k_fft_spec<G, T><<<(unsigned)((tot + 255) / 256), 256, 0, ctx->stream>>>(
            H, nz->n_filters, qtab, sa, reinterpret_cast<T2 *>(sa + tot));
        MM_HIP(hipGetLastError());
        // W_NC^(j 2^c), j < TH, then W_TH^(l 2^c), l < L, c < NW (long double
        // on the host, rounded once)
        constexpr int NW = n_powers(G::X);
        std::vector<T2> tw(NW * G::TH + NW * G::L);
        const long double pi2 = 6.283185307179586476925286766559L;
        auto set = [&](T2 &v, int64_t m, int n) {
            const long double x = pi2 * (m % n) / n;
            v.x = (T)cosl(x);
            v.y = (T)-sinl(x);
        };
        for (int c = 0; c < NW; ++c) {
            for (int j = 0; j < G::TH; ++j) set(tw[c * G::TH + j], (int64_t)j << c, G::NC);
            for (int l = 0; l < G::L; ++l)
                set(tw[NW * G::TH + c * G::L + l], (int64_t)l << c, G::TH);
        }
        tb.tw.alloc(sizeof(T2) * tw.size());
        MM_HIP(hipMemcpyAsync(tb.tw.ptr, tw.data(), sizeof(T2) * tw.size(),
                              hipMemcpyHostToDevice, ctx->stream));
        MM_HIP(hipStreamSynchronize(ctx->stream));
    };
    auto pick = [&](auto GG) {
        if (nz->prec == MM_F32) go(GG, 0.f);
        else go(GG, 0.0);
    };
    pick_geo(tb.n, pick);
}

// Register-resident overlap-save apply with the block length the handle was
// prepared for.
// planar: y is [nrhs][n_samp]; jpix (with bad): and unmasked data, masked as it is read.
void noise_fft_reg_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z,
                             bool planar, const int32_t *jpix, int *bad) {
    Scope sc(ctx->prof, ctx->stream, "Ninv_fft");
    const FftTables &tb = nz->fft;
    // (block, column) pairs on a flat grid padded to a multiple of 8 (see
    // the kernel)
    const int64_t nb = tb.n_blocks;
    MM_CHECK(nb > 0, MM_E_OOM, "FFT: no tables (setting the block length ran out of memory)");
    const dim3 grid((unsigned)((nb * nrhs + 7) / 8 * 8));
    auto go = [&](auto GG, auto TT) {
        using G = decltype(GG);
        using T = decltype(TT);
        using T2 = typename Vec2T<T>::type;
        const T *sa = tb.spec.as<T>();
        auto k = nrhs == 1 ? (jpix ? k_noise_fft_reg<G, T, 1, IN_MASKED>
                                   : k_noise_fft_reg<G, T, 1, IN_INTERLEAVED>)
                           : (jpix     ? k_noise_fft_reg<G, T, 0, IN_MASKED>
                              : planar ? k_noise_fft_reg<G, T, 0, IN_PLANAR>
                                       : k_noise_fft_reg<G, T, 0, IN_INTERLEAVED>);
        k<<<grid, G::TH, 0, ctx->stream>>>(
            tb.blocks.as<int64_t>(), nz->istart.as<int64_t>(), nz->fid.as<int32_t>(), sa,
            reinterpret_cast<const T2 *>(sa + (int64_t)nz->n_filters * spec_len<G>()),
            tb.tw.as<T2>(), nz->half_bw, tb.valid, nrhs, nb,
            static_cast<const T *>(y), static_cast<T *>(z), jpix, nz->n_samp, bad);
    };
    auto pick = [&](auto GG) {
        if (nz->prec == MM_F32) go(GG, 0.f);
        else go(GG, 0.0);
    };
    pick_geo(tb.n, pick);
    MM_HIP(hipGetLastError());
}

}  // namespace mm

// N^-1 by FFT with register-resident overlap-save blocks of N = 2 NC real
// samples, packed as NC complex points (the packed-real scheme of
// noise_fft.hip), V = N - 2 lambda valid outputs.
//
// A block has TH = NC / 32 threads of 32 complex values each and a transform
// is NC = 32 x 32 x L, L = NC / 1,024:
//   pass 1  thread j holds x[j + TH r], r < 32: DFT over r, giving k1, times
//           W_NC^(j k1);
//   pass 2  per k1 a TH-point transform on L lanes of one wave: lane l holds
//           j = l + L q, q < 32; DFT over q, giving k2a, times W_TH^(l k2a);
//   pass 3  lane l takes k2a = l + L p, p < 32 / L, for all L values of l:
//           32 / L DFTs of L points, giving k2b.  Register p L + k2b then
//           holds X[k1 + 32 (k2a + 32 k2b)].
// and the inverse transform runs the passes backwards.  Only the exchange
// between passes 1 and 2 crosses waves: it goes through LDS one component at
// a time (FP64: a whole block does not fit), with three barriers.  A wave owns
// the values k1 of a contiguous stretch of LDS rows, so the exchange between
// passes 2 and 3 and the spectrum step stay inside the wave's own rows and
// need no barrier: 6 barriers per block, and the waves of a block drift apart,
// so that one wave's LDS accesses overlap another's arithmetic.
//
// The spectrum step pairs Z_k with Z_{NC-k}.  A wave's k1 come as pairs (a,
// 32 - a) (wave 0 has 0 and 16, each its own partner), so the partner of
// (k1, lane l, register i) is (32 - k1, lane L-1-l, register 31-i) of the same
// wave; for k1 = 0 it is lane L-l, and lane 0 there pairs its own registers.
//
// Two geometries: L = 16 (NC = 16,384: 512 threads, one block per CU;
// bandwidths up to 12,288) and L = 8 (NC = 8,192: 256 threads, two blocks per
// CU; bandwidths up to 6,144).  512 threads with 32 points each leave 256
// VGPRs for 128 of FP64 data, room for the radix-32 temporaries; 1,024 threads
// with 16 points (radices 16 x 16 x 16 x 4) needed three exchanges per
// direction, each across the whole block, and 25 barriers.
//
// What bounds it (FP64, 32,768-sample blocks, 2^27 samples, lambda 4,096):
// FP64 VALU issue (13 us of a block's 31 us) and LDS traffic (8 us) inside the
// CU, which overlap little because the waves of a block start in step; the
// same kernel without global traffic takes 0.55 ms and its loads and stores
// alone 0.40 ms (5.4 TB/s).  Measured against the 16 x 16 x 16 x 4 kernel:
// FP64 0.910 -> 0.738 ms (0.751 -> 0.586 ms with 16,384-sample blocks at
// lambda 1,024), FP32 0.611 -> 0.368 ms.  FP32 blocks need half the LDS and
// registers, so twice as many share a CU.
#include <cmath>
#include <vector>

#include "fft_common.h"
#include "xcd.h"

namespace mm {
namespace {

using fft::dft16_at;
using fft::dft32;
using fft::dft4;
using fft::dft8_at;
using fft::out32;

// Transform geometry (see the top of the file).
template <int L_> struct Geo {
    static constexpr int L = L_;            // lanes per sub-transform
    static constexpr int NC = 1024 * L;     // complex points
    static constexpr int TH = 32 * L;       // threads; points per sub-transform
    static constexpr int P = 32 / L;        // pass-3 transforms per lane
    static constexpr int H = 32 / L;        // pairs of sub-transforms per wave
    // LDS row of one k1: holds TH values (exchange of passes 1 and 2), or 32
    // groups of L values spaced Q apart (passes 2 and 3).  Odd Q and RS = L
    // (mod 32) put the 64 lanes of every access on distinct bank pairs.
    static constexpr int Q = L + 1;
    static constexpr int RS = 32 * Q + L;
    static_assert(L == 8 || L == 16, "NC must be 8,192 or 16,384");
    static_assert(2 * H * RS >= 2048, "a wave's rows hold its half spectrum, two components");
};
constexpr int BIG_MAX_LAMBDA = 12288;  // 32,768-sample blocks: V = N - 2 lambda >= 8,192
constexpr int MID_MAX_LAMBDA = 6144;   // 16,384-sample blocks: V >= 4,096

// Rows are numbered wave by wave, a wave's first H rows holding k1 = a and
// the next H their partners 32 - a (16 for a = 0), a = H w .. H w + H - 1.
template <typename G> __host__ __device__ constexpr int row_k1(int row) {
    const int w = row / (2 * G::H), s = row % (2 * G::H);
    const int a = G::H * w + s % G::H;
    return s < G::H ? a : (a == 0 ? 16 : 32 - a);
}
template <typename G> __host__ __device__ constexpr int k1_row(int k1) {
    const int a = k1 == 16 ? 0 : (k1 > 16 ? 32 - k1 : k1);
    return (a / G::H) * 2 * G::H + a % G::H + (k1 >= 16 ? G::H : 0);
}
// Partner, among its own 32 registers, of register e of the lane that pairs
// itself (k1 = 0, lane 0: k = 32 L p + 1024 k2b).
template <typename G> __host__ __device__ constexpr int self_partner(int e) {
    const int p = e / G::L, k = e % G::L;
    return p == 0 ? (G::L - k) % G::L : (G::P - p) * G::L + G::L - 1 - k;
}
// That lane's table entries are numbered in order of the pairs' lower
// register; the last register paired with itself, L / 2 (k = NC / 2), is entry 16.
template <typename G> __host__ __device__ constexpr int self_entry(int e) {
    int n = 0;
    for (int f = 0; f < e; ++f) n += f != G::L / 2 && self_partner<G>(f) >= f;
    return e == G::L / 2 ? 16 : n;
}
// Frequency of table entry (i, tid) of a filter's spectrum table, i < 16 (the
// owner's register), and of the one entry past them (i = 16, tid = 0).
template <typename G> __device__ int spec_k(int i, int tid) {
    if (tid == 0) {
        for (int e = 0; e < 32; ++e)
            if ((e == G::L / 2 || self_partner<G>(e) >= e) && self_entry<G>(e) == i)
                return 32 * G::L * (e / G::L) + 1024 * (e % G::L);
        return 0;
    }
    const int k1 = row_k1<G>(tid / G::L), l = tid % G::L;
    return k1 + 32 * l + 32 * G::L * (i / G::L) + 1024 * (i % G::L);
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

// Twiddles w^k, 1 <= k < 32, from w, w^2, w^4, w^8 and w^16 (each a rounded
// table value, S apart at t): w^k is a product of at most five of them, so its
// error does not grow with k as it does for powers of one rounded w.
// f(k, w^k) is called for every k.
template <typename T> struct Cx { T r, i; };
template <typename T> __device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b) {
    return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r};
}
template <int DIR, int S, typename T2, typename F>
__device__ __forceinline__ void powers32(const T2 *__restrict__ t, const F &f) {
    using T = decltype(T2::x);
    Cx<T> w[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
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
    four(16, w[4]);
    four(20, cmul(w[4], w[2]));
    const Cx<T> w24 = cmul(w[4], w[3]);
    four(24, w24);
    four(28, cmul(w24, w[2]));
}

// The L-point DFTs of pass 3.
template <typename G, typename T, int DIR>
__device__ __forceinline__ void dft_lanes(T (&re)[32], T (&im)[32]) {
    if constexpr (G::L == 16) {
        dft16_at<T, DIR, 0>(re, im);
        dft16_at<T, DIR, 16>(re, im);
    } else {
        dft8_at<T, DIR, 0>(re, im);
        dft8_at<T, DIR, 8>(re, im);
        dft8_at<T, DIR, 16>(re, im);
        dft8_at<T, DIR, 24>(re, im);
    }
}

// Forward exchange of passes 1 and 2, one component: thread j stores its 32
// outputs (X[k1] in slot out32(k1)) in column j of the rows k1, then loads its
// own row's elements l + L q.
template <typename G, typename T>
__device__ __forceinline__ void put_cols(T *__restrict__ sh, const T (&v)[32], int tid) {
#pragma unroll
    for (int k = 0; k < 32; ++k) sh[k1_row<G>(k) * G::RS + tid] = v[out32(k)];
}
template <typename G, typename T>
__device__ __forceinline__ void get_row(const T *__restrict__ row, T (&v)[32], int l) {
#pragma unroll
    for (int q = 0; q < 32; ++q) v[q] = row[l + G::L * q];
}
// Inverse: a lane stores y[l + L q] (slot out32(q)) in its row, then thread j
// loads column j of all rows.
template <typename G, typename T>
__device__ __forceinline__ void put_row(T *__restrict__ row, const T (&v)[32], int l) {
#pragma unroll
    for (int q = 0; q < 32; ++q) row[l + G::L * q] = v[out32(q)];
}
template <typename G, typename T>
__device__ __forceinline__ void get_cols(const T *__restrict__ sh, T (&v)[32], int tid) {
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = sh[k1_row<G>(k) * G::RS + tid];
}
// Exchange of passes 2 and 3 within a row: [k2a][l] groups, Q apart.  Forward:
// store k2a (slot out32(k2a)) for the own l, load k2a = l + L p for all l.
template <typename G, typename T>
__device__ __forceinline__ void row_fwd(T *__restrict__ row, T (&v)[32], int l) {
    wave_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) row[k * G::Q + l] = v[out32(k)];
    wave_sync();
#pragma unroll
    for (int p = 0; p < G::P; ++p)
#pragma unroll
        for (int s = 0; s < G::L; ++s) v[p * G::L + s] = row[(l + G::L * p) * G::Q + s];
}
template <typename G, typename T>
__device__ __forceinline__ void row_inv(T *__restrict__ row, T (&v)[32], int l) {
    wave_sync();
#pragma unroll
    for (int p = 0; p < G::P; ++p)
#pragma unroll
        for (int s = 0; s < G::L; ++s) row[(l + G::L * p) * G::Q + s] = v[p * G::L + s];
    wave_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = row[k * G::Q + l];
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
// at k = spec_k(i, tid), entry i TH + tid for i < 16 and one entry past them:
// the A of all filters' entries first, then the W^k B_k / 2.
template <typename G> __host__ __device__ constexpr int spec_len() { return 16 * G::TH + 16; }

// Spectrum step.  A lane owns the pairs of its registers i < 16; the partners
// (registers 31 - i of the partner lane) go through the wave's own LDS rows
// and back.
template <typename G, typename T>
__device__ __forceinline__ void spectrum_step(T *__restrict__ wsh, T (&re)[32], T (&im)[32],
                                              const T *__restrict__ sa,
                                              const typename Vec2T<T>::type *__restrict__ sw,
                                              int tid) {
    const int lane = tid & 63, l = tid % G::L;
    const int k1 = row_k1<G>(tid / G::L);
    wave_sync();
#pragma unroll
    for (int i = 16; i < 32; ++i) {
        wsh[((i - 16) * 2) * 64 + lane] = re[i];
        wsh[((i - 16) * 2 + 1) * 64 + lane] = im[i];
    }
    wave_sync();
    if (tid != 0) {
        // partner lane: rows k1 and 32 - k1 are H rows apart
        const int s = lane / G::L;
        const int pl = k1 == 0 ? G::L - l
                               : ((k1 == 16 ? s : (s < G::H ? s + G::H : s - G::H)) * G::L +
                                  G::L - 1 - l);
        T *ps = wsh + pl;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const auto w = sw[i * G::TH + tid];
            T z2r = ps[(15 - i) * 128], z2i = ps[(15 - i) * 128 + 64];
            spectrum_pair<T>(re[i], im[i], z2r, z2i, sa[i * G::TH + tid], {w.x, w.y});
            ps[(15 - i) * 128] = z2r;
            ps[(15 - i) * 128 + 64] = z2i;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 32; ++e) {
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
        for (int i = 16; i < 32; ++i) {
            wsh[((i - 16) * 2) * 64] = re[i];
            wsh[((i - 16) * 2 + 1) * 64] = im[i];
        }
    }
    wave_sync();
#pragma unroll
    for (int i = 16; i < 32; ++i) {
        re[i] = wsh[((i - 16) * 2) * 64 + lane];
        im[i] = wsh[((i - 16) * 2 + 1) * 64 + lane];
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
    // the entries after the 16 TH + 1 used ones only pad the table
    const int k = s <= 16 * G::TH ? spec_k<G>(s / G::TH, s % G::TH) : 0;
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
// column count is R.  MASK: y is the data as given, column after column
// ([R][n]); flagged samples (jpix < 0) are read as 0 and a non-finite value on
// any other sample sets *bad, so that b = P^T N^-1 (mask . d) needs no masked
// copy of d (2^26 samples, FP64: a pass of 231 us less; with several columns
// the reads are contiguous too).
template <typename G, typename T, int RC, bool MASK>
__global__ void __launch_bounds__(G::TH) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
    k_noise_fft_reg(const int64_t *__restrict__ blocks, const int64_t *__restrict__ istart,
                    const int32_t *__restrict__ fid,
                    const T *__restrict__ sa, const typename Vec2T<T>::type *__restrict__ sw,
                    const typename Vec2T<T>::type *__restrict__ tw, int lam, int V, int R_,
                    int64_t n_blk, const T *__restrict__ y, T *__restrict__ z,
                    const int32_t *__restrict__ jpix, int64_t n, int *__restrict__ bad) {
    __shared__ T sh[32 * G::RS];
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
    T re[32], im[32];
    // pass 1 reads global memory: z_m = y_{base+2m} + i y_{base+2m+1}, m = tid + TH r.
    // The resource spans the window [base, base + 2 NC) clipped to the
    // interval [a, e): samples outside it read as 0.
    const int64_t w0 = base > a ? base : a;
    const int64_t w1 = base + 2 * G::NC < e ? base + 2 * G::NC : e;
    const int RI = MASK ? 1 : R;  // distance of a column's samples in the input
    const auto ry = raw_rsrc(MASK ? y + rr * n + w0 : y + w0 * R,
                             (w1 - w0) * RI * (int64_t)sizeof(T));
    const int off0 = ((int)(base - w0) * RI + (MASK ? 0 : rr)) * (int)sizeof(T);
    const bool pairs = (RC == 1 || MASK) && (((w0 - base) | (w1 - base)) & 1) == 0;
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
        for (int r = 0; r < 32; ++r)
            buf_ld2(ry, off0 + 2 * (tid + G::TH * r) * (int)sizeof(T), re[r], im[r]);
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < 32; ++r) {
                const u32x2 j = __builtin_bit_cast(
                    u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                               rj, offj + 8 * (tid + G::TH * r), 0, 0));
                keep(j.x, re[r]);
                keep(j.y, im[r]);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            const int off = off0 + 2 * (tid + G::TH * r) * RI * (int)sizeof(T);
            int off1 = off + RI * (int)sizeof(T);
            asm volatile("" : "+v"(off1));
            re[r] = buf_ld<T>(ry, off);
            im[r] = buf_ld<T>(ry, off1);
        }
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < 32; ++r) {
                const int off = offj + 8 * (tid + G::TH * r);
                int off1 = off + 4;
                asm volatile("" : "+v"(off1));
                keep(__builtin_amdgcn_raw_buffer_load_b32(rj, off, 0, 0), re[r]);
                keep(__builtin_amdgcn_raw_buffer_load_b32(rj, off1, 0, 0), im[r]);
            }
        }
    }
    if (MASK && nf) atomicOr(bad, 1);
    const int l = tid % G::L;
    T *const row = sh + (tid / G::L) * G::RS;                      // the lane's k1
    T *const wsh = sh + (tid >> 6) * 2 * G::H * G::RS;             // the wave's rows
    // pass 1
    dft32<T, -1>(re, im);
    {
        powers32<-1, G::TH>(tw + tid, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[out32(k)], im[out32(k)]}, v);
            re[out32(k)] = x.r;
            im[out32(k)] = x.i;
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
    dft32<T, -1>(re, im);
    {
        powers32<-1, G::L>(tw + 5 * G::TH + l, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[out32(k)], im[out32(k)]}, v);
            re[out32(k)] = x.r;
            im[out32(k)] = x.i;
        });
    }
    row_fwd<G>(row, re, l);
    row_fwd<G>(row, im, l);
    // pass 3, the spectrum, and back
    dft_lanes<G, T, -1>(re, im);
    spectrum_step<G, T>(wsh, re, im, sa + (int64_t)fid[iv] * spec_len<G>(),
                        sw + (int64_t)fid[iv] * spec_len<G>(), tid);
    dft_lanes<G, T, 1>(re, im);
    row_inv<G>(row, re, l);
    row_inv<G>(row, im, l);
    {
        powers32<1, G::L>(tw + 5 * G::TH + l, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[k], im[k]}, v);
            re[k] = x.r;
            im[k] = x.i;
        });
    }
    dft32<T, 1>(re, im);
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
        powers32<1, G::TH>(tw + tid, [&](int k, Cx<T> v) {
            const Cx<T> x = cmul(Cx<T>{re[k], im[k]}, v);
            re[k] = x.r;
            im[k] = x.i;
        });
    }
    dft32<T, 1>(re, im);
    // slot out32(r) holds z'_m, m = tid + TH r: outputs 2m and 2m + 1 of the
    // block.  Output 2m - lam is valid in [0, nvalid): the resource spans
    // exactly those outputs, the stores of the others are dropped.
    const int64_t nvalid = e - t0 < V ? e - t0 : V;
    const auto rz = raw_rsrc(z + t0 * R, nvalid * R * (int64_t)sizeof(T));
    // pairs as for the loads: the valid range [0, nvalid) starts lam before
    // each pair's even offset 2m, so pairs are whole when lam and nvalid are even
    if (RC == 1 && ((lam | (int)nvalid) & 1) == 0) {
#pragma unroll
        for (int r = 0; r < 32; ++r)
            buf_st2(rz, (2 * (tid + G::TH * r) - lam) * (int)sizeof(T), re[out32(r)],
                    im[out32(r)]);
    } else {
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            const int off = ((2 * (tid + G::TH * r) - lam) * R + rr) * (int)sizeof(T);
            int off1 = off + R * (int)sizeof(T);
            asm volatile("" : "+v"(off1));
            buf_st(rz, off, re[out32(r)]);
            buf_st(rz, off1, im[out32(r)]);
        }
    }
}

}  // namespace

bool noise_fft_big_supported(int half_bw) { return half_bw >= 1 && half_bw <= BIG_MAX_LAMBDA; }
bool noise_fft_mid_supported(int half_bw) { return half_bw >= 1 && half_bw <= MID_MAX_LAMBDA; }
int noise_fft_big_nc() { return Geo<16>::NC; }
int noise_fft_mid_nc() { return Geo<8>::NC; }

// Spectrum and twiddle tables for blocks of 2 nc real samples, from H_k,
// k <= nc, per filter and cos(2 pi m / 2nc), m <= nc / 2.
void noise_fft_tables_dev(mm_ctx *ctx, mm_noise *nz, int nc, const double *H,
                          const double *qtab) {
    auto go = [&](auto GG, auto TT) {
        using G = decltype(GG);
        using T = decltype(TT);
        using T2 = typename Vec2T<T>::type;
        const int64_t tot = (int64_t)nz->n_filters * spec_len<G>();
        nz->fft_spec.alloc(sizeof(T) * 3 * (size_t)tot);
        T *sa = nz->fft_spec.as<T>();
        k_fft_spec<G, T><<<(unsigned)((tot + 255) / 256), 256, 0, ctx->stream>>>(
            H, nz->n_filters, qtab, sa, reinterpret_cast<T2 *>(sa + tot));
        MM_HIP(hipGetLastError());
        // W_NC^(j 2^c), j < TH, then W_TH^(l 2^c), l < L, c < 5 (long double
        // on the host, rounded once)
        std::vector<T2> tw(5 * G::TH + 5 * G::L);
        const long double pi2 = 6.283185307179586476925286766559L;
        auto set = [&](T2 &v, int64_t m, int n) {
            const long double x = pi2 * (m % n) / n;
            v.x = (T)cosl(x);
            v.y = (T)-sinl(x);
        };
        for (int c = 0; c < 5; ++c) {
            for (int j = 0; j < G::TH; ++j) set(tw[c * G::TH + j], (int64_t)j << c, G::NC);
            for (int l = 0; l < G::L; ++l)
                set(tw[5 * G::TH + c * G::L + l], (int64_t)l << c, G::TH);
        }
        nz->fft_tw.alloc(sizeof(T2) * tw.size());
        MM_HIP(hipMemcpyAsync(nz->fft_tw.ptr, tw.data(), sizeof(T2) * tw.size(),
                              hipMemcpyHostToDevice, ctx->stream));
        MM_HIP(hipStreamSynchronize(ctx->stream));
    };
    auto pick = [&](auto GG) {
        if (nz->prec == MM_F32) go(GG, 0.f);
        else go(GG, 0.0);
    };
    if (nc == Geo<16>::NC) pick(Geo<16>());
    else pick(Geo<8>());
}

// Register-resident overlap-save apply with the block size the handle was
// prepared for (nz->fft_n = 32,768 or 16,384).
// jpix (with bad): y is unmasked data [nrhs][n_samp], masked as it is read.
void noise_fft_reg_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z,
                             const int32_t *jpix, int *bad) {
    Scope sc(ctx->prof, ctx->stream, "Ninv_fft");
    // (block, column) pairs on a flat grid padded to a multiple of 8 (see
    // the kernel)
    const int64_t nb = nz->n_fft_blocks;
    const dim3 grid((unsigned)((nb * nrhs + 7) / 8 * 8));
    auto go = [&](auto GG, auto TT) {
        using G = decltype(GG);
        using T = decltype(TT);
        using T2 = typename Vec2T<T>::type;
        const T *sa = nz->fft_spec.as<T>();
        auto k = jpix ? (nrhs == 1 ? k_noise_fft_reg<G, T, 1, true>
                                   : k_noise_fft_reg<G, T, 0, true>)
                      : (nrhs == 1 ? k_noise_fft_reg<G, T, 1, false>
                                   : k_noise_fft_reg<G, T, 0, false>);
        k<<<grid, G::TH, 0, ctx->stream>>>(
            nz->fft_blocks.as<int64_t>(), nz->istart.as<int64_t>(), nz->fid.as<int32_t>(), sa,
            reinterpret_cast<const T2 *>(sa + (int64_t)nz->n_filters * spec_len<G>()),
            nz->fft_tw.as<T2>(), nz->half_bw, nz->fft_valid, nrhs, nb,
            static_cast<const T *>(y), static_cast<T *>(z), jpix, nz->n_samp, bad);
    };
    auto pick = [&](auto GG) {
        if (nz->prec == MM_F32) go(GG, 0.f);
        else go(GG, 0.0);
    };
    if (nz->fft_n == 2 * Geo<16>::NC) pick(Geo<16>());
    else pick(Geo<8>());
    MM_HIP(hipGetLastError());
}

}  // namespace mm

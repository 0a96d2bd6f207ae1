// Pointing build: hit counts, observed-pixel selection, compact pixel ids, the
// pixel-sorted sample permutation with its CSR offsets, and the polarisation
// weights (cos 2psi, sin 2psi) of Eq. datamodel, all on the device.
//
// Integer work only apart from the weights, so every integer output is
// bit-exact and independent of scheduling: one stable LSD radix sort of (pixel,
// time) gives the permutation, and the run boundaries of the sorted keys the hit
// counts (an atomic histogram of 8.4M samples took 180 us, the boundaries 15).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "mm_internal.h"
#include "pol_weights.h"

namespace mm {
namespace {

constexpr int BS = 256;

// Sort key (pixel, flagged samples last) and time of each sample; flags[0] = 1 if a
// pixel lies outside [-1, npt), flags[1] = 1 if an angle is not finite.
__global__ void k_keys(const int32_t *__restrict__ pix, const double *__restrict__ psi, int64_t n,
                       int32_t npt, uint32_t *__restrict__ keys, int32_t *__restrict__ vals,
                       int *__restrict__ flags) {
    int bad_pix = 0, bad_psi = 0;
    for (int64_t t = blockIdx.x * (int64_t)BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
        const int32_t p = pix[t];
        const bool in = p >= 0 && p < npt;
        bad_pix |= p < -1 || p >= npt;
        if (psi) bad_psi |= !isfinite(psi[t]);
        keys[t] = in ? (uint32_t)p : (uint32_t)npt;
        vals[t] = (int32_t)t;
    }
    if (bad_pix) atomicOr(&flags[0], 1);
    if (bad_psi) atomicOr(&flags[1], 1);
}

// Runs of equal keys: run of pixel p = sorted entries [start[p], end[p]) (both zeroed
// before, so 0 without samples).
__global__ void k_runs(const uint32_t *__restrict__ keys, int64_t n, uint32_t npt,
                       int32_t *__restrict__ start, int32_t *__restrict__ end) {
    for (int64_t i = blockIdx.x * (int64_t)BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
        const uint32_t k = keys[i];
        if (k >= npt) continue;
        if (i == 0 || keys[i - 1] != k) start[k] = (int32_t)i;
        if (i == n - 1 || keys[i + 1] != k) end[k] = (int32_t)(i + 1);
    }
}

__global__ void k_obs_flag(const int32_t *__restrict__ start, const int32_t *__restrict__ end,
                           int32_t npt, int32_t min_hits, int32_t *__restrict__ hits,
                           int32_t *__restrict__ flag) {
    int32_t p = blockIdx.x * BS + threadIdx.x;
    if (p >= npt) return;
    const int32_t h = end[p] - start[p];
    hits[p] = h;
    flag[p] = h >= min_hits ? 1 : 0;
}

// cidx[p] = rank among observed pixels (exclusive scan of flags), -1 if not
// observed; obs_pix[rank] = p; obs_hits[rank] = hits[p]; obs_hits[n_obs] = 0.
__global__ void k_compact(const int32_t *__restrict__ hits, const int32_t *__restrict__ flag,
                          const int32_t *__restrict__ scan, int32_t npt,
                          int32_t *__restrict__ cidx, int32_t *__restrict__ obs_pix,
                          int32_t *__restrict__ obs_hits) {
    int32_t p = blockIdx.x * BS + threadIdx.x;
    if (p >= npt) return;
    if (flag[p]) {
        int32_t c = scan[p];
        cidx[p] = c;
        obs_pix[c] = p;
        obs_hits[c] = hits[p];
    } else {
        cidx[p] = -1;
    }
    if (p == npt - 1) obs_hits[scan[p] + flag[p]] = 0;
}

__global__ void k_sample_j(const int32_t *__restrict__ pix, const int32_t *__restrict__ cidx,
                           int64_t n, int32_t npt, int32_t *__restrict__ j) {
    for (int64_t t = blockIdx.x * (int64_t)BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
        const int32_t p = pix[t];
        j[t] = p >= 0 && p < npt ? cidx[p] : -1;
    }
}

// perm: the sorted samples of the observed pixels only.
__global__ void k_perm(const uint32_t *__restrict__ keys, const int32_t *__restrict__ vals,
                       int64_t n, uint32_t npt, const int32_t *__restrict__ cidx,
                       const int32_t *__restrict__ start, const int32_t *__restrict__ off,
                       int32_t *__restrict__ perm) {
    for (int64_t i = blockIdx.x * (int64_t)BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS) {
        const uint32_t k = keys[i];
        if (k >= npt) continue;
        const int32_t c = cidx[k];
        if (c >= 0) perm[off[c] + (int32_t)(i - start[k])] = vals[i];
    }
}

template <typename T2>
__global__ void k_weights(const double *__restrict__ psi, int64_t n, T2 *__restrict__ w) {
    using T = decltype(T2::x);
    for (int64_t t = blockIdx.x * (int64_t)BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
        double s, c;
        pol_weights(psi[t], c, s);
        T2 v;
        v.x = (T)c;
        v.y = (T)s;
        w[t] = v;
    }
}

template <typename T2>
__global__ void k_gather_w(const int32_t *__restrict__ perm, const T2 *__restrict__ w, int64_t n,
                           T2 *__restrict__ ws) {
    for (int64_t i = blockIdx.x * (int64_t)BS + threadIdx.x; i < n; i += (int64_t)gridDim.x * BS)
        ws[i] = w[perm[i]];
}

// order[s] = compact pixel visited s-th when P^T walks the observed pixels in
// square tiles of a row-major grid of the given width: key = (tile row, tile
// column, row in tile, column in tile) of the global id.
__global__ void k_tile_keys(const int32_t *__restrict__ obs_pix, int32_t n_obs, int32_t width,
                            int32_t tile, uint64_t *__restrict__ keys, int32_t *__restrict__ vals) {
    const int32_t c = blockIdx.x * BS + threadIdx.x;
    if (c >= n_obs) return;
    const int64_t g = obs_pix[c];
    const int64_t y = g / width, x = g % width;
    const int64_t tiles_x = ((int64_t)width + tile - 1) / tile;
    const uint64_t k = ((uint64_t)((y / tile) * tiles_x + x / tile) << 24) |
                       (uint64_t)((y % tile) * tile + (x % tile));
    keys[c] = k;
    vals[c] = c;
}

// slot[order[r]] = r
__global__ void k_rank(const int32_t *__restrict__ order, int32_t n, int32_t *__restrict__ slot) {
    const int32_t r = blockIdx.x * BS + threadIdx.x;
    if (r < n) slot[order[r]] = r;
}
// Scan direction of each chunk of DIR_CHUNK consecutive samples: the
// displacement over DIR_STEP samples, where both ends are observed, at most
// DIR_MAXD pixels and not zero, votes for one of DIR_BINS angle bins over
// [0, 180) degrees; the chunk takes the bin with most votes (the lowest on a
// tie), or -1 without any vote.  Integer counts only, so the result does not
// depend on scheduling.
constexpr int DIR_CHUNK = 4096;
constexpr int DIR_STEP = 8;
constexpr int DIR_MAXD = 12;
constexpr int DIR_BINS = 12;
constexpr int MAX_COPIES = 4;  // map copies, scan directions kept
__global__ void __launch_bounds__(BS) k_chunk_dir(const int32_t *__restrict__ j,
                                                  const int32_t *__restrict__ obs_pix, int64_t n,
                                                  int32_t width, int32_t *__restrict__ bin) {
    __shared__ int cnt[DIR_BINS];
    if (threadIdx.x < DIR_BINS) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * DIR_CHUNK;
    const int64_t c1 = min(c0 + DIR_CHUNK, n) - DIR_STEP;
    for (int64_t t = c0 + threadIdx.x; t < c1; t += BS) {
        const int32_t a = j[t], b = j[t + DIR_STEP];
        if (a < 0 || b < 0) continue;
        const int32_t ga = obs_pix[a], gb = obs_pix[b];
        const int dx = gb % width - ga % width, dy = gb / width - ga / width;
        if ((dx == 0 && dy == 0) || abs(dx) > DIR_MAXD || abs(dy) > DIR_MAXD) continue;
        float ang = atan2f((float)dy, (float)dx) * (180.0f / 3.14159265f);
        if (ang < 0) ang += 180.0f;
        int k = (int)(ang * (DIR_BINS / 180.0f));
        k = k < 0 ? 0 : (k >= DIR_BINS ? DIR_BINS - 1 : k);
        atomicAdd(&cnt[k], 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int best = -1, bc = 0;
        for (int k = 0; k < DIR_BINS; ++k)
            if (cnt[k] > bc) {
                bc = cnt[k];
                best = k;
            }
        bin[blockIdx.x] = best;
    }
}

// Of the samples of each pixel (pixel, then time order) and scan direction g < G of
// their chunks: how many, cnt[g n_obs + c], and the first, first[g n_obs + c] (n
// without any).  One wave per pixel, so neither needs atomics.
__global__ void __launch_bounds__(BS) k_pixel_dirs(const int32_t *__restrict__ off,
                                                   const int32_t *__restrict__ perm,
                                                   const int32_t *__restrict__ grp, int32_t n_obs,
                                                   int G, int32_t n, int32_t *__restrict__ cnt,
                                                   int32_t *__restrict__ first) {
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * BS) >> 6;
    for (int64_t c = ((int64_t)blockIdx.x * BS + threadIdx.x) >> 6; c < n_obs; c += nw) {
        const int64_t a = off[c], b = off[c + 1];
        int32_t num[MAX_COPIES], fst[MAX_COPIES];
#pragma unroll
        for (int g = 0; g < MAX_COPIES; ++g) {
            num[g] = 0;
            fst[g] = n;
        }
        for (int64_t i = a; i < b; i += 64) {
            const bool in = i + lane < b;
            const int32_t t = in ? perm[i + lane] : 0;
            const int q = in ? grp[t / DIR_CHUNK] : -1;
#pragma unroll
            for (int g = 0; g < MAX_COPIES; ++g) {
                const unsigned long long m = __ballot(q == g);
                if (m != 0 && fst[g] == n) fst[g] = __shfl(t, __ffsll(m) - 1);
                num[g] += __popcll(m);
            }
        }
        if (lane != 0) continue;
#pragma unroll
        for (int g = 0; g < MAX_COPIES; ++g)
            if (g < G) {
                cnt[(int64_t)g * n_obs + c] = num[g];
                first[(int64_t)g * n_obs + c] = fst[g];
            }
    }
}

// The pixel-sorted samples (and weights) regrouped by (direction, pixel), time order
// kept: virtual pixel g n_obs + c takes entries from off2[g n_obs + c] on.
template <typename V>
__global__ void __launch_bounds__(BS) k_dir_scatter(const int32_t *__restrict__ off,
                                                    const int32_t *__restrict__ perm,
                                                    const V *__restrict__ w,
                                                    const int32_t *__restrict__ grp,
                                                    int32_t n_obs, int G,
                                                    const int32_t *__restrict__ off2,
                                                    int32_t *__restrict__ perm2,
                                                    V *__restrict__ w2) {
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * BS) >> 6;
    for (int64_t c = ((int64_t)blockIdx.x * BS + threadIdx.x) >> 6; c < n_obs; c += nw) {
        const int64_t a = off[c], b = off[c + 1];
        int32_t at[MAX_COPIES];
#pragma unroll
        for (int g = 0; g < MAX_COPIES; ++g) at[g] = g < G ? off2[(int64_t)g * n_obs + c] : 0;
        for (int64_t i = a; i < b; i += 64) {
            const bool in = i + lane < b;
            const int32_t t = in ? perm[i + lane] : 0;
            const int q = in ? grp[t / DIR_CHUNK] : -1;
#pragma unroll
            for (int g = 0; g < MAX_COPIES; ++g) {
                const unsigned long long m = __ballot(q == g);
                if (q == g) {
                    const int32_t d = at[g] + __popcll(m & ((1ull << lane) - 1));
                    perm2[d] = t;
                    if (w) w2[d] = w[i + lane];
                }
                at[g] += __popcll(m);
            }
        }
    }
}

// Sort keys: copy, then the first touch (unhit pixels last, in compact id order
// through the stable sort), below bit nb; value = g n_obs + c.
__global__ void k_touch_keys(const int32_t *__restrict__ first, int64_t total, int32_t n_obs,
                             int nb, uint64_t *__restrict__ keys, int32_t *__restrict__ vals) {
    for (int64_t e = blockIdx.x * (int64_t)BS + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * BS) {
        keys[e] = ((uint64_t)(e / n_obs) << nb) | (uint64_t)first[e];
        vals[e] = (int32_t)e;
    }
}

// p_j[t] = slot of sample t's pixel in its chunk's copy (-1 flagged).
__global__ void k_slot_of_sample_g(const int32_t *__restrict__ j, const int32_t *__restrict__ grp,
                                   const int32_t *__restrict__ slot, int64_t n, int32_t n_obs,
                                   int32_t *__restrict__ pj) {
    for (int64_t t = blockIdx.x * (int64_t)BS + threadIdx.x; t < n; t += (int64_t)gridDim.x * BS) {
        const int32_t c = j[t];
        pj[t] = c >= 0 ? slot[(int64_t)grp[t / DIR_CHUNK] * n_obs + c] : -1;
    }
}

// Sliced P^T per scan direction: the lane pixels are copy d's first-touch order of
// the virtual pixels d n_obs + c, a block of G slices per direction.
__global__ void k_sl_pix_dir(const int32_t *__restrict__ slot, int64_t total, int32_t n_obs,
                             int32_t G, int32_t *__restrict__ sl_pix) {
    for (int64_t v = blockIdx.x * (int64_t)BS + threadIdx.x; v < total;
         v += (int64_t)gridDim.x * BS) {
        const int64_t d = v / n_obs;
        const int64_t r = slot[v] - d * n_obs;  // rank in copy d
        sl_pix[d * G * 64 + r] = (int32_t)v;
    }
}

__global__ void k_iota(int32_t n, int32_t *__restrict__ v) {
    const int32_t i = blockIdx.x * BS + threadIdx.x;
    if (i < n) v[i] = i;
}

// Sliced P^T layout.  Lane (g, l) finds, by binary search in its pixel's
// time-sorted list perm[off[c], off[c+1]), where each time segment
// [n s / S, n (s+1) / S) starts; cnt / start are stored per (s G + g, l).
__global__ void k_sl_bounds(const int32_t *__restrict__ sl_pix, int32_t G, int32_t S,
                            int64_t n_samp, const int32_t *__restrict__ off,
                            const int32_t *__restrict__ perm, int32_t *__restrict__ cnt,
                            int32_t *__restrict__ start) {
    const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
    if (i >= (int64_t)G * 64) return;
    const int64_t g = i >> 6, l = i & 63;
    const int32_t c = sl_pix[i];
    int32_t prev = c >= 0 ? off[c] : 0;
    const int32_t end = c >= 0 ? off[c + 1] : 0;
    for (int32_t sg = 0; sg < S; ++sg) {
        int32_t hi = end;
        if (sg + 1 < S) {
            const int64_t T = n_samp * (sg + 1) / S;
            int32_t lo = prev;
            hi = end;
            while (lo < hi) {  // first entry with perm >= T
                const int32_t mid = lo + ((hi - lo) >> 1);
                if (perm[mid] < T)
                    lo = mid + 1;
                else
                    hi = mid;
            }
        }
        const int64_t o = ((int64_t)sg * G + g) * 64 + l;
        cnt[o] = hi - prev;
        start[o] = prev;
        prev = hi;
    }
}

// sizes[w] = 64 x (largest lane count of wave w); sizes[n_waves] = 0.
__global__ void k_sl_width(const int32_t *__restrict__ cnt, int64_t n_waves,
                           int64_t *__restrict__ sizes) {
    const int64_t w = ((int64_t)blockIdx.x * BS + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (w > n_waves) return;
    if (w == n_waves) {
        if (lane == 0) sizes[w] = 0;
        return;
    }
    int32_t m = cnt[w * 64 + lane];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d));
    if (lane == 0) sizes[w] = 64 * (int64_t)m;
}

// Entries of wave w: lane l's k-th sample of its pixel in the segment (or
// padding).  V is the per-entry weight record: the stored weights (FP32
// form) or the angle psi gathered from time order (FP64 form, weights formed
// on the fly).
template <typename V>
__device__ __forceinline__ V sl_value(const V *__restrict__ src, int64_t i, int32_t t) {
    return src[i];
}
template <>
__device__ __forceinline__ double sl_value<double>(const double *__restrict__ psi, int64_t,
                                                   int32_t t) {
    return psi[t];
}
__device__ __forceinline__ void sl_zero(float2 &v) { v = make_float2(0.f, 0.f); }
__device__ __forceinline__ void sl_zero(double &v) { v = 0.0; }

// W = false: no weight records (I).
template <typename V, bool W = true>
__global__ void k_sl_fill(const int64_t *__restrict__ base, const int32_t *__restrict__ cnt,
                          const int32_t *__restrict__ start, const int32_t *__restrict__ perm,
                          const V *__restrict__ src, int64_t n_waves,
                          int32_t *__restrict__ sl_perm, V *__restrict__ sl_w) {
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * BS) >> 6;
    for (int64_t w = ((int64_t)blockIdx.x * BS + threadIdx.x) >> 6; w < n_waves; w += nw) {
        const int64_t b0 = base[w];
        const int64_t len = (base[w + 1] - b0) >> 6;
        const int32_t c = cnt[w * 64 + lane];
        const int32_t st = start[w * 64 + lane];
        // eight entries in flight per lane: their samples, then their records
        for (int64_t k = 0; k < len; k += 8) {
            int32_t t[8];
            V v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) t[q] = k + q < c ? perm[st + k + q] : -1;
            if (W) {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (t[q] >= 0) v[q] = sl_value<V>(src, st + k + q, t[q]);
                    else sl_zero(v[q]);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (k + q >= len) break;
                const int64_t idx = b0 + 64 * (k + q) + lane;
                sl_perm[idx] = t[q];
                if (W) sl_w[idx] = v[q];
            }
        }
    }
}

int grid_for(int64_t n, int max_blocks = 8192) {
    int64_t g = (n + BS - 1) / BS;
    if (g > max_blocks) g = max_blocks;
    return (int)(g < 1 ? 1 : g);
}

// Blocks for a wave per pixel; the kernels go round where a launch of that many threads
// (2^26 pixels) would be refused.
unsigned pixel_waves_grid(int32_t n_obs) {
    return (unsigned)std::min<int64_t>(((int64_t)n_obs + 3) / 4, (int64_t)1 << 22);
}

// rocPRIM with its temporary storage from the call's scratch.
template <typename K, typename V>
void sort_pairs(mm_ctx *ctx, Scratch &tmp, const K *k, K *ko, const V *v, V *vo, int64_t n,
                unsigned end_bit) {
    MM_HIP(hipGetLastError());  // of the launches before: rocPRIM would clear it
    size_t tb = 0;
    MM_HIP(rocprim::radix_sort_pairs(nullptr, tb, k, ko, v, vo, (size_t)n, 0u, end_bit,
                                     ctx->stream));
    MM_HIP(rocprim::radix_sort_pairs(tmp.get<char>(tb + 16), tb, k, ko, v, vo, (size_t)n, 0u,
                                     end_bit, ctx->stream));
}
template <typename T>
void exclusive_sum(mm_ctx *ctx, Scratch &tmp, const T *in, T *out, int64_t n) {
    MM_HIP(hipGetLastError());
    size_t tb = 0;
    MM_HIP(rocprim::exclusive_scan(nullptr, tb, in, out, (T)0, (size_t)n, rocprim::plus<T>(),
                                   ctx->stream));
    MM_HIP(rocprim::exclusive_scan(tmp.get<char>(tb + 16), tb, in, out, (T)0, (size_t)n,
                                   rocprim::plus<T>(), ctx->stream));
}

// Map copies of the single-column P (width > 0), or none.  The lanes of
// a wave gather the map at consecutive samples, i.e. along the scan, so the
// gather touches few cache lines when pixels met one after the other along
// the scan sit next to each other in memory.  One order cannot do that for
// several scan directions, so the map is kept in up to MAX_COPIES copies,
// one per scan direction found (chunks of samples voting by their
// displacement), each ordered by the first sample of its chunks that hits
// each pixel.  The values gathered, hence P's output, do not depend on it.
}  // namespace

// Time segments for the sliced P^T: enough (segment, slice) waves to fill
// the device (8,192 = 32 per CU on 256 CUs), and at least one segment per 2^22
// samples of time, so that the stretch of the TOD the resident waves gather from at
// any moment stays small enough for the L2 (at 1.34e8 samples: 32 segments,
// measured best among 8..128); at most 64, and at least 32 entries per lane,
// segment and scan direction on average.  A function of the problem size only, so the
// summation order (and the bits of the result) does not depend on the device.
static int32_t slice_segments(int64_t n_samp, int64_t n_valid, int32_t n_obs, int32_t G,
                              int32_t D) {
    int64_t S = 8192 / G;
    if (S < (n_samp >> 22)) S = n_samp >> 22;
    if (S > 64) S = 64;
    const int64_t cap = n_obs > 0 ? n_valid / n_obs / 32 / D : 0;
    if (S > cap) S = cap;
    return (int32_t)(S < 1 ? 1 : S);
}

// Whether the sliced P^T has waves enough: below about 2,048 the one-wave-per-pixel
// kernel is the faster one.
static bool slice_waves(const mm_pointing *p) {
    const int32_t G0 = (p->n_obs + 63) / 64;
    return p->n_valid > 0 &&
           (int64_t)G0 * slice_segments(p->n_samp, p->n_valid, p->n_obs, G0, 1) >= 2048;
}

void pointing_p_slots_device(mm_ctx *ctx, mm_pointing *p, int32_t width, Scratch &sc,
                             const int32_t **dir_cnt) {
    hipStream_t s = ctx->stream;
    const int32_t n_obs = p->n_obs;
    // the old slots go with the count: P gathers from copies where p_j is there
    p->p_copies = 0;
    p->p_j.release();
    if (width <= 0 || n_obs == 0) {
        p->p_slot.release();
        p->p_chunk_grp.release();
        return;
    }
    const int64_t n = p->n_samp;
    const int64_t n_chunks = (n + DIR_CHUNK - 1) / DIR_CHUNK;
    int32_t *dbin = sc.get<int32_t>(n_chunks);
    k_chunk_dir<<<(unsigned)n_chunks, BS, 0, s>>>(p->j.as<int32_t>(), p->obs_pix.as<int32_t>(), n,
                                                  width, dbin);
    MM_HIP(hipGetLastError());
    std::vector<int32_t> bin(n_chunks);
    MM_HIP(hipMemcpyAsync(bin.data(), dbin, sizeof(int32_t) * n_chunks, hipMemcpyDeviceToHost, s));
    MM_HIP(hipStreamSynchronize(s));
    // directions holding at least 1/16 of the directed chunks, most first; a
    // bin next to a kept one is not kept (a direction on a bin boundary
    // splits its chunks between two bins)
    int64_t cnt[DIR_BINS] = {};
    int64_t directed = 0;
    for (int32_t b : bin)
        if (b >= 0) {
            ++cnt[b];
            ++directed;
        }
    std::vector<int> kept;
    {
        std::vector<int> byc(DIR_BINS);
        for (int k = 0; k < DIR_BINS; ++k) byc[k] = k;
        std::stable_sort(byc.begin(), byc.end(), [&](int a, int b) { return cnt[a] > cnt[b]; });
        for (int k : byc) {
            if (cnt[k] == 0 || cnt[k] * 16 < directed || (int)kept.size() == MAX_COPIES) continue;
            bool near = false;
            for (int q : kept) {
                const int d = std::abs(k - q);
                near |= std::min(d, DIR_BINS - d) <= 1;
            }
            if (!near) kept.push_back(k);
        }
    }
    int G = kept.empty() ? 1 : (int)kept.size();
    if ((int64_t)G * n_obs >= (int64_t)1 << 31) G = 1;
    // I and QU: the packed copies fit in a TOD vector, where the A apply that
    // allocates nothing puts them (they would not only for a few hits per pixel)
    if (p->nc != 3) {
        const size_t te = p->prec == MM_F32 ? sizeof(float) : sizeof(double);
        const size_t tod = te * (size_t)n;
        if (sizeof(double) * (size_t)(p->n() * G) > tod) G = 1;
        if (sizeof(double) * (size_t)p->n() > tod) {
            p->p_slot.release();
            p->p_chunk_grp.release();
            return;
        }
    }
    // the slots and the chunks' directions only where P gathers from the copies or P^T
    // is cut by them
    const bool gathers = gathers_copies(n, n_obs);
    if (!gathers && !slice_waves(p)) {
        p->p_slot.release();
        p->p_chunk_grp.release();
        p->p_copies = G;
        return;
    }
    // each chunk to the copy of the nearest kept direction (angles mod 180),
    // undirected chunks to the most common one
    std::vector<int32_t> grp(n_chunks, 0);
    if (G > 1)
        for (int64_t c = 0; c < n_chunks; ++c) {
            if (bin[c] < 0) continue;
            int bg = 0, bd = DIR_BINS;
            for (int g = 0; g < G; ++g) {
                int d = std::abs(bin[c] - kept[g]);
                d = std::min(d, DIR_BINS - d);
                if (d < bd) {
                    bd = d;
                    bg = g;
                }
            }
            grp[c] = bg;
        }
    DBuf &dgrp = p->p_chunk_grp;
    dgrp.alloc(sizeof(int32_t) * n_chunks);
    MM_HIP(hipMemcpyAsync(dgrp.ptr, grp.data(), sizeof(int32_t) * n_chunks,
                          hipMemcpyHostToDevice, s));
    MM_HIP(hipStreamSynchronize(s));  // grp goes out of scope
    const int64_t total = (int64_t)G * n_obs;
    int32_t *first = sc.get<int32_t>(total), *dcnt = sc.get<int32_t>(total + 1);
    MM_HIP(hipMemsetAsync(dcnt + total, 0, sizeof(int32_t), s));
    k_pixel_dirs<<<pixel_waves_grid(n_obs), BS, 0, s>>>(p->off.as<int32_t>(),
                                                           p->perm.as<int32_t>(),
                                                           dgrp.as<int32_t>(), n_obs, G,
                                                           (int32_t)n, dcnt, first);
    uint64_t *keys = sc.get<uint64_t>(total), *ko = sc.get<uint64_t>(total);
    int32_t *vals = sc.get<int32_t>(total), *order = sc.get<int32_t>(total);
    const unsigned nb = bits((uint64_t)n);
    k_touch_keys<<<grid_for(total), BS, 0, s>>>(first, total, n_obs, (int)nb, keys, vals);
    // copy g's slots are [g n_obs, (g + 1) n_obs): the key's top bits are g
    sort_pairs(ctx, sc, keys, ko, vals, order, total, nb + 2);
    p->p_slot.alloc(sizeof(int32_t) * total);
    k_rank<<<(unsigned)((total + BS - 1) / BS), BS, 0, s>>>(order, (int32_t)total,
                                                           p->p_slot.as<int32_t>());
    if (gathers) {
        p->p_j.alloc(sizeof(int32_t) * n);
        k_slot_of_sample_g<<<grid_for(n), BS, 0, s>>>(p->j.as<int32_t>(), dgrp.as<int32_t>(),
                                                      p->p_slot.as<int32_t>(), n, n_obs,
                                                      p->p_j.as<int32_t>());
    }
    MM_HIP(hipGetLastError());
    p->p_copies = G;
    *dir_cnt = dcnt;
}

// Visiting order of the one-wave-per-pixel P^T: square tiles of the grid.
static void pointing_tile_order(mm_ctx *ctx, mm_pointing *p, int32_t width, int32_t tile,
                                Scratch &sc, int32_t *order) {
    const int32_t n_obs = p->n_obs;
    uint64_t *keys = sc.get<uint64_t>(n_obs), *ko = sc.get<uint64_t>(n_obs);
    int32_t *vals = sc.get<int32_t>(n_obs);
    k_tile_keys<<<(n_obs + BS - 1) / BS, BS, 0, ctx->stream>>>(p->obs_pix.as<int32_t>(), n_obs,
                                                              width, tile, keys, vals);
    sort_pairs(ctx, sc, keys, ko, vals, order, n_obs, tile_key_bits(p->n_pix_total, width, tile));
}

// dir_cnt: samples per virtual pixel (with map copies of several directions).
static void pointing_slices_device(mm_ctx *ctx, mm_pointing *p, int32_t width, Scratch &sc,
                                   const int32_t *dir_cnt) {
    hipStream_t s = ctx->stream;
    p->sl_G = p->sl_S = 0;
    p->sl_D = 1;
    // a rebuilt layout takes the old one's buffers where they are large enough; without
    // sl_perm, P^T takes a wave per pixel
    auto drop = [&]() {
        p->sl_pix.release();
        p->sl_base.release();
        p->sl_perm.release();
        p->sl_w.release();
    };
    const int32_t n_obs = p->n_obs;
    if (n_obs == 0 || p->n_valid == 0) return drop();
    if (!slice_waves(p)) return drop();
    const int32_t G0 = (n_obs + 63) / 64;
    // per scan direction when the map copies of P are there
    const bool dirs = width > 0 && p->p_copies > 0 && p->p_chunk_grp.ptr;
    const int32_t D = dirs ? p->p_copies : 1;
    const int32_t S = slice_segments(p->n_samp, p->n_valid, n_obs, G0, D);
    const int32_t G = G0 * D;
    const int64_t nv = p->n_valid;
    const bool f32 = p->prec == MM_F32;
    // I and QU: the partial maps too fit in a TOD vector (see the map copies)
    if (p->nc != 3 && sizeof(double) * (size_t)(p->n() * S * D) >
                          (f32 ? sizeof(float) : sizeof(double)) * (size_t)p->n_samp)
        return drop();
    // the pixel-sorted samples and their CSR offsets, over virtual pixels
    // d n_obs + c when cut by direction
    const int32_t *perm_u = p->perm.as<int32_t>();
    const int32_t *off_u = p->off.as<int32_t>();
    const void *ws_u = f32 ? p->ws.ptr : nullptr;
    if (dirs && D > 1) {
        const int64_t nvp = (int64_t)D * n_obs;
        int32_t *off2 = sc.get<int32_t>(nvp + 1), *perm2 = sc.get<int32_t>(nv);
        exclusive_sum(ctx, sc, dir_cnt, off2, nvp + 1);
        const bool w32 = f32 && p->nc > 1;
        float2 *ws2 = w32 ? sc.get<float2>(nv) : nullptr;
        k_dir_scatter<float2><<<pixel_waves_grid(n_obs), BS, 0, s>>>(
            p->off.as<int32_t>(), perm_u, w32 ? p->ws.as<float2>() : nullptr,
            p->p_chunk_grp.as<int32_t>(), n_obs, D, off2, perm2, ws2);
        MM_HIP(hipGetLastError());
        perm_u = perm2;
        off_u = off2;
        ws_u = ws2;
    }

    p->sl_pix.alloc(sizeof(int32_t) * (size_t)G * 64);
    MM_HIP(hipMemsetAsync(p->sl_pix.ptr, 0xff, sizeof(int32_t) * (size_t)G * 64, s));
    if (dirs) {
        const int64_t nvp = (int64_t)D * n_obs;
        k_sl_pix_dir<<<grid_for(nvp), BS, 0, s>>>(p->p_slot.as<int32_t>(), nvp, n_obs, G0,
                                                  p->sl_pix.as<int32_t>());
    } else if (width > 0) {
        pointing_tile_order(ctx, p, width, 8, sc, p->sl_pix.as<int32_t>());
    } else {
        k_iota<<<(n_obs + BS - 1) / BS, BS, 0, s>>>(n_obs, p->sl_pix.as<int32_t>());
    }

    const int64_t n_waves = (int64_t)G * S;
    int32_t *cnt = sc.get<int32_t>(n_waves * 64), *start = sc.get<int32_t>(n_waves * 64);
    int64_t *sizes = sc.get<int64_t>(n_waves + 1);
    p->sl_base.alloc(sizeof(int64_t) * (n_waves + 1));
    k_sl_bounds<<<(unsigned)((G * 64 + BS - 1) / BS), BS, 0, s>>>(
        p->sl_pix.as<int32_t>(), G, S, p->n_samp, off_u, perm_u, cnt, start);
    k_sl_width<<<(unsigned)((n_waves + 1) * 64 / BS + 1), BS, 0, s>>>(cnt, n_waves, sizes);
    exclusive_sum(ctx, sc, sizes, p->sl_base.as<int64_t>(), n_waves + 1);
    int64_t total = 0;
    MM_HIP(hipMemcpyAsync(&total, p->sl_base.as<int64_t>() + n_waves, sizeof(int64_t),
                          hipMemcpyDeviceToHost, s));
    MM_HIP(hipStreamSynchronize(s));
    p->sl_G = G;
    p->sl_S = S;
    p->sl_D = D;
    if (!slices_pay(p->nc, p->n_samp, nv, total)) return drop();
    p->sl_perm.alloc(sizeof(int32_t) * (size_t)total);
    if (p->nc > 1) p->sl_w.alloc(sizeof(double) * (size_t)total);  // psi, or two FP32 weights
    const unsigned fb = (unsigned)std::min<int64_t>((n_waves * 64 + BS - 1) / BS, 16384);
    if (p->nc == 1)
        k_sl_fill<double, false><<<fb, BS, 0, s>>>(p->sl_base.as<int64_t>(), cnt,
                                                   start, perm_u, nullptr, n_waves,
                                                   p->sl_perm.as<int32_t>(), nullptr);
    else if (f32)
        k_sl_fill<float2><<<fb, BS, 0, s>>>(p->sl_base.as<int64_t>(), cnt,
                                            start, perm_u,
                                            static_cast<const float2 *>(ws_u), n_waves,
                                            p->sl_perm.as<int32_t>(), p->sl_w.as<float2>());
    else
        k_sl_fill<double><<<fb, BS, 0, s>>>(p->sl_base.as<int64_t>(), cnt,
                                            start, perm_u, p->psi.as<double>(),
                                            n_waves, p->sl_perm.as<int32_t>(),
                                            p->sl_w.as<double>());
    MM_HIP(hipGetLastError());
}

// A failure leaves the pointing without the layouts (as with no grid and too few waves
// for the sliced P^T), so that no apply reads a half-written one.
void pointing_layout_device(mm_ctx *ctx, mm_pointing *p, int32_t width) {
    try {
        Scratch sc(ctx);
        if (width <= 0) {
            p->seg_order.release();
        } else if (p->n_obs > 0) {
            p->seg_order.alloc(sizeof(int32_t) * p->n_obs);
            pointing_tile_order(ctx, p, width, 32, sc, p->seg_order.as<int32_t>());
        }
        p->grid_width = width;
        // P's map copies first: the sliced P^T is cut by the same scan directions
        const int32_t *dir_cnt = nullptr;
        pointing_p_slots_device(ctx, p, width, sc, &dir_cnt);
        pointing_slices_device(ctx, p, width, sc, dir_cnt);
        MM_HIP(hipStreamSynchronize(ctx->stream));
    } catch (...) {
        p->grid_width = p->p_copies = p->sl_G = p->sl_S = 0;
        p->sl_D = 1;
        for (DBuf *b : {&p->seg_order, &p->p_slot, &p->p_j, &p->p_chunk_grp, &p->sl_pix,
                        &p->sl_base, &p->sl_perm, &p->sl_w})
            b->release();
        throw;
    }
}

void pointing_build_device(mm_ctx *ctx, mm_pointing *p, const int32_t *pix, const double *psi,
                           int32_t min_hits) {
    hipStream_t s = ctx->stream;
    const int64_t n = p->n_samp;
    const int32_t npt = p->n_pix_total;

    Scratch sc(ctx);
    uint32_t *keys = sc.get<uint32_t>(n), *keys_o = sc.get<uint32_t>(n);
    int32_t *vals = sc.get<int32_t>(n), *vals_o = sc.get<int32_t>(n);
    int *flags = sc.get<int>(2);
    int32_t *start = sc.get<int32_t>(npt), *end = sc.get<int32_t>(npt);
    MM_HIP(hipMemsetAsync(flags, 0, 2 * sizeof(int), s));
    MM_HIP(hipMemsetAsync(start, 0, sizeof(int32_t) * npt, s));
    MM_HIP(hipMemsetAsync(end, 0, sizeof(int32_t) * npt, s));
    k_keys<<<grid_for(n), BS, 0, s>>>(pix, psi, n, npt, keys, vals, flags);
    sort_pairs(ctx, sc, keys, keys_o, vals, vals_o, n, bits((uint64_t)npt));
    k_runs<<<grid_for(n), BS, 0, s>>>(keys_o, n, (uint32_t)npt, start, end);

    int32_t *flag = sc.get<int32_t>(npt), *scan = sc.get<int32_t>(npt);
    int32_t *cidx = sc.get<int32_t>(npt);
    p->hits.alloc(sizeof(int32_t) * npt);
    k_obs_flag<<<(npt + BS - 1) / BS, BS, 0, s>>>(start, end, npt, min_hits,
                                                   p->hits.as<int32_t>(), flag);
    exclusive_sum(ctx, sc, flag, scan, npt);
    int hf[2];
    int32_t last[2];
    MM_HIP(hipMemcpyAsync(hf, flags, sizeof(hf), hipMemcpyDeviceToHost, s));
    MM_HIP(hipMemcpyAsync(&last[0], scan + npt - 1, 4, hipMemcpyDeviceToHost, s));
    MM_HIP(hipMemcpyAsync(&last[1], flag + npt - 1, 4, hipMemcpyDeviceToHost, s));
    MM_HIP(hipStreamSynchronize(s));
    MM_CHECK(!hf[0], MM_E_INVALID, "pointing: pixel index outside [-1, n_pix_total)");
    MM_CHECK(!hf[1], MM_E_NONFINITE, "pointing: non-finite angle psi");
    const int32_t n_obs = last[0] + last[1];
    p->n_obs = n_obs;

    p->obs_pix.alloc(sizeof(int32_t) * (n_obs > 0 ? n_obs : 1));
    int32_t *obs_hits = sc.get<int32_t>(n_obs + 1);
    k_compact<<<(npt + BS - 1) / BS, BS, 0, s>>>(p->hits.as<int32_t>(), flag, scan, npt, cidx,
                                                  p->obs_pix.as<int32_t>(), obs_hits);
    p->off.alloc(sizeof(int32_t) * (n_obs + 1));
    exclusive_sum(ctx, sc, obs_hits, p->off.as<int32_t>(), n_obs + 1);
    int32_t nv;
    MM_HIP(hipMemcpyAsync(&nv, p->off.as<int32_t>() + n_obs, 4, hipMemcpyDeviceToHost, s));
    // compact pixel per sample and the sorted samples of the observed pixels
    p->j.alloc(sizeof(int32_t) * n);
    k_sample_j<<<grid_for(n), BS, 0, s>>>(pix, cidx, n, npt, p->j.as<int32_t>());
    MM_HIP(hipStreamSynchronize(s));
    p->n_valid = nv;
    p->perm.alloc(sizeof(int32_t) * (nv > 0 ? nv : 1));
    k_perm<<<grid_for(n), BS, 0, s>>>(keys_o, vals_o, n, (uint32_t)npt, cidx, start,
                                      p->off.as<int32_t>(), p->perm.as<int32_t>());
    MM_HIP(hipGetLastError());

    // weights in time order and in pixel-sorted order; the FP64 form also
    // keeps the angles, from which its single-column P and P^T form the
    // weights on the fly (8 bytes per sample read instead of 16).  An
    // intensity-only pointing has unit weights and keeps neither.
    const bool f32 = p->prec == MM_F32;
    if (p->nc == 1) {
        pointing_slices_device(ctx, p, 0, sc, nullptr);
        MM_HIP(hipStreamSynchronize(s));
        return;
    }
    if (!f32) {
        p->psi.alloc(sizeof(double) * n);
        MM_HIP(hipMemcpyAsync(p->psi.ptr, psi, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
    }
    const size_t wsz = f32 ? sizeof(float2) : sizeof(double2);
    p->w.alloc(wsz * n);
    p->ws.alloc(wsz * (nv > 0 ? nv : 1));
    if (f32) {
        k_weights<float2><<<grid_for(n), BS, 0, s>>>(psi, n, p->w.as<float2>());
        if (nv) k_gather_w<float2><<<grid_for(nv), BS, 0, s>>>(p->perm.as<int32_t>(),
                                                              p->w.as<float2>(), nv,
                                                              p->ws.as<float2>());
    } else {
        k_weights<double2><<<grid_for(n), BS, 0, s>>>(psi, n, p->w.as<double2>());
        if (nv) k_gather_w<double2><<<grid_for(nv), BS, 0, s>>>(p->perm.as<int32_t>(),
                                                                p->w.as<double2>(), nv,
                                                                p->ws.as<double2>());
    }
    MM_HIP(hipGetLastError());

    pointing_slices_device(ctx, p, 0, sc, nullptr);
    MM_HIP(hipStreamSynchronize(s));
}

}  // namespace mm

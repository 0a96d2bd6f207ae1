// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdint>
#include <cstdio>
#include <map>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../include/mapmaker.h"

namespace mm {

// An error carried from deep inside a call up to the C-ABI boundary, where it
// becomes the call's status and the context's last-error message.
struct Error : std::runtime_error {
    mm_status code;
    Error(mm_status c, const std::string &m) : std::runtime_error(m), code(c) {}
};

#define MM_HIP(expr)                                                                   \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            throw ::mm::Error(e_ == hipErrorOutOfMemory ? MM_E_OOM : MM_E_DEVICE,      \
                              std::string(#expr) + ": " + hipGetErrorString(e_));      \
    } while (0)

#define MM_CHECK(cond, code, msg)                                                      \
    do {                                                                               \
        if (!(cond)) throw ::mm::Error((code), (msg));                                 \
    } while (0)

// Device memory of the library's buffers.  dev_free waits for the device, as hipFree
// does, and keeps the block for a later dev_alloc of about its size (registering a
// strategy of 8.4M samples and dropping it: 4.1 ms, or up to 13 ms in a process that
// holds more memory, without this; 2.0 ms with it).
// At most POOL_MAX_BYTES per device are kept, and given back when the device's last
// context goes, or when a hipMalloc fails.  Any thread may call them.
constexpr size_t POOL_MAX_BYTES = (size_t)1 << 30;
void *dev_alloc(size_t bytes, size_t *got);  // nullptr when there is no memory
void dev_free(void *ptr, size_t bytes) noexcept;  // bytes: what dev_alloc gave
void dev_pool_ctx(int device, int delta);    // a context was created (+1) or destroyed (-1)
void dev_pool_trim(int device) noexcept;     // gives back what is kept for the device

// Owning device buffer.
struct DBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    DBuf() = default;
    DBuf(const DBuf &) = delete;
    DBuf &operator=(const DBuf &) = delete;
    DBuf(DBuf &&o) noexcept : ptr(o.ptr), bytes(o.bytes) { o.ptr = nullptr; o.bytes = 0; }
    DBuf &operator=(DBuf &&o) noexcept {
        if (this != &o) { release(); ptr = o.ptr; bytes = o.bytes; o.ptr = nullptr; o.bytes = 0; }
        return *this;
    }
    ~DBuf() { release(); }
    void release() {
        if (ptr) dev_free(ptr, bytes);
        ptr = nullptr;
        bytes = 0;
    }
    // Grow-only.  Growing a buffer that queued kernels may still use waits
    // for the device first.
    void alloc(size_t b) {
        if (b <= bytes && ptr) return;
        release();
        if (b == 0) return;
        ptr = dev_alloc(b, &bytes);
        if (!ptr) {
            bytes = 0;
            throw Error(MM_E_OOM, "hipMalloc of " + std::to_string(b) + " bytes failed");
        }
    }
    template <typename T> T *as() const { return static_cast<T *>(ptr); }
};

// Per-stage timing with HIP events on the context's stream.
struct Profiler {
    bool on = false;
    struct Stage { double ms = 0; int64_t calls = 0; };
    std::map<std::string, Stage> stages;
    struct Pending { std::string name; hipEvent_t a, b; };
    std::vector<Pending> pending;
    std::vector<hipEvent_t> pool;
    hipEvent_t get();
    void flush();  // synchronises on the recorded events
    ~Profiler();
};

struct Scope {
    Profiler *pr;
    hipStream_t s;
    const char *name;
    hipEvent_t a{}, b{};
    Scope(Profiler &p, hipStream_t st, const char *n);
    ~Scope();
};

}  // namespace mm

struct mm_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    std::string last_error;
    mm::Profiler prof;
    // reusable workspace
    mm::DBuf tod_a, tod_b;         // TOD temporaries for A applies
    mm::DBuf red;                  // reduction partials
    mm::DBuf scal;                 // small device scalars
    mm::DBuf gram_part, coef_g;    // MFMA Gram partials, coarse right-hand sides
    mm::DBuf xpack;                // map repacked for P: (I, Q, U, 0) records, or I and (Q, U) split
    mm::DBuf pt_part;              // per-segment partial maps of the sliced P^T
    mm::DBuf flag;                 // device error flag of a call
    mm::DBuf build_ws;             // scratch of the build calls (Scratch below)
    size_t build_off = 0;          // bytes of it in use
    mm::DBuf tod_c;                // template filter: filtered TOD, ground sums and amplitudes
    // Bumped whenever one of the workspaces above is reallocated: captured
    // graphs hold their addresses and are re-captured when it changes.
    uint64_t ws_gen = 0;
    hipStream_t cap = nullptr;     // private stream for graph capture
    double *pinned = nullptr;      // host pinned scratch (scalar readback)
    size_t pinned_bytes = 0;
    int n_cu = 256;
};

namespace mm {
// Grow a context workspace, recording the reallocation.
inline void ws_alloc(mm_ctx *ctx, DBuf &b, size_t bytes) {
    if (b.ptr && bytes <= b.bytes) return;
    b.alloc(bytes);
    ++ctx->ws_gen;
}
// Temporaries of a build call, cut from the context's build_ws: a build takes dozens
// of them, and a hipMalloc and hipFree each cost more than the kernels (6 of 10 ms
// at 8.4M samples, several times that in a process holding much memory).  What does
// not fit is allocated for the call; at the end of the outermost call the workspace
// grows to what was needed, up to MAX_KEPT.  Only work on the context's stream may
// use the memory.  Not to be held across another context's calls.
class Scratch {
  public:
    static constexpr size_t MAX_KEPT = (size_t)512 << 20;
    explicit Scratch(mm_ctx *c) : ctx(c), off0(c->build_off) {}
    Scratch(const Scratch &) = delete;
    Scratch &operator=(const Scratch &) = delete;
    ~Scratch() {
        ctx->build_off = off0;
        if (extra.empty()) return;
        (void)hipStreamSynchronize(ctx->stream);
        extra.clear();
        if (off0 == 0 && used <= MAX_KEPT) {
            try {
                ctx->build_ws.alloc(used);
            } catch (...) {  // the next call allocates its own again
            }
        }
    }
    template <typename T> T *get(int64_t n) {
        if (n < 0 || n > (int64_t)1 << 50)  // a size that overflowed on the way here
            throw Error(MM_E_OOM, "scratch of " + std::to_string(n) + " elements");
        const size_t b = (sizeof(T) * (size_t)(n > 0 ? n : 1) + 255) / 256 * 256;
        used += b;
        if (ctx->build_off + b <= ctx->build_ws.bytes) {
            T *p = reinterpret_cast<T *>(static_cast<char *>(ctx->build_ws.ptr) + ctx->build_off);
            ctx->build_off += b;
            return p;
        }
        // a block as large as all taken so far (64 KiB to 256 MiB), so that a first
        // call makes few of them
        if (extra.empty() || extra_off + b > extra.back().bytes) {
            size_t blk = used < ((size_t)64 << 10) ? (size_t)64 << 10 : used;
            if (blk > ((size_t)256 << 20)) blk = (size_t)256 << 20;
            extra.emplace_back();
            extra.back().alloc(blk > b ? blk : b);
            extra_off = 0;
        }
        T *p = reinterpret_cast<T *>(static_cast<char *>(extra.back().ptr) + extra_off);
        extra_off += b;
        return p;
    }

  private:
    mm_ctx *ctx;
    size_t off0, used = 0, extra_off = 0;
    std::vector<DBuf> extra;
};

}  // namespace mm

struct mm_pointing {
    int64_t n_samp = 0;
    int32_t n_pix_total = 0;
    int32_t n_obs = 0;
    int64_t n_valid = 0;
    mm_precision prec = MM_F64;
    // map components: IQU (3 per pixel), I (1: weights 1, no angles kept) or
    // QU (2: weights cos 2psi, sin 2psi)
    mm_stokes stokes = MM_STOKES_IQU;
    int32_t nc = 3;
    int64_t n() const { return (int64_t)nc * n_obs; }
    mm::DBuf hits, obs_pix, j, w, perm, ws, off;
    mm::DBuf psi;  // f64[n_samp] angles (FP64 form only)
    // Map copies of the single-column P (with a grid): p_copies copies,
    // one per scan direction found, each ordered by first touch along its
    // samples; p_slot and p_chunk_grp only where P or the sliced P^T takes them,
    // p_j where P does.  p_slot[g n_obs + c] is pixel c's slot in copy g (counted over
    // all copies) and p_j[t] the slot of sample t's pixel in its chunk's copy
    // (-1 flagged), so the pixels a wave gathers along the scan share cache
    // lines.  Without a grid the slot is the compact id and there is one copy.
    mm::DBuf p_slot, p_j;
    int32_t p_copies = 0;
    mm::DBuf p_chunk_grp;  // int32 copy (scan direction) of each 4,096-sample chunk
    // Order in which P^T visits the compact pixels (empty = ascending).  Each
    // pixel's own sum is independent of it; it only shapes cache locality.
    mm::DBuf seg_order;
    int32_t grid_width = 0;
    int32_t p_blocks[7] = {0, 0, 0, 0, 0, 0, 0};  // tuned P grid of several columns per log2(nrhs); 0 = default
    // tuned: visit pixels in seg_order (1) or ascending (0) in the
    // one-wave-per-pixel P^T, per log2(nrhs); -1 = default (seg_order if set)
    int32_t pt_order[7] = {-1, -1, -1, -1, -1, -1, -1};
    // Sliced single-column P^T: observed pixels in slices of 64 (one pixel per
    // lane; neighbours on the map when a grid is set), the samples cut into
    // sl_S equal time segments.  Wave (s, g) walks its lanes' entries of
    // segment s in time order from sl_perm / sl_w, stored interleaved (entry k
    // of lane l at sl_base[s G + g] + 64 k + l, padding t = -1, w = 0).
    // With map copies (grid hint) the slices are cut per scan direction d:
    // lane pixels are virtual ids v = d n_obs + c in copy d's first-touch
    // order, each walking only its pixel's samples of direction d, so sl_G
    // counts sl_D direction blocks of slices and wave (s, g) writes partial
    // map s sl_D + g / (sl_G / sl_D).
    int32_t sl_G = 0, sl_S = 0, sl_D = 1;
    mm::DBuf sl_pix;   // int32[G * 64] compact pixel per lane, -1 past n_obs
    mm::DBuf sl_base;  // int64[G * S + 1] entry offsets, segment-major
    mm::DBuf sl_perm;  // int32 sample index per entry
    mm::DBuf sl_w;     // per entry: psi (FP64 form) or the weights (FP32 form); I: none
};

namespace mm {
// Tables of the FFT N^-1 for one block length.
struct FftTables {
    int32_t n = 0;      // real block length
    int32_t valid = 0;  // valid outputs per block
    DBuf spec;          // per filter: A_k, then W^k B_k / 2, in the kernel's order
    DBuf tw;            // twiddles of the transform's first two passes
    DBuf blocks;        // int64 pairs (first output sample, interval index)
    int64_t n_blocks = 0;
};
}  // namespace mm

struct mm_noise {
    int64_t n_samp = 0;
    int32_t n_int = 0, n_filters = 0, half_bw = 0;
    mm_noise_method method = MM_NOISE_DIRECT;
    mm_precision prec = MM_F64;
    std::vector<int64_t> h_istart;
    std::vector<int32_t> h_fid;
    std::vector<double> h_band;
    mm::DBuf istart, fid, band, band64;
    mm::DBuf band_full;  // direct band: the symmetric filters [n_filters][2 half_bw + 1]
    // direct band: per column count R = 2^li (li = 0..6), the number of
    // tiles in the intervals before each interval, int64[14][n_int + 1]: of N^-1
    // alone, and of A with P inside the band by rows
    // (device copy and host copy); built with the handle, read-only after
    mm::DBuf tile_pref;
    std::vector<int64_t> h_tile_pref;
    int32_t band_cl[7] = {0, 0, 0, 0, 0, 0, 0};  // tuned taps per LDS chunk per log2(nrhs); 0 = default
    bool band_small = false;  // one column in 512-sample tiles of 128 threads (short streams)
    // FFT: per-filter packed spectrum and block table
    int32_t fft_n = 0;       // block length set or reported (mm_noise_fft_block)
    bool fft_auto = false;   // picked by the library: fft.n may be another length
    mm::FftTables fft;       // of the blocks that run
    // polynomial template filter (method MM_NOISE_POLY): subscan table, the
    // weight of each subscan's interval, G_s^-1 per subscan ((p+1)^2 FP64,
    // zeros for a subscan fitted exactly) and the flag mask as bits
    int32_t pf_order = 0;
    int64_t pf_n_sub = 0;
    int64_t pf_max_len = 0;  // longest subscan (picks the apply's register cache)
    mm::DBuf pf_sub, pf_omega, pf_ginv, pf_mask;
    // ground templates (pf_nb bins, 0 = none): each sample's bin, 1 / sum of
    // w per bin, and the bin-sorted samples interleaved per wave
    // (wave w = a chunk of a group of 64 bins: entries [gbase[w], gbase[w+1]),
    // lane = bin; gfirst[g] = first wave of group g)
    int32_t pf_nb = 0;
    int32_t pf_n_gwave = 0;
    int32_t pf_n_gwave512 = 0;  // waves that chunks of 512 entries would make (scratch count)
    mm::DBuf pf_gbin, pf_gwinv, pf_gbase, pf_gfirst, pf_gsp;
};

struct mm_precond {
    int kind = 0;  // 0 = M_BD, 1 = M_2l
    int32_t n_obs = 0;
    int32_t nc = 3;  // map components per pixel (the pointing's)
    int64_t n() const { return (int64_t)nc * n_obs; }
    // f64[n_obs][nc (nc + 1) / 2] packed symmetric B_j^-1: (00, 01, 02, 11,
    // 12, 22) for IQU, (00, 01, 11) for QU, (00) for I; for M_BD also the
    // assembled blocks B_j themselves, packed the same way (M_BD^-1, used to
    // form A Z from the Arnoldi factorisation)
    mm::DBuf inv, blk;
    double rcond_min = 0;
    // M_2l
    int32_t k = 0;
    // Z, AZ: f64[k][n]; E: f64[k][k]; Einv: E^-1, column r at Einv[r k]
    mm::DBuf Z, AZ, E, Einv;
    // Arnoldi record
    int32_t arn_m = 0;
    mm::DBuf W;
    std::vector<double> H;  // (m+1) x m column-major
};

namespace mm {

// ---- launchers (defined in the .hip files) ----
// pointing.hip
void pointing_build_device(mm_ctx *ctx, mm_pointing *p, const int32_t *pix, const double *psi,
                           int32_t min_hits);
// bits(x): the smallest b with x < 2^b.
inline unsigned bits(uint64_t x) {
    unsigned b = 1;
    while (b < 64 && (x >> b) != 0) ++b;
    return b;
}
// Bits of the tile keys (tile number << 24, then the place in the tile) of a row-major
// grid of n_pix pixels.
inline unsigned tile_key_bits(int32_t n_pix, int32_t width, int32_t tile) {
    const int64_t tiles_x = ((int64_t)width + tile - 1) / tile;
    const int64_t tiles_y = (n_pix - 1) / width / tile + 1;
    return 24 + bits((uint64_t)(tiles_x * tiles_y));
}
// Whether the one-column P gathers from map copies: that saves cache lines per sample,
// packing them costs a launch and a pass over copies x n_obs.  It pays from 2^22 samples and 256
// per pixel on (us, copies / x itself, IQU FP64, three directions: 64 x 64 pixels, 2^20
// samples 8.3 / 6.2; 128 x 128, 2^21 14.0 / 12.4, 2^23 38.8 / 43.6; 256 x 256, 2^23 44.7 /
// 42.5, 2^25 138 / 160, 2^27 520 / 632).
inline bool gathers_copies(int64_t n_samp, int32_t n_obs) {
    return n_samp >= (int64_t)1 << 22 && n_samp >= 256 * (int64_t)n_obs;
}
// Whether the sliced P^T (entries with padding: the longest lane of each wave) is taken
// for a pointing of nc components that has waves enough for it: IQU always.  I and QU,
// whose sums read less per sample, only where the lanes of a wave have about equally
// many samples: one wave per pixel and sliced, us, QU FP64, with entries / n_valid:
// 2^23 samples on 128 x 128 pixels, 1.02: 43 and 37, 1.6: 70 and 69 (I 41 and 50), 4.7:
// 104 and 182; on 256 x 256, 1.3: 51 and 57, 4.4: 74 and 242; from 2^24 on z no longer
// stays in the cache: 2^24 on 128 x 128, 1.6: 180 and 114, 4.7: 284 and 301; 2^25 on
// 256 x 256, 1.3: 400 and 216, 4.5: 515 and 783.
inline bool slices_pay(int nc, int64_t n_samp, int64_t n_valid, int64_t entries) {
    if (nc == 3) return true;
    return 5 * entries <= (n_samp >= (int64_t)1 << 24 ? 10 : 6) * n_valid;
}
// (Re)build everything that depends on the grid hint (width 0 = none): the visiting
// order of the one-wave-per-pixel P^T, P's map copies and the sliced P^T layout.
void pointing_layout_device(mm_ctx *ctx, mm_pointing *p, int32_t width);

// tod_ops.hip
// The P and P^T launchers take an optional device scratch region of at least
// *_scratch_bytes(...) bytes (256-byte aligned); with nullptr they use (and grow)
// the context's workspaces instead.
size_t apply_P_scratch_bytes(const mm_pointing *p, int nrhs);
size_t apply_PT_scratch_bytes(const mm_pointing *p, int nrhs);
size_t noise_scratch_bytes(const mm_noise *nz, int nrhs);
void apply_P_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const double *x, void *y,
                 char *scratch = nullptr, bool planar = false);
// Consecutive samples of a wave of the P of several columns, a multiple of step = 256 / R
// (what it takes at a time): step, or what `blocks` blocks of four waves make (blocks >
// 0); more where the launch would pass 2^22 blocks, as one of 2^32 threads is refused.
// From 32 columns on, with a map beyond the L2s (x over 20 MB), runs of 16 steps: a
// wave's gathers then stay among neighbouring pixels, us, step / 16 steps: 1M samples x
// 64, FP32, 128 x 128 pixels (25 MB) 196 / 110, 96 x 96 (14 MB, FP64) 168 / 176, 256 x 256
// (101 MB), sweeps along rows 261 / 152; x 32, (50 MB) 130 / 68; x 16 (25 MB) 51 / 56.
inline int64_t p_wave_samples(int64_t n, int step, int64_t blocks, int64_t map_bytes = 0) {
    if (blocks <= 0 || blocks > (1 << 22)) {
        const bool far = step <= 8 && map_bytes > 20000000 && n >= (int64_t)step << 17;
        const int64_t per = far ? 16 * step : step;
        if ((n + 4 * per - 1) / (4 * per) <= (1 << 22)) return per;
        blocks = 1 << 22;
    }
    const int64_t per = (n + 4 * blocks - 1) / (4 * blocks);
    return (per + step - 1) / step * step;
}
void apply_PT_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const void *z, double *x,
                  char *scratch = nullptr);
// The P^T of a wave or block per pixel: one column per lane, two columns per lane, or
// the latter with four waves per pixel (measured beside k_apply_PT_cols).
enum class PtForm { LANES, COLUMNS, BLOCK };
inline PtForm pt_form(int32_t n_obs, int64_t n_valid, int nrhs, int n_cu) {
    const int64_t work = n_valid * nrhs;  // n_obs h R
    if (nrhs < 8 || work < 256 * (int64_t)n_obs) return PtForm::LANES;
    return n_obs < 8 * (int64_t)n_cu && work >= 4096 * (int64_t)n_obs ? PtForm::BLOCK
                                                                      : PtForm::COLUMNS;
}
void noise_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z);
void mask_tod_dev(mm_ctx *ctx, const mm_pointing *p, int nrhs, const void *tod_rm, void *y,
                  int *nonfinite_flag);
// z = N^-1 (mask . tod) by the FFT method, tod [nrhs][n_samp] masked as it is
// read; *bad = 1 if a kept sample is not finite.
void noise_fft_masked_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, int nrhs,
                          const void *tod, void *z, int *bad);
void pair_sum_diff_dev(mm_ctx *ctx, int64_t n, mm_precision prec, const void *a, const void *b,
                       void *plus, void *minus);
// FFT tables (spectra, twiddles, block table) for overlap-save blocks of
// n_fft real samples (16,384 or 32,768; 0 = pick by the measured time model)
void noise_fft_prepare(mm_ctx *ctx, mm_noise *nz, int n_fft);
// polyfilter.hip
int polyfilter_max_order();
void polyfilter_prepare(mm_ctx *ctx, const mm_pointing *p, mm_noise *nz,
                        const int32_t *ground_bin, int32_t n_ground_bins);
size_t polyfilter_scratch_bytes(const mm_noise *nz, int nrhs);
void polyfilter_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z);
// F P x into one of the two TOD vectors (returned); the other one is free after.
// scratch (ground sums) and map_scratch (apply_P_scratch_bytes; may be ta): NULL =
// the context's workspaces.
const void *polyfilter_apply_P_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz,
                                   int nrhs, const double *x, void *ta, void *tb, char *scratch,
                                   char *map_scratch);
// y = P^T N^-1 P x with the TOD vectors ta and tb.  scratch: at least
// apply_A_scratch_bytes, or NULL to use the context's workspaces.
size_t apply_A_scratch_bytes(const mm_pointing *p, const mm_noise *nz, int nrhs);
void apply_A_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, int nrhs,
                 const double *x, double *y, void *ta, void *tb, char *scratch);
bool noise_fft_supported(int half_bw, int64_t min_len);

// map_ops.hip
void mbd_build_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, mm_precond *M,
                   int *n_bad);
void mbd_apply_dev(mm_ctx *ctx, const double *inv, int32_t n_obs, int nc, int nrhs,
                   const double *v, double *out, const double *dot_with, double *dot_partial,
                   int n_part);
inline int packed_sym(int nc) { return nc * (nc + 1) / 2; }

// Deterministic dot products of columns: out[r] = sum_i a[i R + r] b[i R + r]
// over n rows (two stages, fixed order).
void dot_cols(mm_ctx *ctx, int64_t n, int nrhs, const double *a, const double *b, double *out);
// Blocks of a two-stage column reduction over n_rows x nrhs elements.
int reduction_parts(int64_t n_rows, int nrhs = 1);

// Small dense helpers
void gram_mfma(mm_ctx *ctx, int64_t n, int ka, int kb, const double *X, int64_t x_rs,
               int64_t x_cs, const double *Y, int64_t y_rs, int64_t y_cs, double *C);
void gemv_t(mm_ctx *ctx, int64_t n, int ncol, const double *W, const double *v, double *h);
void gemv_n_sub(mm_ctx *ctx, int64_t n, int ncol, const double *W, const double *h, double *v);
void scale_copy(mm_ctx *ctx, int64_t n, const double *src, const double *s_dev, double *dst,
                int invert);
// U[c n + i] += g[c] r[i] (U column-major n x k; g on the device).
void rank1_add(mm_ctx *ctx, int64_t n, int k, const double *r, const double *g, double *U);
void matmul_small_right(mm_ctx *ctx, int64_t n, int kin, int kout, const double *V,
                        const double *Y, double *Zout);  // Zout = V Y, col-major
// Cholesky factor Lc of the k x k matrix E; E is symmetrised in place first.
void chol_small_dev(mm_ctx *ctx, int k, double *E, double *Lc, int *flag);
// E^-1 (column r at Einv[r k]) from the lower Cholesky factor Lc of E.
void coarse_inverse_dev(mm_ctx *ctx, int k, const double *Lc, double *Einv);
void m2l_apply_dev(mm_ctx *ctx, const mm_precond *M, int nrhs, const double *v, double *out,
                   double *dot_partial, int n_part);
void m2l_coef_dev(mm_ctx *ctx, const mm_precond *M, int nrhs, const double *v, double *c);

// PCG vector kernels on column-batched map vectors
struct PcgDev {
    double *rho, *pq, *alpha, *beta, *rn2, *bn2, *tol2;
    int *done, *brk, *iters;
    double *hist;   // rn2 per iteration, [hist_len][R], or null
    int hist_len;
    double *rzo;    // flexible beta: r'.z_old per column, or null (beta = rho'/rho)
};
void pcg_init_scalars(mm_ctx *ctx, int nrhs, PcgDev s, double tol);
void axpby_cols(mm_ctx *ctx, int64_t n, int nrhs, const double *b, const double *Ax, double *r);
// alpha from the p.q partials, then x += alpha p, r -= alpha q with the
// ||r||^2 partials (into a buffer other than pq_part)
void pcg_update_xr(mm_ctx *ctx, int64_t n, int nrhs, PcgDev s, const double *pq_part,
                   const double *p, const double *q, double *x, double *r, double *partial,
                   int n_part);
// The same with z = M r of an M_BD and its r.z partials (into a buffer other than pq_part).
void pcg_update_xrz(mm_ctx *ctx, const mm_precond *M, int nrhs, PcgDev s, const double *pq_part,
                    const double *p, const double *q, double *x, double *r, double *z,
                    double *part_rn, double *part_rz, int n_part);
// breakdown flag, iteration count and convergence from ||r||^2, then rho', beta
void pcg_after_rnrz(mm_ctx *ctx, int nrhs, PcgDev s, const double *part_rn,
                    const double *part_rz, int n_part);
void pcg_after_rn(mm_ctx *ctx, int nrhs, PcgDev s, const double *partial, int n_part,
                  int count_iter);
void pcg_after_rz(mm_ctx *ctx, int nrhs, PcgDev s, const double *partial, int n_part, int init);
// s.rzo[r] = sum of the column's partial dot products (flexible beta)
void pcg_store_rzo(mm_ctx *ctx, int nrhs, PcgDev s, const double *partial, int n_part);
void pcg_update_p(mm_ctx *ctx, int64_t n, int nrhs, PcgDev s, const double *z, double *p);
void dot_partial_cols(mm_ctx *ctx, int64_t n, int nrhs, const double *a, const double *b,
                      double *partial, int n_part);
void col_set(mm_ctx *ctx, int64_t n, int R, int slot, const double *src, double *dst);
void gemm_rows_small(mm_ctx *ctx, int64_t n, int R, const double *In, const double *S,
                     double alpha, double beta, double *Out);
void chol_inv_drop(mm_ctx *ctx, int R, const double *G, double tau, double *U, int *rank);
void col_get(mm_ctx *ctx, int64_t n, int R, int slot, const double *src, double *dst);
// dst (k columns over the n_dst_obs pixels obs_dst) = src's rows of the same
// global pixels (k columns over obs_src), 0 where obs_src lacks the pixel
void transfer_rows(mm_ctx *ctx, int32_t n_dst_obs, const int32_t *obs_dst, int32_t n_src_obs,
                   const int32_t *obs_src, int nc, int k, const double *src, double *dst);
void slot_ctl(mm_ctx *ctx, PcgDev s, int slot, int mode, double tol);
void copy_cols_masked(mm_ctx *ctx, int64_t n, int nrhs, const int *done, const double *src,
                      double *dst);

// host
void hessenberg_eig(int m, const double *H, double *wr, double *wi, double *vr, double *vi);
// Eigen-decomposition of a small symmetric matrix (cyclic Jacobi rotations):
// A (n x n, row-major) is destroyed; w = eigenvalues, U column j = vector j.
void sym_eig_jacobi(int n, std::vector<double> &A, std::vector<double> &w, std::vector<double> &U);

template <typename T> struct Vec2T;
template <> struct Vec2T<float> { using type = float2; };
template <> struct Vec2T<double> { using type = double2; };

void build_band_tiles(mm_ctx *ctx, mm_noise *nz);
void autotune(mm_ctx *ctx, mm_pointing *p, mm_noise *nz, int nrhs, int flags, double *report,
              int *n_report, int max_report);

inline int log2i(int r) { int l = 0; while ((1 << l) < r) ++l; return l; }
inline int pow2_ok(int r) { return r >= 1 && r <= 64 && (r & (r - 1)) == 0; }

}  // namespace mm

// Error handling at the C-ABI boundary: an mm::Error (or a host allocation
// failure) inside API_BEGIN(ctx) ... API_END becomes the call's status and the
// context's last-error message.
#define API_BEGIN(ctxp)                                   \
    mm_ctx *api_ctx_ = (ctxp);                            \
    try {                                                 \
        if (api_ctx_) {                                   \
            api_ctx_->last_error.clear();                 \
            MM_HIP(hipSetDevice(api_ctx_->device));       \
        }

#define API_END                                                            \
    }                                                                      \
    catch (const mm::Error &e) {                                           \
        if (api_ctx_) api_ctx_->last_error = e.what();                     \
        return e.code;                                                     \
    }                                                                      \
    catch (const std::bad_alloc &) {                                       \
        if (api_ctx_) api_ctx_->last_error = "host allocation failed";     \
        return MM_E_OOM;                                                   \
    }                                                                      \
    catch (const std::exception &e) {                                      \
        if (api_ctx_) api_ctx_->last_error = e.what();                     \
        return MM_E_DEVICE;                                                \
    }

namespace mm {
// Looks up, once per device and with that device current, the device address
// of the static scratch array of mm_apply_A_noalloc (called at context
// creation).
void noalloc_init(int device);
}  // namespace mm

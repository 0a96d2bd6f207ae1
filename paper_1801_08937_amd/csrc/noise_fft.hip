// N^-1 by FFT: overlap-save convolution per stationary interval -- the
// spectrum tables, the block table and the choice of block size.  The
// transforms run in noise_fft_big.hip (register-resident kernels for 16,384-
// and 32,768-sample blocks).
//
// For an interval [a, e) with half bandwidth lambda, the outputs
// t in [t0, t0 + V) need the inputs u in [t0 - lambda, t0 - lambda + N)
// (zero outside the interval), N = 2 NC real samples, V = N - 2 lambda.  A
// circular convolution of length N with the symmetric kernel
// h = (c_0, c_1 .. c_lambda, 0 .., c_lambda .. c_1) is then exact on those V
// outputs: no wrapped-around term reaches them.  The banded matrix is never
// formed; its spectrum H_k = c_0 + 2 sum_d c_d cos(2 pi k d / N) is real.
//
// The N real inputs of a block are packed as NC complex values
// z_m = y_{2m} + i y_{2m+1}, transformed by an NC-point complex FFT,
// multiplied by the spectrum in the packed domain
//     Z'_k = A_k Z_k + B_k (W^k O_k + i W^-k E_k),
//     E_k = (Z_k + conj Z_{NC-k}) / 2,  O_k = (Z_k - conj Z_{NC-k}) / 2i,
//     A_k = (H_k + H_{k+NC}) / 2NC,     B_k = (H_k - H_{k+NC}) / 2NC,  W = e^{-2 pi i / N},
// and transformed back; the real and imaginary parts of the result are the
// even and odd outputs.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "fft_common.h"

namespace mm {
namespace {

// H_k = c_0 + 2 sum_d c_d cos(2 pi k d / N) for k in [0, N/2], in two steps with
// d = d1 + 64 d2:
//   S_{d1, m} = sum_{d2} c_{d1 + 64 d2} W^(64 m d2),  m = k mod N/64  (c_0 halved),
//   H_k = 2 Re sum_{d1} W^(k d1) S_{d1, k mod N/64},  W = e^{-2 pi i / N}.
// lambda / 64 + 64 terms per value instead of lambda (32 filters of lambda 2,048:
// 720 -> 72 us).  The cosines come from a quarter-period table (integer angles
// reduced mod N and folded by symmetry), so every angle is exact.
constexpr int QMAX = 8192;  // N/4 for the largest block
constexpr int SP_B = 64;    // values of d1

__device__ __forceinline__ double2 quarter_cs(const double *__restrict__ q, int m, int N) {
    // (cos, sin)(2 pi m / N), 0 <= m < N, from cos(2 pi i / N), i <= N / 4
    const int Q = N / 4, h = m & (Q - 1);
    const double a = q[h], b = q[Q - h];
    switch (m / Q) {
        case 0: return make_double2(a, b);
        case 1: return make_double2(-b, a);
        case 2: return make_double2(-a, -b);
        default: return make_double2(b, -a);
    }
}

__global__ void __launch_bounds__(256)
    k_spec_sub(const double *__restrict__ band, int lam, int N, const double *__restrict__ qtab,
               double2 *__restrict__ S) {
    __shared__ double2 cs[2 * QMAX / 32];  // W^(64 m), m < N / 64
    const int NB = N / SP_B;
    for (int m = threadIdx.x; m < NB; m += 256) cs[m] = quarter_cs(qtab, SP_B * m, N);
    __syncthreads();
    const int f = blockIdx.z, d1 = blockIdx.y, m = blockIdx.x * 256 + threadIdx.x;
    if (m >= NB) return;
    const double *c = band + (int64_t)f * (lam + 1);
    double sr = 0, si = 0;
    for (int d = d1, d2 = 0; d <= lam; d += SP_B, ++d2) {
        const double2 w = cs[(m * d2) & (NB - 1)];
        const double v = d == 0 ? 0.5 * c[0] : c[d];
        sr += v * w.x;
        si -= v * w.y;
    }
    S[((int64_t)f * SP_B + d1) * NB + m] = make_double2(sr, si);
}

__global__ void __launch_bounds__(256)
    k_spec_sum(int N, const double *__restrict__ qtab, const double2 *__restrict__ S,
               double *__restrict__ H) {
    __shared__ double q[QMAX + 1];
    for (int m = threadIdx.x; m <= N / 4; m += 256) q[m] = qtab[m];
    __syncthreads();
    const int NC = N / 2, NB = N / SP_B, f = blockIdx.y;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k > NC) return;
    const double2 *s = S + (int64_t)f * SP_B * NB + (k & (NB - 1));
    double h = 0;
#pragma unroll 8
    for (int d1 = 0; d1 < SP_B; ++d1) {
        const double2 v = s[(int64_t)d1 * NB];
        const double2 w = quarter_cs(q, (k * d1) & (N - 1), N);
        h += w.x * v.x + w.y * v.y;
    }
    H[(int64_t)f * (NC + 1) + k] = 2.0 * h;
}

}  // namespace

bool noise_fft_big_supported(int half_bw);
bool noise_fft_mid_supported(int half_bw);
int noise_fft_big_nc();
int noise_fft_mid_nc();
int noise_fft_short_nc();
bool noise_fft_short_supported(int half_bw);
void noise_fft_tables_dev(mm_ctx *ctx, const mm_noise *nz, FftTables &tb, const double *H,
                          const double *qtab);
void noise_fft_reg_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z,
                             bool planar, const int32_t *jpix, int *bad);

bool noise_fft_supported(int half_bw, int64_t min_len) {
    (void)min_len;
    return half_bw >= 1 && noise_fft_big_supported(half_bw);
}

static int64_t fft_n_blocks(const mm_noise *nz, int N) {
    const int64_t V = N - 2 * (int64_t)nz->half_bw;
    int64_t nb = 0;
    for (int i = 0; i < nz->n_int; ++i)
        nb += (nz->h_istart[i + 1] - nz->h_istart[i] + V - 1) / V;
    return nb;
}

// The length that mm_noise_fft_block reports where the library picks (the pick of the
// two larger lengths; fft_run_model picks what runs): rounds of n_cu x (blocks per CU) blocks, 40
// (16,384) or 42 (32,768) time units each.
static double fft_time_model(const mm_noise *nz, int N, int n_cu) {
    if (N <= 2 * nz->half_bw) return 1e300;
    const bool mid = N == 2 * noise_fft_mid_nc();
    const int64_t per_wave = (int64_t)n_cu * (mid ? 2 : 1) * (nz->prec == MM_F32 ? 2 : 1);
    return (double)((fft_n_blocks(nz, N) + per_wave - 1) / per_wave) * (mid ? 40.0 : 42.0);
}

// The length that runs: 8,192-, 16,384- and 32,768-sample blocks share a CU by four,
// two and one (FP64; FP32 about 0.6 of these times, in the same proportions).
// Measured, us (one column): up to one block per CU 11.5, 14 to 20 and 25 to 33; 2, 3
// and 4 of the small ones 17, 23 and 27, two of the middle ones 29; longer streams 22.5,
// 27 and 33 per round and a quarter of one more.  2^20 samples, lambda 1,024: 11.4,
// 16.0, 26.6; 2^23: 38, 42, 59; 2^26: 255, 298, 391 (lambda 2,048: 361, 333, 400;
// 4,096: -, 423, 419).  With more than three times the blocks, the small ones lose on
// several columns what they gain on one (2^20 samples, lambda 3,072, 4 columns: 62
// against 48 us).
static double fft_run_model(const mm_noise *nz, int N, int n_cu) {
    const double nb = (double)fft_n_blocks(nz, N) / n_cu;
    if (N == 2 * noise_fft_short_nc()) {
        if (nb <= 4) return nb <= 1 ? 11.5 : nb <= 2 ? 17 : nb <= 3 ? 23 : 27;
        return 22.5 * (nb / 4 + 0.25);
    }
    if (N == 2 * noise_fft_mid_nc()) {
        if (nb <= 2) return nb <= 1 ? 14 + 6 * nb : 29;
        return 27 * (nb / 2 + 0.25);
    }
    return nb <= 1 ? 25 + 8 * nb : 33 * (nb + 0.25);
}

static int fft_run_length(const mm_noise *nz, int n_cu) {
    const int ns = 2 * noise_fft_short_nc(), nm = 2 * noise_fft_mid_nc();
    int best = 2 * noise_fft_big_nc();
    if (!noise_fft_mid_supported(nz->half_bw)) return best;
    if (fft_run_model(nz, nm, n_cu) <= fft_run_model(nz, best, n_cu)) best = nm;
    if (noise_fft_short_supported(nz->half_bw) &&
        fft_n_blocks(nz, ns) <= 3 * fft_n_blocks(nz, nm) &&
        fft_run_model(nz, ns, n_cu) <= fft_run_model(nz, best, n_cu))
        best = ns;
    return best;
}

// Spectra, twiddles and block list for blocks of N real samples.
static void fft_tables(mm_ctx *ctx, const mm_noise *nz, FftTables &tb, int N) {
    hipStream_t s = ctx->stream;
    const int lam = nz->half_bw, NC = N / 2;
    tb.n_blocks = 0;  // until the tables are whole: a failure on the way leaves none
    tb.n = N;
    tb.valid = N - 2 * lam;
    // quarter period of cos(2 pi m / N) (long double on the host, rounded once)
    std::vector<double> qtab(N / 4 + 1);
    const long double pi2 = 6.283185307179586476925286766559L;
    for (int m = 0; m <= N / 4; ++m) qtab[m] = (double)cosl(pi2 * m / N);
    // spectra
    Scratch sc(ctx);
    double *dq = sc.get<double>((int64_t)qtab.size());
    double *H = sc.get<double>((int64_t)nz->n_filters * (NC + 1));
    MM_HIP(hipMemcpyAsync(dq, qtab.data(), sizeof(double) * qtab.size(), hipMemcpyHostToDevice,
                          s));
    // 256 filters at a time: their S is 32 to 128 MiB, which the next ones use again
    const unsigned nf = (unsigned)nz->n_filters, step = std::min(nf, 256u);
    double2 *S = sc.get<double2>((int64_t)step * N);
    for (unsigned f0 = 0; f0 < nf; f0 += step) {
        const unsigned cnt = std::min(nf - f0, step);
        k_spec_sub<<<dim3((N / SP_B + 255) / 256, SP_B, cnt), 256, 0, s>>>(
            nz->band64.as<double>() + (int64_t)f0 * (lam + 1), lam, N, dq, S);
        k_spec_sum<<<dim3((NC + 1 + 255) / 256, cnt), 256, 0, s>>>(
            N, dq, S, H + (int64_t)f0 * (NC + 1));
    }
    MM_HIP(hipGetLastError());
    noise_fft_tables_dev(ctx, nz, tb, H, dq);
    // block table
    std::vector<int64_t> blocks;
    for (int i = 0; i < nz->n_int; ++i)
        for (int64_t t = nz->h_istart[i]; t < nz->h_istart[i + 1]; t += tb.valid) {
            blocks.push_back(t);
            blocks.push_back(i);
        }
    tb.blocks.alloc(sizeof(int64_t) * blocks.size());
    MM_HIP(hipMemcpyAsync(tb.blocks.ptr, blocks.data(), sizeof(int64_t) * blocks.size(),
                          hipMemcpyHostToDevice, s));
    MM_HIP(hipStreamSynchronize(s));
    tb.n_blocks = (int64_t)blocks.size() / 2;
}

// Tables for blocks of n_fft real samples (0 = pick by the models above).
void noise_fft_prepare(mm_ctx *ctx, mm_noise *nz, int n_fft) {
    const int lam = nz->half_bw;
    MM_CHECK(noise_fft_supported(lam, 0), MM_E_INVALID, "FFT: bandwidth unsupported");
    const int ns = 2 * noise_fft_short_nc(), nm = 2 * noise_fft_mid_nc();
    const int nb = 2 * noise_fft_big_nc();
    MM_CHECK(n_fft == 0 || n_fft == nb || (n_fft == nm && noise_fft_mid_supported(lam)) ||
                 (n_fft == ns && noise_fft_short_supported(lam)),
             MM_E_INVALID,
             "FFT: block length must be 8,192 (lambda <= 3,072), 16,384 (lambda <= 6,144) or "
             "32,768");
    int run = n_fft, shown = n_fft;
    if (n_fft == 0) {
        run = fft_run_length(nz, ctx->n_cu);
        shown = noise_fft_mid_supported(lam) &&
                        fft_time_model(nz, nm, ctx->n_cu) <= fft_time_model(nz, nb, ctx->n_cu)
                    ? nm
                    : nb;
    }
    fft_tables(ctx, nz, nz->fft, run);
    nz->fft_n = shown;
    nz->fft_auto = n_fft == 0;
}

void noise_fft_apply_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z) {
    noise_fft_reg_apply_dev(ctx, nz, nrhs, y, z, false, nullptr, nullptr);
}

// y column after column, [R][n]; z interleaved.
void noise_fft_planar_dev(mm_ctx *ctx, const mm_noise *nz, int nrhs, const void *y, void *z) {
    noise_fft_reg_apply_dev(ctx, nz, nrhs, y, z, true, nullptr, nullptr);
}

void noise_fft_masked_dev(mm_ctx *ctx, const mm_pointing *p, const mm_noise *nz, int nrhs,
                          const void *tod, void *z, int *bad) {
    noise_fft_reg_apply_dev(ctx, nz, nrhs, tod, z, true, p->j.as<int32_t>(), bad);
}


}  // namespace mm

// The pointing row of a sample as the one-column kernels read it: the map gathered
// at the sample's slot and the weights (1, cos 2psi, sin 2psi) of Eq. datamodel.
#pragma once

#include "mm_internal.h"
#include "pol_weights.h"

namespace mm {

template <typename T> struct Vec2;
template <> struct Vec2<float> { using type = float2; };
template <> struct Vec2<double> { using type = double2; };

// A once-read stream element loaded with the non-temporal cache policy: a
// double, or a float2 moved as one 64-bit word.
__device__ __forceinline__ double nt_load_w(const double *p) {
    return __builtin_nontemporal_load(p);
}
__device__ __forceinline__ float2 nt_load_w(const float2 *p) {
    return __builtin_bit_cast(
        float2, __builtin_nontemporal_load(reinterpret_cast<const unsigned long long *>(p)));
}
__device__ __forceinline__ double2 nt_load_w(const double2 *p) { return *p; }

// Weight record of an entry: FP64 stores the angle and forms the weights
// here; FP32 stores the two weights.
template <typename T> struct SlRec;
template <> struct SlRec<double> {
    using type = double;
    __device__ static void weights(double psi, double &c, double &s) { pol_weights(psi, c, s); }
};
template <> struct SlRec<float> {
    using type = float2;
    __device__ static void weights(float2 w, float &c, float &s) {
        c = w.x;
        s = w.y;
    }
};

// The map as the one-column P gathers it (p_map_dev).
enum { PK_I = 1, PK_QU = 2, PK_IQU = 3, PK_PACKED = 4 };
struct PMap {
    int kind;             // PK_I, PK_QU, PK_IQU: NC values per slot at xm; PK_PACKED: below
    const int32_t *slot;  // of each sample, -1 unobserved
    const void *w;        // weight record of each sample (not for PK_I)
    const double *xm;     // PK_PACKED FP64: I per slot
    const double2 *xq;    // PK_PACKED FP64: (Q, U) per slot; FP32: records (I, Q), (U, 0)
};

// The values P x of N samples, one column: slots and weights, read once and so
// non-temporally (they do not push the gathered map lines out of the L2), then all
// gathers (from slot 0 where the sample is unobserved, so that none waits behind
// a branch), then the products.  get: samples t[q]; get_pair: t0 (even) and t0 + 1,
// each stream read in one access.
template <typename T, int KIND> struct PSrc {
    using W = typename SlRec<T>::type;
    const int32_t *__restrict__ slot;
    const W *__restrict__ w;
    const double *__restrict__ xm;
    const double2 *__restrict__ xq;
    __host__ explicit PSrc(const PMap &m)
        : slot(m.slot), w(static_cast<const W *>(m.w)), xm(m.xm), xq(m.xq) {}
    template <int N>
    __device__ __forceinline__ void values(const int32_t (&j)[N], const W (&ww)[N],
                                           T (&v)[N]) const {
        double x0[N], x1[N], x2[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int64_t jj = j[q] < 0 ? 0 : j[q];
            if constexpr (KIND == PK_I) {
                x0[q] = xm[jj];
            } else if constexpr (KIND == PK_QU) {
                x1[q] = xm[2 * jj];
                x2[q] = xm[2 * jj + 1];
            } else if constexpr (KIND == PK_IQU) {
                x0[q] = xm[3 * jj];
                x1[q] = xm[3 * jj + 1];
                x2[q] = xm[3 * jj + 2];
            } else if constexpr (sizeof(T) == 8) {
                const double2 qu = xq[jj];
                x0[q] = xm[jj];
                x1[q] = qu.x;
                x2[q] = qu.y;
            } else {
                const double2 iq = xq[2 * jj];
                x0[q] = iq.x;
                x1[q] = iq.y;
                x2[q] = xq[2 * jj + 1].x;
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            T r;
            if constexpr (KIND == PK_I) {
                r = (T)x0[q];
            } else {
                T c, s;
                SlRec<T>::weights(ww[q], c, s);
                if constexpr (KIND == PK_QU) r = c * (T)x1[q] + s * (T)x2[q];
                else r = (T)x0[q] + c * (T)x1[q] + s * (T)x2[q];
            }
            v[q] = j[q] < 0 ? (T)0 : r;
        }
    }
    template <int N> __device__ __forceinline__ void get(const int64_t (&t)[N], T (&v)[N]) const {
        int32_t j[N];
        W ww[N]{};
#pragma unroll
        for (int q = 0; q < N; ++q) {
            j[q] = __builtin_nontemporal_load(slot + t[q]);
            if constexpr (KIND != PK_I) ww[q] = nt_load_w(w + t[q]);
        }
        values(j, ww, v);
    }
    __device__ __forceinline__ void get_pair(int64_t t0, T (&v)[2]) const {
        // W is 8 bytes in both precisions
        typedef int i2 __attribute__((ext_vector_type(2)));
        typedef unsigned long long w2 __attribute__((ext_vector_type(2)));
        const i2 jj = __builtin_nontemporal_load(reinterpret_cast<const i2 *>(slot + t0));
        const int32_t j[2] = {jj.x, jj.y};
        W ww[2]{};
        if constexpr (KIND != PK_I) {
            const w2 u = __builtin_nontemporal_load(reinterpret_cast<const w2 *>(w + t0));
            ww[0] = __builtin_bit_cast(W, (unsigned long long)u.x);
            ww[1] = __builtin_bit_cast(W, (unsigned long long)u.y);
        }
        values(j, ww, v);
    }
};

// f(PSrc) of the map's kind.
template <typename T, typename F> void dispatch_src(const PMap &m, F &&f) {
    switch (m.kind) {
        case PK_I: f(PSrc<T, PK_I>(m)); break;
        case PK_QU: f(PSrc<T, PK_QU>(m)); break;
        case PK_IQU: f(PSrc<T, PK_IQU>(m)); break;
        default: f(PSrc<T, PK_PACKED>(m));
    }
}

// The gather map of x for the one-column P: copies per scan direction packed into
// scratch (at least apply_P_scratch_bytes; NULL = the context's workspace) where
// the pointing has them and is long enough to repay the launch, else x itself.
PMap p_map_dev(mm_ctx *ctx, const mm_pointing *p, const double *x, char *scratch);

}  // namespace mm

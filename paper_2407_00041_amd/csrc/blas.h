// Solver vector kernels (internal).
#pragma once

#include "common.h"

namespace wd {

constexpr int kGS = 32;           // basis vectors per FP64 update pass (a restart-30 step in one pass)
constexpr int kMdot = 8;          // basis vectors per FP64 inner-product pass (8 accumulators keep occupancy)
constexpr int kGSSite = 8;        // basis vectors per pass of the per-site (low-precision) kernels
constexpr int kRedThreads = 256;  // threads per reduction work-group
constexpr int kRedBlocks = 1024;  // reduction work-groups (fixed: deterministic sums)

struct VecList {
    const void *v[kGS];
    int n;
};

// host-side coefficients travel as kernel arguments (no host-to-device copy)
struct CoefList {
    double2 c[kGS];
};
struct ScaleList {
    double s[kGS];
};
// Sums of ND doubles per thread over the work-group: thread i < ND returns the i-th sum.  The lanes of a wave halve
// their values between them at every step (lane i keeps one half, its partner the other), 21 exchanges for 18 values
// instead of 108 of a full butterfly each; the waves meet in lds ([waves][ND]).  Fixed order.
// `index` of the lane's value and how many of the lane's set exist (0: padding of an odd split).
template <int ND, int OFF>
__device__ __forceinline__ double lane_sums(const double (&v)[ND], int &index, int &count) {
    if constexpr (OFF == 0) {
        return v[0];
    } else if constexpr (ND == 1) {
        const double h[1] = {v[0] + __shfl_xor(v[0], OFF, 64)};
        return lane_sums<1, OFF / 2>(h, index, count);
    } else {
        constexpr int H = (ND + 1) / 2;
        const bool up = (threadIdx.x & OFF) != 0;
        double h[H];
#pragma unroll
        for (int i = 0; i < H; i++) {
            const double lo = v[i], hi = i + H < ND ? v[i + H < ND ? i + H : 0] : 0.0;
            h[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, OFF, 64);
        }
        index += up ? H : 0;
        count = up ? count - H : (count < H ? count : H);
        return lane_sums<H, OFF / 2>(h, index, count);
    }
}
template <int ND> __device__ __forceinline__ double group_sums(const double (&v)[ND], double *lds) {
    static_assert(ND <= 64, "one value per lane at the end");
    int index = 0, count = ND;
    const double s = lane_sums<ND, 32>(v, index, count);
    if (count > 0) lds[(threadIdx.x >> 6) * ND + index] = s;  // lanes of equal index hold equal sums
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < ND)
        for (int w = 0; w < (int)(blockDim.x >> 6); w++) t += lds[w * ND + threadIdx.x];
    return t;
}

// work-group chunks of the all-vector inner products: partial needs
// kMdotChunks * ceil(min(nv, kGS) / kMdot) * (kMdot + 1) entries
constexpr int kMdotChunks = kRedBlocks;


// out[i] = <v_i, w> = v_i^H w for i < nv, out[nv].x = |w|^2, in one launch per
// kGS vectors (w read about once from HBM, see k_mdot_all); partial as
// documented at kMdotChunks.  Optional: scaled[i] = cscale[i] out[i] (cscale on
// the host), and host[i] = out[i] (host memory the device can write, valid once
// the stream is synchronised).  S = double2 (FP64 storage).
template <typename S>
hipError_t mdot_all(const void *const *v, int nv, const void *w, long long N, double2 *partial, double2 *out,
                    hipStream_t st, const double *cscale = nullptr, double2 *scaled = nullptr,
                    double2 *host = nullptr);
// w -= sum_i coef[i] v_i (coef on the device); norm_out[0].x = |w_new|^2 when
// norm_out != null, and host[0].x too when host != null.  partial needs
// kRedBlocks entries
template <typename S>
hipError_t axpy_multi(const void *const *v, int nv, const double2 *coef, void *w, long long N, double2 *partial,
                      double2 *norm_out, hipStream_t st, double2 *host = nullptr);
// out = in * s * mult, s = sc[0].x or 1/sqrt(sc[0].x) (1 for null sc);
// SI == SO == double2 (flat element order)
template <typename SI, typename SO>
hipError_t scale(const void *in, void *out, const double2 *sc, bool inv_sqrt, double mult, long long N,
                 hipStream_t st);
// r = b - w; norm_out[0].x = |r|^2, and host[0].x too when host != null
hipError_t residual(const double2 *b, const double2 *w, double2 *r, long long N, double2 *partial, double2 *norm_out,
                    hipStream_t st, double2 *host = nullptr);
// x += sum_i coef[i] z_i (same precision: S = double2); coef is HOST memory
template <typename S>
hipError_t update(const void *const *z, int nz, const double2 *coef, double2 *x, long long N, hipStream_t st);

// Per-site operations on native fields of precision prec (WDIRAC_F64, _F32 or
// _F16S) for several right-hand sides in one launch (blockIdx.y), FP64
// accumulation; results re-encoded in the field's precision, in passes of
// kGSSite vectors.  hdr is the device header of an inner cycle: hdr[0] =
// (completed steps, active flag), hdr[1].x = normalisation factor; with
// hdr[0].y == 0 the kernels of mdot and axpy do nothing.
struct SiteItem {
    const void *const *v;  // host array of vectors
    void *w;
    double2 *partial;
    const double2 *coef;  // device
    const double2 *hdr;
};
// work-groups per right-hand side of mdot and axpy (rows of their partials)
int site_groups(int V);
// partial[row][i] = part of v_i^H w (i < nv), partial[row][nv].x of |w|^2, rows of nv + 1 entries
hipError_t site_mdot(int prec, const SiteItem *items, int n, int nv, int V, hipStream_t st);
// w = f (w - sum_i coef[i] v_i), f = hdr[1].x; partial[row].x = part of |w_new|^2 (before re-encoding)
hipError_t site_axpy(int prec, const SiteItem *items, int n, int nv, int V, hipStream_t st);
// out (precision pout) = in (precision pin) * mult; pin == pout or pin = F64
hipError_t site_scale(int pin, int pout, const void *in, void *out, double mult, int V, hipStream_t st);
// w (native FP64) = sum_{i < n} coef[i] v_i with n = hdr[0].x <= nmax, v_i of precision prec (w overwritten; n = 0
// gives w = 0)
hipError_t site_combine(int prec, const SiteItem *items, int n, int nmax, int V, hipStream_t st);

}  // namespace wd

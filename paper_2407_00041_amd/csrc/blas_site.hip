// Krylov vector kernels on native fields of any storage precision (FP64,
// FP32, FP16 with a per-site scale), one thread per lattice site: a site's
// 12 complex components are decoded with the stencil's own loaders, every sum
// is accumulated in FP64, and results are re-encoded with the stencil's
// stores (FP16S: a fresh per-site scale).  With these the inner GMRES of the
// mixed solver keeps its Krylov basis in the low-precision operator's layout,
// so the operator reads and writes basis vectors directly.
//
// The kernels can follow a device-side state header hdr of the inner cycle
// (hdr[0] = (completed steps, active flag), hdr[1].x = normalisation factor):
// they return at once for a right-hand side whose cycle has ended, and take
// their coefficients from device memory, so a whole cycle can be issued
// without host decisions (and captured as a graph).
//
// Reductions are deterministic: a fixed grid of at most kRedBlocks work-groups
// per right-hand side, each thread summing a fixed strided subset of sites,
// group_sums per work-group; the inner cycle's state kernels add the per-group
// partials in a fixed order.
#include "blas.h"
#include "spinor_io.h"

namespace wd {

namespace {

template <int P> struct SiteIO {
    using T = typename Store<P>::T;
    static __device__ __forceinline__ void load(const void *f, int V, int s, double2 v[12]) {
        cx<T> a[12];
        Store<P>::load_spinor(f, V, s, a);
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = make_double2((double)a[k].r, (double)a[k].i);
    }
    static __device__ __forceinline__ void store(void *f, int V, int s, const double2 v[12]) {
        cx<T> a[12];
#pragma unroll
        for (int k = 0; k < 12; k++) a[k] = {(T)v[k].x, (T)v[k].y};
        Store<P>::store_spinor(f, V, s, a);
    }
};

// the kernels' right-hand sides (blockIdx.y) and one pass of their vectors
constexpr int kSiteBatch = 16;
struct SiteRhs {
    const void *v[kGSSite];
    void *w;
    double2 *partial;
    const double2 *coef, *hdr;
};
struct SiteBatch {
    SiteRhs r[kSiteBatch];
};

}  // namespace

// columns i0 .. i0 + n of the partials (rows of nv + 1): sums of v_i^H w over the group's sites, with the last pass
// (NORM) |w|^2 in column nv
template <int P, int N, bool NORM>
__global__ __launch_bounds__(kRedThreads) void k_site_mdot(SiteBatch b, int i0, int nv, int V) {
    const SiteRhs &q = b.r[blockIdx.y];
    if (q.hdr[0].y == 0.0) return;
    constexpr int ND = 2 * N + (NORM ? 1 : 0);
    __shared__ double lds[kRedThreads / 64 * ND];
    double acc[ND];
#pragma unroll
    for (int i = 0; i < ND; i++) acc[i] = 0.0;
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < V; s += gridDim.x * blockDim.x) {
        double2 wv[12];
        SiteIO<P>::load(q.w, V, s, wv);
        if constexpr (NORM) {
#pragma unroll
            for (int k = 0; k < 12; k++) acc[2 * N] += wv[k].x * wv[k].x + wv[k].y * wv[k].y;
        }
#pragma unroll
        for (int i = 0; i < N; i++) {
            double2 vv[12];
            SiteIO<P>::load(q.v[i], V, s, vv);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                acc[2 * i] += vv[k].x * wv[k].x + vv[k].y * wv[k].y;
                acc[2 * i + 1] += vv[k].x * wv[k].y - vv[k].y * wv[k].x;
            }
            // one vector's loads behind the last one's sums: 48^3 x 96 FP16S 706 -> 568 us per pass (every two: 634);
            // without it whole mixed solves from 8^4 to 48 x 24^3 are 1-8 % slower at FP16S, 0-4 % at FP32
            asm volatile("" : "+v"(acc[2 * i]), "+v"(acc[2 * i + 1]) : : "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const double t = group_sums(acc, lds);
    if (threadIdx.x < ND) reinterpret_cast<double *>(q.partial + (size_t)blockIdx.x * (nv + 1) + i0)[threadIdx.x] = t;
}

// w = f (w - sum_i coef[i] v_i), coefficients on the device; f = hdr[1].x with the last pass, else 1, which also
// leaves partial[blk] = |w_new|^2 of the re-encoded values' source (before rounding)
template <int P, int N>
__global__ __launch_bounds__(kRedThreads) void k_site_axpy(SiteBatch b, int i0, int last, int V) {
    const SiteRhs &q = b.r[blockIdx.y];
    if (q.hdr[0].y == 0.0) return;
    __shared__ double lds[kRedThreads / 64];
    const double f = last ? q.hdr[1].x : 1.0;
    double nrm[1] = {0.0};
    double2 c[N];
#pragma unroll
    for (int i = 0; i < N; i++) c[i] = q.coef[i0 + i];
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < V; s += gridDim.x * blockDim.x) {
        double2 wv[12];
        SiteIO<P>::load(q.w, V, s, wv);
#pragma unroll
        for (int i = 0; i < N; i++) {
            double2 vv[12];
            SiteIO<P>::load(q.v[i], V, s, vv);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                wv[k].x -= c[i].x * vv[k].x - c[i].y * vv[k].y;
                wv[k].y -= c[i].x * vv[k].y + c[i].y * vv[k].x;
            }
        }
#pragma unroll
        for (int k = 0; k < 12; k++) wv[k] = make_double2(wv[k].x * f, wv[k].y * f);
        SiteIO<P>::store(q.w, V, s, wv);
#pragma unroll
        for (int k = 0; k < 12; k++) nrm[0] += wv[k].x * wv[k].x + wv[k].y * wv[k].y;
    }
    if (last) {
        const double t = group_sums(nrm, lds);
        if (threadIdx.x == 0) q.partial[blockIdx.x] = make_double2(t, 0.0);
    }
}

// out (precision PO) = in (precision PI) * mult
template <int PI, int PO>
__global__ __launch_bounds__(kRedThreads) void k_site_scale(const void *__restrict__ in, void *__restrict__ out,
                                                             double mult, int V) {
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < V; s += gridDim.x * blockDim.x) {
        double2 v[12];
        SiteIO<PI>::load(in, V, s, v);
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = make_double2(v[k].x * mult, v[k].y * mult);
        SiteIO<PO>::store(out, V, s, v);
    }
}

// w (native FP64) = keep * w + sum_{i < n} coef[i] v_i, v_i of precision P,
// n = min(kGSSite, count - i0) with count = hdr[0].x (device coefficients)
template <int P>
__global__ __launch_bounds__(kRedThreads) void k_site_combine(SiteBatch b, int i0, int V) {
    const SiteRhs &q = b.r[blockIdx.y];
    const int count = (int)q.hdr[0].x;
    const int n = count - i0 < kGSSite ? count - i0 : kGSSite;
    if (i0 > 0 && n <= 0) return;
    double2 c[kGSSite];
#pragma unroll
    for (int i = 0; i < kGSSite; i++) c[i] = i < n ? q.coef[i0 + i] : make_double2(0, 0);
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < V; s += gridDim.x * blockDim.x) {
        double2 xv[12];
        if (i0 > 0) {
            SiteIO<WDIRAC_F64>::load(q.w, V, s, xv);
        } else {
#pragma unroll
            for (int k = 0; k < 12; k++) xv[k] = make_double2(0, 0);
        }
#pragma unroll
        for (int i = 0; i < kGSSite; i++) {
            if (i < n) {
                double2 zv[12];
                SiteIO<P>::load(q.v[i], V, s, zv);
#pragma unroll
                for (int k = 0; k < 12; k++) {
                    xv[k].x += c[i].x * zv[k].x - c[i].y * zv[k].y;
                    xv[k].y += c[i].x * zv[k].y + c[i].y * zv[k].x;
                }
            }
        }
        SiteIO<WDIRAC_F64>::store(q.w, V, s, xv);
    }
}

// ---------------------------------------------------------------------------

static int site_grid(int V) {
    const int g = (V + kRedThreads - 1) / kRedThreads;
    return g < kRedBlocks ? g : kRedBlocks;
}
int site_groups(int V) { return site_grid(V); }

// vectors i0 .. i0 + n of items r0 ..
static SiteBatch site_batch(const SiteItem *items, int r0, int nr, int i0, int n) {
    SiteBatch b;
    for (int r = 0; r < kSiteBatch; r++) {
        const SiteItem &q = items[r0 + (r < nr ? r : 0)];
        for (int i = 0; i < kGSSite; i++) b.r[r].v[i] = i < n ? q.v[i0 + i] : q.w;
        b.r[r].w = q.w;
        b.r[r].partial = q.partial;
        b.r[r].coef = q.coef;
        b.r[r].hdr = q.hdr;
    }
    return b;
}

#define WD_SITE_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
static_assert(kGSSite == 8, "WD_SITE_CASES lists 1 .. kGSSite");

template <int P>
static hipError_t site_mdot_p(const SiteItem *items, int nr, int nv, int V, hipStream_t st) {
    for (int r0 = 0; r0 < nr; r0 += kSiteBatch) {
        const int m = nr - r0 < kSiteBatch ? nr - r0 : kSiteBatch;
        const dim3 grid(site_grid(V), m), blk(kRedThreads);
        for (int i0 = 0; i0 < nv; i0 += kGSSite) {
            const int n = nv - i0 < kGSSite ? nv - i0 : kGSSite;
            const bool last = i0 + kGSSite >= nv;
            const SiteBatch b = site_batch(items, r0, m, i0, n);
            if (!last) {
                hipLaunchKernelGGL((k_site_mdot<P, kGSSite, false>), grid, blk, 0, st, b, i0, nv, V);
                continue;
            }
            switch (n) {
#define WD_CASE(k) \
    case k: hipLaunchKernelGGL((k_site_mdot<P, k, true>), grid, blk, 0, st, b, i0, nv, V); break;
                WD_SITE_CASES(WD_CASE)
#undef WD_CASE
            }
        }
    }
    return hipGetLastError();
}

template <int P>
static hipError_t site_axpy_p(const SiteItem *items, int nr, int nv, int V, hipStream_t st) {
    for (int r0 = 0; r0 < nr; r0 += kSiteBatch) {
        const int m = nr - r0 < kSiteBatch ? nr - r0 : kSiteBatch;
        const dim3 grid(site_grid(V), m), blk(kRedThreads);
        for (int i0 = 0; i0 < nv; i0 += kGSSite) {
            const int n = nv - i0 < kGSSite ? nv - i0 : kGSSite;
            const int last = i0 + kGSSite >= nv ? 1 : 0;
            const SiteBatch b = site_batch(items, r0, m, i0, n);
            switch (n) {
#define WD_CASE(k) \
    case k: hipLaunchKernelGGL((k_site_axpy<P, k>), grid, blk, 0, st, b, i0, last, V); break;
                WD_SITE_CASES(WD_CASE)
#undef WD_CASE
            }
        }
    }
    return hipGetLastError();
}

template <int P>
static hipError_t site_combine_p(const SiteItem *items, int nr, int nmax, int V, hipStream_t st) {
    for (int r0 = 0; r0 < nr; r0 += kSiteBatch) {
        const int m = nr - r0 < kSiteBatch ? nr - r0 : kSiteBatch;
        for (int i0 = 0;; i0 += kGSSite) {
            int n = nmax - i0 < kGSSite ? nmax - i0 : kGSSite;
            if (n < 0) n = 0;
            const SiteBatch b = site_batch(items, r0, m, i0, n);
            hipLaunchKernelGGL(k_site_combine<P>, dim3(site_grid(V), m), dim3(kRedThreads), 0, st, b, i0, V);
            if (i0 + kGSSite >= nmax) break;
        }
    }
    return hipGetLastError();
}

hipError_t site_mdot(int prec, const SiteItem *items, int n, int nv, int V, hipStream_t st) {
    switch (prec) {
    case WDIRAC_F64: return site_mdot_p<WDIRAC_F64>(items, n, nv, V, st);
    case WDIRAC_F32: return site_mdot_p<WDIRAC_F32>(items, n, nv, V, st);
    case WDIRAC_F16S: return site_mdot_p<WDIRAC_F16S>(items, n, nv, V, st);
    }
    return hipErrorInvalidValue;
}

hipError_t site_axpy(int prec, const SiteItem *items, int n, int nv, int V, hipStream_t st) {
    switch (prec) {
    case WDIRAC_F64: return site_axpy_p<WDIRAC_F64>(items, n, nv, V, st);
    case WDIRAC_F32: return site_axpy_p<WDIRAC_F32>(items, n, nv, V, st);
    case WDIRAC_F16S: return site_axpy_p<WDIRAC_F16S>(items, n, nv, V, st);
    }
    return hipErrorInvalidValue;
}

hipError_t site_scale(int pin, int pout, const void *in, void *out, double mult, int V, hipStream_t st) {
    const dim3 g(site_grid(V)), b(kRedThreads);
#define WD_SITE_SCALE(PI, PO)                                                      \
    if (pin == PI && pout == PO) {                                                 \
        hipLaunchKernelGGL((k_site_scale<PI, PO>), g, b, 0, st, in, out, mult, V); \
        return hipGetLastError();                                                  \
    }
    WD_SITE_SCALE(WDIRAC_F64, WDIRAC_F64)
    WD_SITE_SCALE(WDIRAC_F64, WDIRAC_F32)
    WD_SITE_SCALE(WDIRAC_F64, WDIRAC_F16S)
    WD_SITE_SCALE(WDIRAC_F32, WDIRAC_F32)
    WD_SITE_SCALE(WDIRAC_F16S, WDIRAC_F16S)
#undef WD_SITE_SCALE
    return hipErrorInvalidValue;
}

hipError_t site_combine(int prec, const SiteItem *items, int n, int nmax, int V, hipStream_t st) {
    switch (prec) {
    case WDIRAC_F64: return site_combine_p<WDIRAC_F64>(items, n, nmax, V, st);
    case WDIRAC_F32: return site_combine_p<WDIRAC_F32>(items, n, nmax, V, st);
    case WDIRAC_F16S: return site_combine_p<WDIRAC_F16S>(items, n, nmax, V, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace wd

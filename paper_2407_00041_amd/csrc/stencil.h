// Per-site building blocks of the Wilson-clover stencil (Eq. (1.13)), shared
// by the full-lattice kernels and the even-odd kernels: spin projection to a
// half-spinor, the SU(3) product, reconstruction of the lower half, and the
// products with the 6x6 chirality blocks of the site-local term.
//
// Gamma basis: gamma_mu = [[0, B_mu], [B_mu^H, 0]], B_T = 1, B_Z = -i s3,
// B_Y = -i s2, B_X = -i s1, so the projector (I + s gamma_mu) maps
// (u, d) -> (h, s B_mu^H h) with h = u + s B_mu d.
#pragma once

#include "spinor_io.h"

namespace wd {

// Fence between hops.  A site's work is one basic block, so the compiler would
// issue every hop's loads first and do all the arithmetic afterwards (all
// eight hops in flight, far beyond the register file).  The empty asm takes
// the accumulators as in/out operands, so a hop's arithmetic must be done
// before it, and clobbers memory, so the next hop's loads stay after it.
template <typename T, int NR> __device__ __forceinline__ void hop_boundary(cx<T> (&acc)[NR][12]) {
#pragma unroll
    for (int r = 0; r < NR; r++)
#pragma unroll
        for (int k = 0; k < 12; k++) asm volatile("" : "+v"(acc[r][k].r), "+v"(acc[r][k].i) : : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// h = f (u + S B_mu d)  (u = spins 0,1; d = spins 2,3)
template <int MU, int S, typename T>
__device__ __forceinline__ void project(const cx<T> p[12], cx<T> h[6], T f) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        cx<T> d0 = p[6 + c], d1 = p[9 + c], b0, b1;
        if (MU == 0) { b0 = d0; b1 = d1; }
        else if (MU == 1) { b0 = times_mi(d0); b1 = times_i(d1); }
        else if (MU == 2) { b0 = mk<T>(-d1.r, -d1.i); b1 = d0; }
        else { b0 = times_mi(d1); b1 = times_mi(d0); }
        if (S > 0) { h[c] = f * (p[c] + b0); h[3 + c] = f * (p[3 + c] + b1); }
        else { h[c] = f * (p[c] - b0); h[3 + c] = f * (p[3 + c] - b1); }
    }
}

// h = u + S B_mu d (no factor)
template <int MU, int S, typename T>
__device__ __forceinline__ void project_unit(const cx<T> p[12], cx<T> h[6]) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        cx<T> d0 = p[6 + c], d1 = p[9 + c], b0, b1;
        if (MU == 0) { b0 = d0; b1 = d1; }
        else if (MU == 1) { b0 = times_mi(d0); b1 = times_i(d1); }
        else if (MU == 2) { b0 = mk<T>(-d1.r, -d1.i); b1 = d0; }
        else { b0 = times_mi(d1); b1 = times_mi(d0); }
        if (S > 0) { h[c] = p[c] + b0; h[3 + c] = p[3 + c] + b1; }
        else { h[c] = p[c] - b0; h[3 + c] = p[3 + c] - b1; }
    }
}

// upper += chi; lower += S B_mu^H chi
template <int MU, int S, typename T>
__device__ __forceinline__ void reconstruct(cx<T> acc[12], const cx<T> chi[6]) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        cx<T> c0 = chi[c], c1 = chi[3 + c], l0, l1;
        acc[c] = acc[c] + c0;
        acc[3 + c] = acc[3 + c] + c1;
        if (MU == 0) { l0 = c0; l1 = c1; }
        else if (MU == 1) { l0 = times_i(c0); l1 = times_mi(c1); }
        else if (MU == 2) { l0 = c1; l1 = mk<T>(-c0.r, -c0.i); }
        else { l0 = times_i(c1); l1 = times_i(c0); }
        if (S > 0) { acc[6 + c] = acc[6 + c] + l0; acc[9 + c] = acc[9 + c] + l1; }
        else { acc[6 + c] = acc[6 + c] - l0; acc[9 + c] = acc[9 + c] - l1; }
    }
}

// h = u + S B_mu d of a stored FP16S site without its scale.  Each component is one multiply-add on two fp16
// operands (their sum, rounded once to FP32: exact unless they are more than 13 binary places apart); `one` is opaque
// so that it stays one.
template <int MU, int S> __device__ __forceinline__ void project_half(const half8 q[3], cx<float> h[6]) {
    float one;
    asm("s_mov_b32 %0, 1.0" : "=s"(one));
    auto re = [&](int k) { return (float)q[k >> 2][2 * (k & 3)]; };
    auto im = [&](int k) { return (float)q[k >> 2][2 * (k & 3) + 1]; };
#pragma unroll
    for (int c = 0; c < 3; c++) {
        // S B_mu d of the two spins
        float b0r, b0i, b1r, b1i;
        const int d0 = 6 + c, d1 = 9 + c;
        if (MU == 0) { b0r = re(d0); b0i = im(d0); b1r = re(d1); b1i = im(d1); }
        else if (MU == 1) { b0r = im(d0); b0i = -re(d0); b1r = -im(d1); b1i = re(d1); }
        else if (MU == 2) { b0r = -re(d1); b0i = -im(d1); b1r = re(d0); b1i = im(d0); }
        else { b0r = im(d1); b0i = -re(d1); b1r = im(d0); b1i = -re(d0); }
        if (S < 0) { b0r = -b0r; b0i = -b0i; b1r = -b1r; b1i = -b1i; }
        h[c] = {__builtin_fmaf(b0r, one, re(c)), __builtin_fmaf(b0i, one, im(c))};
        h[3 + c] = {__builtin_fmaf(b1r, one, re(3 + c)), __builtin_fmaf(b1i, one, im(3 + c))};
    }
}

// upper += f chi; lower += g B_mu^H chi
template <int MU, typename T>
__device__ __forceinline__ void reconstruct_parts(cx<T> acc[12], const cx<T> chi[6], T f, T g) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cx<T> c0 = chi[c], c1 = chi[3 + c];
        cx<T> l0, l1;
        acc[c] = {fma(f, c0.r, acc[c].r), fma(f, c0.i, acc[c].i)};
        acc[3 + c] = {fma(f, c1.r, acc[3 + c].r), fma(f, c1.i, acc[3 + c].i)};
        if (MU == 0) { l0 = c0; l1 = c1; }
        else if (MU == 1) { l0 = times_i(c0); l1 = times_mi(c1); }
        else if (MU == 2) { l0 = c1; l1 = mk<T>(-c0.r, -c0.i); }
        else { l0 = times_i(c1); l1 = times_i(c0); }
        acc[6 + c] = {fma(g, l0.r, acc[6 + c].r), fma(g, l0.i, acc[6 + c].i)};
        acc[9 + c] = {fma(g, l1.r, acc[9 + c].r), fma(g, l1.i, acc[9 + c].i)};
    }
}

// upper += f chi; lower += f S B_mu^H chi
template <int MU, int S, typename T>
__device__ __forceinline__ void reconstruct_scaled(cx<T> acc[12], const cx<T> chi[6], T f) {
    reconstruct_parts<MU>(acc, chi, f, S > 0 ? f : -f);
}

// A neighbour's spinor as loaded: FP64 and FP32 values, or FP16S halves and
// their scale.  project_raw leaves the scale out; the hop's factor times the
// scale (weight) enters once, where the product is added (reconstruct_scaled).
// The factors are +-1/2, so at FP64 and FP32 this is the projection with the
// factor, bit for bit, without its multiplications.
template <int P> struct Raw {
    using T = typename Store<P>::T;
    cx<T> p[12];
    __device__ __forceinline__ void load(const void *base, int V, int s) { Store<P>::load_spinor(base, V, s, p); }
    __device__ __forceinline__ T weight(T f) const { return f; }
    __device__ __forceinline__ void half(int b, cx<T> v[6]) const {
#pragma unroll
        for (int k = 0; k < 6; k++) v[k] = p[6 * b + k];
    }
};
template <> struct Raw<WDIRAC_F16S> {
    half8 q[3];
    float sc;
    __device__ __forceinline__ void load(const void *base, int V, int s) {
        sc = Store<WDIRAC_F16S>::load_raw(base, V, s, q);
    }
    __device__ __forceinline__ float weight(float f) const { return f * sc; }
    __device__ __forceinline__ void half(int b, cx<float> v[6]) const {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const int e = 6 * b + k;
            v[k] = {sc * (float)q[e >> 2][2 * (e & 3)], sc * (float)q[e >> 2][2 * (e & 3) + 1]};
        }
    }
};
template <int MU, int S, int P>
__device__ __forceinline__ void project_raw(const Raw<P> &x, cx<typename Store<P>::T> h[6]) {
    if constexpr (P == WDIRAC_F16S) project_half<MU, S>(x.q, h);
    else project_unit<MU, S>(x.p, h);
}

// chi_s = U h_s (DAGU = false) or U^H h_s (DAGU = true), s = 0, 1
template <bool DAGU, typename T>
__device__ __forceinline__ void su3_mul(const cx<T> U[9], const cx<T> h[6], cx<T> chi[6]) {
#pragma unroll
    for (int sp = 0; sp < 2; sp++)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            cx<T> acc = mk<T>(0, 0);
#pragma unroll
            for (int b = 0; b < 3; b++)
                acc = DAGU ? cjfma(acc, U[3 * b + a], h[3 * sp + b]) : cfma(acc, U[3 * a + b], h[3 * sp + b]);
            chi[3 * sp + a] = acc;
        }
}

// y = A_blk x for one 6x6 Hermitian chirality block (real diagonal d, strict
// upper u in row-major pair order)
template <typename T>
__device__ __forceinline__ void clover_block(const T d[6], const cx<T> u[15], const cx<T> x[6], cx<T> y[6]) {
#pragma unroll
    for (int i = 0; i < 6; i++) y[i] = d[i] * x[i];
    int k = 0;
#pragma unroll
    for (int i = 0; i < 6; i++)
#pragma unroll
        for (int j = i + 1; j < 6; j++, k++) {
            y[i] = cfma(y[i], u[k], x[j]);
            y[j] = cjfma(y[j], u[k], x[i]);
        }
}

// y = A_blk x for a compact chirality block: A_00 = dg + H, A_11 = dg - H, A_01
// (row-major), A_10 = A_01^H; r = (h00, h11, h22, h01, h02, h12 as re/im,
// A_01 as re/im, pad)
template <typename T>
__device__ __forceinline__ void clover_block_compact(T dg, const T r[28], const cx<T> x[6], cx<T> y[6]) {
    const cx<T> u01 = {r[3], r[4]}, u02 = {r[5], r[6]}, u12 = {r[7], r[8]};
    // off-diagonal entries of +H (spin 0) and -H (spin 1), then the diagonal
#pragma unroll
    for (int sp = 0; sp < 2; sp++) {
        const cx<T> *v = x + 3 * sp;
        cx<T> t[3] = {cmul(u01, v[1]), cjmul(u01, v[0]), cjmul(u02, v[0])};
        t[0] = cfma(t[0], u02, v[2]);
        t[1] = cfma(t[1], u12, v[2]);
        t[2] = cjfma(t[2], u12, v[1]);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const T a = sp ? dg - r[c] : dg + r[c];
            y[3 * sp + c] = sp ? cx<T>{fma(a, v[c].r, -t[c].r), fma(a, v[c].i, -t[c].i)}
                               : cx<T>{fma(a, v[c].r, t[c].r), fma(a, v[c].i, t[c].i)};
        }
    }
    // spin-off-diagonal block A_01 and its adjoint
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const cx<T> m = {r[9 + 2 * (3 * i + j)], r[10 + 2 * (3 * i + j)]};
            y[i] = cfma(y[i], m, x[3 + j]);
            y[3 + j] = cjfma(y[3 + j], m, x[i]);
        }
}

}  // namespace wd

// Clover term from the links, once at operator creation (Sec. 2.2: the
// self-coupling matrices do not change between applications).
//
//   Q_mu,nu(x) : sum of the four plaquettes around x in the mu-nu plane,
//                Eq. (1.12);
//   C(x)       : -(1/32) sum_{mu,nu} (gamma_mu gamma_nu) (x) (Q_mu,nu - Q_nu,mu),
//                Eq. (1.11).
// Q_nu,mu(x) is the same four plaquettes traversed the other way, i.e.
// Q_mu,nu(x)^H, and the (mu,nu) and (nu,mu) terms of the sum are equal, so
// C(x) = -(1/16) sum_{mu<nu} (gamma_mu gamma_nu) (x) (Q_mu,nu - Q_mu,nu^H).
// In the chiral basis gamma_mu gamma_nu = diag(B_mu B_nu^H, B_mu^H B_nu),
// which gives the two 6x6 chirality blocks that are stored.
//
// FP64, canonical AoS links in, canonical packed [V][42] out (entry order
// documented in wdirac.h).
//
// Each plane's four leaves are two products instead of four: with
// W - W^H unchanged (up to sign) under W -> W^H, the leaves that begin or end
// with U_mu(x) share it, and so do the two with U_mu(x-mu):
//   X_1 = U_mu(x) [U_nu(x+mu) (U_nu(x) U_mu(x+nu))^H
//                  - U_nu(x-nu+mu)^H U_mu(x-nu)^H U_nu(x-nu)]
//   X_2 = [U_nu(x) (U_nu(x-mu) U_mu(x-mu+nu))^H
//          - (U_mu(x-mu-nu) U_nu(x-nu))^H U_nu(x-mu-nu)] U_mu(x-mu)
//   Q - Q^H = (X_1 + X_2) - (X_1 + X_2)^H,
// ten 3x3 products per plane instead of twelve.
//
// A work-group is six waves over the same 64 sites, wave p the plane p, so a
// lane holds one plane's matrices and nothing is indexed at run time (one
// thread per site with all six planes and both 6x6 blocks live took 256 VGPRs
// and 824 B of scratch); the planes' Q - Q^H meet in LDS, and the work-group
// writes the 64 x 42 outputs in order.  Bound by the links' way from the L2: a
// plane reads 12 matrices per site, each 144 B that touch two 128-byte lines.
// Turning them through LDS (nine consecutive lanes per matrix), with or without
// the next pair in flight, and three waves per SIMD (spills) measured the same
// or slower.  32^4: 2714 -> 1272 us.
#include "spinor_io.h"

namespace wd {

namespace {

constexpr int kSites = 64;   // sites per work-group
constexpr int kPlanes = 6;   // (T,Z) (T,Y) (T,X) (Z,Y) (Z,X) (Y,X), one wave each

struct M3 {
    cx<double> a[9];
};

// x y; DX, DY: the adjoint of x, y
template <bool DX, bool DY> __device__ __forceinline__ M3 mul(const M3 &x, const M3 &y) {
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; e++) m.a[e] = mk<double>(0, 0);
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const cx<double> u = x.a[DX ? 3 * k + i : 3 * i + k];
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const cx<double> v = y.a[DY ? 3 * j + k : 3 * k + j];
                cx<double> &s = m.a[3 * i + j];
                s = DX ? cjfma(s, u, v) : DY ? cjfma(s, v, u) : cfma(s, u, v);
            }
        }
    return m;
}
// m += f x, f = +-1.  Products are rounded by themselves before they are added: chaining one product's multiply-adds
// onto another's sum rounds every term at the larger magnitude (error of Q - Q^H against 80-bit arithmetic, smooth
// links: 1.98e-16 chained, 1.79e-16 apart, four separate leaves 1.83e-16)
__device__ __forceinline__ void add(M3 &m, const M3 &x, double f) {
#pragma unroll
    for (int e = 0; e < 9; e++) m.a[e] = {fma(f, x.a[e].r, m.a[e].r), fma(f, x.a[e].i, m.a[e].i)};
}

__device__ __forceinline__ M3 link(const d2v *links, int site, int mu) {
    const d2v *p = links + (size_t)(4 * site + mu) * 9;
    M3 o;
#pragma unroll
    for (int e = 0; e < 9; e++) {
        const d2v a = p[e];
        o.a[e] = {a.x, a.y};
    }
    return o;
}

// keeps the next product's loads behind this one's arithmetic (registers)
__device__ __forceinline__ void step() { __builtin_amdgcn_sched_barrier(0); }

// entry (i, j) of the chirality block packed at position k of a block's 21
__device__ __forceinline__ void packed_pair(int k, int &i, int &j) {
    if (k < 6) {
        i = j = k;
        return;
    }
    k -= 6;
    i = 0;
    for (int n = 5; k >= n; n--) {
        k -= n;
        i++;
    }
    j = i + 1 + k;
}

}  // namespace

// SLABS: the tiles' eighths are of a slab of several T-slices, the last slab possibly a shorter one, not of one slice
template <bool SLABS>
__global__ __launch_bounds__(kPlanes * 64) void clover_build_kernel(double2 *__restrict__ out,
                                                                    const double2 *__restrict__ links, Geom g,
                                                                    int eighth, int slab) {
    __shared__ d2v lds[kPlanes][9 * kSites];
    const int lane = threadIdx.x & 63;
    const int plane = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // tiles as in the link force: XCD k (work-groups go to the 8 XCDs in turn) takes the k-th eighth of every
    // T-slice and all XCDs walk the slices together, so most neighbour links are in the XCD's own L2
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int tpe = eighth / kSites;
    const int t = q / tpe, slice = SLABS ? slab : g.stride[0];
    const int lo = xcd * eighth + (q - t * tpe) * kSites;
    const int base = t * slice + lo;
    int nsite = min(kSites, min((xcd + 1) * eighth, slice) - lo);
    if (SLABS) nsite = min(nsite, g.V - base);
    if (nsite <= 0) return;
    {
        const int mu = plane < 3 ? 0 : (plane < 5 ? 1 : 2);
        const int nu = plane < 3 ? plane + 1 : (plane < 5 ? plane - 1 : 3);
        const int s = base + min(lane, nsite - 1);  // idle lanes repeat the last site
        const int sm = mu == 0 ? g.stride[0] : (mu == 1 ? g.stride[1] : g.stride[2]);
        const int Lm = mu == 0 ? g.n[0] : (mu == 1 ? g.n[1] : g.n[2]);
        const int sn = nu == 1 ? g.stride[1] : (nu == 2 ? g.stride[2] : 1);
        const int Ln = nu == 1 ? g.n[1] : (nu == 2 ? g.n[2] : g.n[3]);
        const int cm = s / sm % Lm, cn = s / sn % Ln;
        const int mf = cm == Lm - 1 ? -(Lm - 1) * sm : sm, mb = cm == 0 ? (Lm - 1) * sm : -sm;
        const int nf = cn == Ln - 1 ? -(Ln - 1) * sn : sn, nb = cn == 0 ? (Ln - 1) * sn : -sn;
        const d2v *L = reinterpret_cast<const d2v *>(links);
        auto U = [&](int site, int dir) { return link(L, site, dir); };
        M3 P, S, F;
        P = mul<false, false>(U(s, nu), U(s + nf, mu));
        step();
        S = mul<false, true>(U(s + mf, nu), P);
        step();
        P = mul<true, false>(U(s + nb, mu), U(s + nb, nu));
        step();
        add(S, mul<true, false>(U(s + nb + mf, nu), P), -1.0);
        step();
        F = mul<false, false>(U(s, mu), S);
        step();
        P = mul<false, false>(U(s + mb, nu), U(s + mb + nf, mu));
        step();
        S = mul<false, true>(U(s, nu), P);
        step();
        P = mul<false, false>(U(s + mb + nb, mu), U(s + nb, nu));
        step();
        add(S, mul<true, false>(P, U(s + mb + nb, nu)), -1.0);
        step();
        add(F, mul<false, false>(S, U(s + mb, mu)), 1.0);
        // Q - Q^H, entry e of this lane's site at [e][lane]
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const cx<double> a = F.a[3 * i + j], b = F.a[3 * j + i];
                lds[plane][(3 * i + j) * kSites + lane] = d2v{a.r - b.r, a.i + b.i};
            }
    }
    __syncthreads();
    // gamma_mu gamma_nu in the chiral basis: with F_p = Q - Q^H of plane p and t = +1 (block +) or -1 (block -),
    //   C = -(i/16) [s3 (x) (t F_TZ - F_YX) + s2 (x) (t F_TY + F_ZX) + s1 (x) (t F_TX - F_ZY)]
    for (int w = threadIdx.x; w < nsite * 42; w += kPlanes * 64) {
        const int l = w / 42, e = w - 42 * l;
        const int b = e >= 21 ? 1 : 0;
        const double tb = b ? -1.0 : 1.0;
        int i, j;
        packed_pair(e - 21 * b, i, j);
        const int at = (3 * (i % 3) + j % 3) * kSites + l;
        d2v v;  // C = -(i/16) v
        if (i < 3 && j >= 3) {
            const d2v tx = lds[2][at], zy = lds[3][at], ty = lds[1][at], zx = lds[4][at];
            // s1 - i s2 of the spin-off-diagonal entry
            v.x = (tb * tx.x - zy.x) + (tb * ty.y + zx.y);
            v.y = (tb * tx.y - zy.y) - (tb * ty.x + zx.x);
        } else {
            const double sgn = i < 3 ? 1.0 : -1.0;
            const d2v tz = lds[0][at], yx = lds[5][at];
            v.x = sgn * (tb * tz.x - yx.x);
            v.y = sgn * (tb * tz.y - yx.y);
        }
        out[(size_t)base * 42 + w] = make_double2((1.0 / 16.0) * v.y, (-1.0 / 16.0) * v.x);
    }
}

hipError_t clover_build_launch(double *out, const double *links, const Geom &g, hipStream_t st) {
    // slices of less than a tile per eighth, in slabs of up to 4096 sites: by slices the 64 sites of a 4^3 slice are
    // one XCD's (1024 x 4^3: 480 us, in slabs 69; 96 x 6^3: 57, 35)
    const int q = g.stride[0] < 8 * kSites ? slab_slices(g.n[0], g.stride[0], 4096) : 1, slab = q * g.stride[0];
    const int eighth = ((slab + 7) / 8 + kSites - 1) / kSites * kSites;
    const dim3 grid((g.n[0] + q - 1) / q * 8 * (eighth / kSites)), blk(kPlanes * 64);
    double2 *o = reinterpret_cast<double2 *>(out);
    const double2 *l = reinterpret_cast<const double2 *>(links);
    if (q > 1)
        hipLaunchKernelGGL(clover_build_kernel<true>, grid, blk, 0, st, o, l, g, eighth, slab);
    else
        hipLaunchKernelGGL(clover_build_kernel<false>, grid, blk, 0, st, o, l, g, eighth, slab);
    return hipGetLastError();
}

}  // namespace wd

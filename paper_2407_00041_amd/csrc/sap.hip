// Schwarz alternating procedure (SAP) on non-overlapping lattice blocks: the
// domain-decomposition smoother that Sec. 1.3 names (additive and red-black
// multiplicative Schwarz) used as the flexible preconditioner M_j^{-1} of
// FGMRES (Algorithm 2).
//
// A block of b_T x b_Z x b_Y x b_X sites (at most 256) is one work-group, one
// lane per site.  Its block operator D_B is D with the hops that leave the
// block dropped; the local solve is mr_iters minimal-residual steps
// (e = 0, rho = r_B; q = D_B rho, alpha = <q, rho>/<q, q>, e += alpha rho,
// rho -= alpha q), run entirely on chip: the block's rho lives in LDS so
// every lane reads its in-block neighbours there, the two dot products are
// reduced across the work-group through LDS in a fixed order (deterministic),
// and at FP32 the block's forward links are staged in LDS and its compact
// clover blocks held in registers, so the MR steps read no memory at all.
// The residual r_B = (b - D x)_B that starts a block solve is computed by the
// same kernel from the full operator: the block's own x staged in the same LDS
// slots, neighbour values from other blocks read from memory by the lanes on a
// face.  One launch per colour (red-black) or one for all
// blocks (additive) per cycle; x is FP64 in memory, the block arithmetic is
// FP64 or FP32 (the operator data of that precision), dot products are
// accumulated in FP64.
//
// Blocks of one colour are enumerated in pairs along a direction with an
// even block count (the last such of T, Z, Y, X): the i-th block of colour c
// takes the other block coordinates from i and the paired coordinate so that
// the coordinate sum has parity c.
#include <algorithm>

#include "blas.h"
#include "sap.h"
#include "stencil.h"

namespace wd {

namespace {

constexpr int kSapMaxBlock = 256;

template <int P> using TOf = typename Store<P>::T;

// FP64 field value at site s, converted to the arithmetic type
template <typename T> __device__ __forceinline__ void load_x(const double2 *f, int V, int s, cx<T> v[12]) {
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const double2 a = f[(size_t)k * V + s];
        v[k] = {(T)a.x, (T)a.y};
    }
}

// lexicographic block coordinates of the i-th block of a pass
__device__ __forceinline__ void block_coords(const SapGeom &sg, int colour, int i, int bc[4]) {
    int ext[4] = {sg.nb[0], sg.nb[1], sg.nb[2], sg.nb[3]};
    const int m = colour >= 0 ? sg.pair_dir : -1;
    if (m >= 0) ext[m] >>= 1;
    int r = i;
    bc[3] = r % ext[3]; r /= ext[3];
    bc[2] = r % ext[2]; r /= ext[2];
    bc[1] = r % ext[1];
    bc[0] = r / ext[1];
    if (m >= 0) {
        int other = 0;
#pragma unroll
        for (int mu = 0; mu < 4; mu++)
            if (mu != m) other += bc[mu];
        bc[m] = 2 * bc[m] + ((colour + other) & 1);
    }
}

// site-local term A(x) psi: clover blocks kept in registers (FP32 compact) or loaded at each use
template <int P, bool REGC> struct SiteTerm {
    using T = TOf<P>;
    T cr[2][REGC ? 28 : 1];
    __device__ __forceinline__ void init(const OpData &d, int V, int s) {
        if constexpr (REGC) {
            Store<P>::load_clover_compact(d.clover, V, 0, s, cr[0]);
            Store<P>::load_clover_compact(d.clover, V, 1, s, cr[1]);
        }
    }
    __device__ __forceinline__ void apply(const OpData &d, int V, int s, const cx<T> in[12], cx<T> out[12]) const {
#pragma unroll
        for (int b = 0; b < 2; b++) {
            if constexpr (REGC) {
                clover_block_compact((T)d.diag, cr[b], &in[6 * b], &out[6 * b]);
            } else if (d.clover_compact) {
                T r[28];
                Store<P>::load_clover_compact(d.clover, V, b, s, r);
                clover_block_compact((T)d.diag, r, &in[6 * b], &out[6 * b]);
            } else {
                T dd[6];
                cx<T> uu[15];
                Store<P>::load_clover(d.clover, V, b, s, dd, uu);
                clover_block(dd, uu, &in[6 * b], &out[6 * b]);
            }
        }
    }
};

// deterministic sum over the work-group of three doubles (every lane gets the totals)
__device__ __forceinline__ void group_sum3(double (&v)[3], double (*red)[3]) {
    int index = 0, count = 3;
    const double t = lane_sums<3, 32>(v, index, count);
    if (count > 0) red[threadIdx.x >> 6][index] = t;
    __syncthreads();
    const int nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        v[k] = 0.0;
        for (int q = 0; q < nw; q++) v[k] += red[q][k];
    }
}

// One lane's place in its block: sites, neighbours and boundary crossings
struct SapSite {
    int s, l;
    int nf[4], nbk[4];  // in-block neighbours (local index, or -1 when the hop leaves the block)
    bool wf, wb;        // in-block hops that cross the T boundary
};

// q += the hops of direction MU that stay inside the block, of the field in LDS
template <int P, bool LDSL, int MU, int NL>
__device__ __forceinline__ void block_hops(const cx<TOf<P>> (*f_lds)[kSapMaxBlock], const f4v (*link_lds)[NL],
                                           const OpData &d, const Geom &g, const SapGeom &sg, const SapSite &a,
                                           bool apbc, cx<TOf<P>> q[12]) {
    using T = TOf<P>;
    auto link = [&](int n, cx<T> U[9]) {
        if constexpr (LDSL) {
#pragma unroll
            for (int e = 0; e < 3; e++) {
                const f4v u = link_lds[3 * MU + e][n];
                U[2 * e] = {u.x, u.y};
                U[2 * e + 1] = {u.z, u.w};
            }
            third_row(U);
        } else {
            Store<P>::load_link(d.links, g.V, MU, a.s + (n - a.l) / sg.lstr[MU] * g.stride[MU], U, d.rows);
        }
    };
    if (a.nf[MU] >= 0) {
        cx<T> U[9], p[12], h[6], chi[6];
        link(a.l, U);
#pragma unroll
        for (int k = 0; k < 12; k++) p[k] = f_lds[k][a.nf[MU]];
        project_unit<MU, -1>(p, h);
        su3_mul<false>(U, h, chi);
        reconstruct_scaled<MU, -1>(q, chi, (MU == 0 && apbc && a.wf) ? T(0.5) : T(-0.5));
    }
    if (a.nbk[MU] >= 0) {
        cx<T> U[9], p[12], h[6], chi[6];
        link(a.nbk[MU], U);
#pragma unroll
        for (int k = 0; k < 12; k++) p[k] = f_lds[k][a.nbk[MU]];
        project_unit<MU, +1>(p, h);
        su3_mul<true>(U, h, chi);
        reconstruct_scaled<MU, +1>(q, chi, (MU == 0 && apbc && a.wb) ? T(0.5) : T(-0.5));
    }
}

// The hop of a lane that leaves the block along one direction, as loaded.  With two-row FP32 links the values stay
// as loaded until they are used, so the arithmetic between load and add runs while they are on their way.
template <int P, bool LDSL> struct HaloHop {
    using T = TOf<P>;
    double2 x[12];
    f4v u[LDSL ? 3 : 1];
    int sn, sl;  // the neighbour, the site that holds the link
    T f, sign;   // factor and projector sign (forward -1, backward +1)
    __device__ __forceinline__ void load(const double2 *xin, const OpData &d, const Geom &g, int mu, int s, int coord,
                                         bool forward, bool apbc) {
        const int st = g.stride[mu], L = g.n[mu];
        const bool wrap = coord == (forward ? L - 1 : 0);
        const int step = wrap ? (L - 1) * st : st;
        sn = (forward != wrap) ? s + step : s - step;
        sl = forward ? s : sn;
        f = (mu == 0 && apbc && wrap) ? T(0.5) : T(-0.5);
        sign = forward ? T(-1) : T(1);
#pragma unroll
        for (int k = 0; k < 12; k++) x[k] = xin[(size_t)k * g.V + sn];
        if constexpr (LDSL) {
            const f4v *q = static_cast<const f4v *>(d.links);
#pragma unroll
            for (int e = 0; e < 3; e++) u[e] = q[op_idx(3 * mu + e, 12, sl)];
        }
    }
    template <int MU> __device__ __forceinline__ void add(const OpData &d, const Geom &g, cx<T> acc[12]) const {
        cx<T> U[9], W[9], p[12], h[6], chi[6];
        if constexpr (LDSL) {
#pragma unroll
            for (int e = 0; e < 3; e++) {
                U[2 * e] = {u[e].x, u[e].y};
                U[2 * e + 1] = {u[e].z, u[e].w};
            }
            third_row(U);
        } else {
            Store<P>::load_link(d.links, g.V, MU, sl, U, d.rows);
        }
        const bool fw = sign < T(0);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const cx<T> v = U[3 * i + j], w = U[3 * j + i];
                W[3 * i + j] = {fw ? v.r : w.r, fw ? v.i : -w.i};
            }
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const T c = k < 6 ? T(1) : sign;
            p[k] = {c * (T)x[k].x, c * (T)x[k].y};
        }
        project_unit<MU, +1>(p, h);
        su3_mul<false>(W, h, chi);
        reconstruct_parts<MU>(acc, chi, f, f * sign);
    }
};

// What bounds it, at 32 x 16^2 x 32 and FP32 (512 blocks of 4^4 per colour, two per CU, one round of work-groups): an
// MR step takes 6 us, the FP32 issue rate of its 1900 instructions per site; the rest of a pass is its memory traffic,
// 128-byte lines of which a colour uses half.  Two cycles of red-black with four steps: 409 us with every neighbour of
// x read from memory, 290 now; FP64 902 -> 777 (an MR step 34 us: one work-group per CU, registers).  Loading the next
// direction's face hop one direction ahead gained nothing (300).
//
// One Schwarz pass: every block of the pass (colour c, or all blocks for c < 0) computes its residual
// r_B = (b - D x)_B, solves D_B e = r_B approximately by nmr MR steps and writes x_out = x_in + e on its
// sites.  xzero: x_in is zero everywhere (r = b); own_zero: x_in is zero on the pass's blocks (their
// in-block terms are skipped, halo values come from x_in).  LDSL: links staged in LDS (FP32, two rows);
// REGC: compact clover blocks in registers (FP32).
template <int P, bool LDSL, bool REGC>
__global__ __launch_bounds__(kSapMaxBlock) void sap_pass_kernel(const double2 *__restrict__ b, const double2 *xin,
                                                                double2 *xout, size_t rhs_stride, OpData d, Geom g,
                                                                SapGeom sg, int colour, int xzero, int own_zero,
                                                                int nmr, int apbc, double bscale) {
    using T = TOf<P>;
    constexpr int NL = LDSL ? kSapMaxBlock : 1;
    __shared__ cx<T> rho_lds[12][kSapMaxBlock];
    __shared__ f4v link_lds[LDSL ? 12 : 1][NL];
    __shared__ double red[kSapMaxBlock / 64][3];
    // FP64: the correction e is kept in the lane's LDS slot too (registers hold the hop in flight)
    constexpr bool ELDS = P == WDIRAC_F64;
    __shared__ cx<T> e_lds[ELDS ? 12 : 1][ELDS ? kSapMaxBlock : 1];

    const int V = g.V;
    const int l = threadIdx.x;
    const bool active = l < sg.bvol;
    b += blockIdx.y * rhs_stride;
    if (xin) xin += blockIdx.y * rhs_stride;
    xout += blockIdx.y * rhs_stride;

    int bc[4];
    // consecutive blocks on one XCD, which read each other's faces and halves of the same 128-byte lines through one
    // L2 (work-group i runs on XCD i mod 8); additive, two cycles: 347 -> 229 us
    const int per = (int)(gridDim.x >> 3), part = (int)(blockIdx.x >> 3);
    block_coords(sg, colour, part < per ? (int)(blockIdx.x & 7) * per + part : (int)blockIdx.x, bc);
    int lc[4], s = 0;
    {
        int r = active ? l : 0;
        lc[3] = r % sg.b[3]; r /= sg.b[3];
        lc[2] = r % sg.b[2]; r /= sg.b[2];
        lc[1] = r % sg.b[1];
        lc[0] = r / sg.b[1];
#pragma unroll
        for (int mu = 0; mu < 4; mu++) s += (bc[mu] * sg.b[mu] + lc[mu]) * g.stride[mu];
    }
    SapSite at;
    at.s = s;
    at.l = l;
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        const int st = sg.lstr[mu], B = sg.b[mu];
        at.nf[mu] = lc[mu] + 1 < B ? l + st : (sg.span[mu] ? l - (B - 1) * st : -1);
        at.nbk[mu] = lc[mu] > 0 ? l - st : (sg.span[mu] ? l + (B - 1) * st : -1);
    }
    at.wf = sg.span[0] && lc[0] == sg.b[0] - 1;
    at.wb = sg.span[0] && lc[0] == 0;

    SiteTerm<P, REGC> A;
    if (active) A.init(d, V, s);
    if constexpr (LDSL) {
        if (active) {
            const f4v *q = static_cast<const f4v *>(d.links);
#pragma unroll
            for (int e = 0; e < 12; e++) link_lds[e][l] = q[op_idx(e, 12, s)];
        }
    }

    // ---- residual r = b - D x.  The block's own x is read once, into the LDS slots that will hold rho: the hops
    // inside the block read it there, and only the lanes on a face read neighbours from memory, their loads in
    // flight during that direction's hops inside the block.  Then r goes into the lane's slot.
    {
        cx<T> accs[1][12];
        cx<T>(&acc)[12] = accs[0];
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = mk<T>(0, 0);
        const bool inner = !xzero && !own_zero;
        if (inner) {
            if (active) {
                cx<T> xs[12];
                load_x<T>(xin, V, s, xs);
#pragma unroll
                for (int k = 0; k < 12; k++) rho_lds[k][l] = xs[k];
                A.apply(d, V, s, xs, acc);
            }
            __syncthreads();
        }
        if (!xzero) {
#define WD_SAP_RES_HOP(MU)                                                                                        \
            {                                                                                                     \
                const int c = bc[MU] * sg.b[MU] + lc[MU];                                                         \
                const bool lf = active && at.nf[MU] < 0, lb = active && at.nbk[MU] < 0;                           \
                HaloHop<P, LDSL> halo;                                                                            \
                if (lf || lb) halo.load(xin, d, g, MU, s, c, lf, apbc);                                           \
                if (inner && active) block_hops<P, LDSL, MU, NL>(rho_lds, link_lds, d, g, sg, at, apbc, acc);     \
                if (lf || lb) halo.template add<MU>(d, g, acc);                                                   \
                if (lf && lb) { /* a block of extent one */                                                       \
                    halo.load(xin, d, g, MU, s, c, false, apbc);                                                  \
                    halo.template add<MU>(d, g, acc);                                                             \
                }                                                                                                 \
            }                                                                                                     \
            hop_boundary<T, 1>(accs);
            hop_boundary<T, 1>(accs);
            WD_SAP_RES_HOP(0)
            WD_SAP_RES_HOP(1)
            WD_SAP_RES_HOP(2)
            WD_SAP_RES_HOP(3)
#undef WD_SAP_RES_HOP
        }
        if (inner) __syncthreads();  // every lane has read its neighbours' x
#pragma unroll
        for (int k = 0; k < 12; k++) {
            cx<T> r = mk<T>(0, 0);
            if (active) {
                const double2 a = b[(size_t)k * V + s];
                r = mk<T>((T)(bscale * a.x), (T)(bscale * a.y)) - acc[k];
            }
            rho_lds[k][l] = r;
        }
    }

    // ---- minimal-residual steps on D_B e = rho; rho lives only in LDS (each lane updates its own slot once
    // every lane has finished reading its neighbours, i.e. after the reduction's barrier)
    cx<T> e[ELDS ? 1 : 12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        if constexpr (ELDS) e_lds[k][l] = mk<T>(0, 0);
        else e[k] = mk<T>(0, 0);
    }
    for (int it = 0; it < nmr; it++) {
        __syncthreads();
        cx<T> qs[1][12];
        cx<T>(&q)[12] = qs[0];
#pragma unroll
        for (int k = 0; k < 12; k++) q[k] = mk<T>(0, 0);
        if (active) {
            {
                cx<T> own[12];
#pragma unroll
                for (int k = 0; k < 12; k++) own[k] = rho_lds[k][l];
                A.apply(d, V, s, own, q);
            }
            hop_boundary<T, 1>(qs);
            block_hops<P, LDSL, 0, NL>(rho_lds, link_lds, d, g, sg, at, apbc, q);
            hop_boundary<T, 1>(qs);
            block_hops<P, LDSL, 1, NL>(rho_lds, link_lds, d, g, sg, at, apbc, q);
            hop_boundary<T, 1>(qs);
            block_hops<P, LDSL, 2, NL>(rho_lds, link_lds, d, g, sg, at, apbc, q);
            hop_boundary<T, 1>(qs);
            block_hops<P, LDSL, 3, NL>(rho_lds, link_lds, d, g, sg, at, apbc, q);
            hop_boundary<T, 1>(qs);
        }
        // <q, rho> and <q, q> over the block, accumulated in FP64
        double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<T> r = rho_lds[k][l];
            const double qr = q[k].r, qi = q[k].i, rr = r.r, ri = r.i;
            v[0] += qr * rr + qi * ri;
            v[1] += qr * ri - qi * rr;
            v[2] += qr * qr + qi * qi;
        }
        group_sum3(v, red);  // its barrier also ends every lane's reads of rho_lds for this step
        const double ar = v[2] > 0.0 ? v[0] / v[2] : 0.0, ai = v[2] > 0.0 ? v[1] / v[2] : 0.0;
        const cx<T> alpha = {(T)ar, (T)ai};
        const bool more = it + 1 < nmr;
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const cx<T> r = rho_lds[k][l];
            if constexpr (ELDS) e_lds[k][l] = e_lds[k][l] + cmul(alpha, r);
            else e[k] = e[k] + cmul(alpha, r);
            if (more) rho_lds[k][l] = r - cmul(alpha, q[k]);
        }
    }

    // ---- x_out = x_in + e
    if (active) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            cx<T> ek;
            if constexpr (ELDS) ek = e_lds[k][l];
            else ek = e[k];
            double2 o = make_double2((double)ek.r, (double)ek.i);
            if (!xzero && !own_zero) {
                const double2 a = xin[(size_t)k * V + s];
                o.x += a.x;
                o.y += a.y;
            }
            xout[(size_t)k * V + s] = o;
        }
    }
}

template <int P, bool LDSL, bool REGC>
hipError_t launch_pass(const dirac_op *op, const SapGeom &sg, int colour, int nblk, const double2 *b,
                       const double2 *xin, double2 *xout, bool xzero, bool own_zero, int nmr, int nrhs,
                       double bscale, hipStream_t st) {
    const int threads = (sg.bvol + 63) / 64 * 64;
    const int apbc = (op->flags & WDIRAC_ANTIPERIODIC_T) ? 1 : 0;
    hipLaunchKernelGGL((sap_pass_kernel<P, LDSL, REGC>), dim3(nblk, nrhs), dim3(threads), 0, st, b, xin, xout,
                       (size_t)12 * op->g.V, op->data(P), op->g, sg, colour, xzero ? 1 : 0, own_zero ? 1 : 0, nmr,
                       apbc, bscale);
    return hipGetLastError();
}

hipError_t sap_pass(const dirac_op *op, const sap_params &p, const SapGeom &sg, int colour, const double2 *b,
                    const double2 *xin, double2 *xout, bool xzero, bool own_zero, int nrhs, double bs,
                    hipStream_t st) {
    int nblk = sg.nblocks;
    int dec = colour;
    if (colour >= 0) {
        if (sg.pair_dir < 0) {
            if (colour == 1) return hipSuccess;  // a single block, of colour 0
            dec = -1;
        } else {
            nblk = sg.nblocks / 2;
        }
    }
    if (p.prec == WDIRAC_F64)
        return launch_pass<WDIRAC_F64, false, false>(op, sg, dec, nblk, b, xin, xout, xzero, own_zero, p.mr_iters,
                                                     nrhs, bs, st);
    const bool ldsl = op->link_rows == 2, regc = op->clover_compact;
    if (ldsl && regc)
        return launch_pass<WDIRAC_F32, true, true>(op, sg, dec, nblk, b, xin, xout, xzero, own_zero, p.mr_iters,
                                                   nrhs, bs, st);
    if (ldsl)
        return launch_pass<WDIRAC_F32, true, false>(op, sg, dec, nblk, b, xin, xout, xzero, own_zero, p.mr_iters,
                                                    nrhs, bs, st);
    if (regc)
        return launch_pass<WDIRAC_F32, false, true>(op, sg, dec, nblk, b, xin, xout, xzero, own_zero, p.mr_iters,
                                                    nrhs, bs, st);
    return launch_pass<WDIRAC_F32, false, false>(op, sg, dec, nblk, b, xin, xout, xzero, own_zero, p.mr_iters, nrhs,
                                                 bs, st);
}

}  // namespace

int sap_geometry(const dirac_op *op, const sap_params *p, SapGeom &sg) {
    if (!op || !p) return fail(WDIRAC_EINVAL, "null operator or SAP parameters");
    if (p->prec != WDIRAC_F64 && p->prec != WDIRAC_F32)
        return fail(WDIRAC_EINVAL, "SAP precision must be WDIRAC_F64 or WDIRAC_F32");
    if (!op->data(p->prec).links) return fail(WDIRAC_EUNSUPPORTED, "SAP precision not materialised at create");
    if (p->cycles < 1 || p->mr_iters < 1) return fail(WDIRAC_EINVAL, "SAP cycles and mr_iters must be >= 1");
    if (p->additive != 0 && p->additive != 1) return fail(WDIRAC_EINVAL, "SAP additive must be 0 or 1");
    long long vol = 1;
    sg.pair_dir = -1;
    for (int mu = 0; mu < 4; mu++) {
        const int B = p->block[mu], L = op->g.n[mu];
        if (B < 1 || L % B) return fail(WDIRAC_EINVAL, "SAP block extents must divide the lattice extents");
        sg.b[mu] = B;
        sg.nb[mu] = L / B;
        if (sg.nb[mu] != 1 && sg.nb[mu] % 2)
            return fail(WDIRAC_EINVAL, "SAP blocks per direction must be even or 1 (red-black colouring)");
        sg.span[mu] = sg.nb[mu] == 1 ? 1 : 0;
        if (sg.nb[mu] % 2 == 0) sg.pair_dir = mu;
        vol *= B;
    }
    if (vol > kSapMaxBlock) return fail(WDIRAC_EINVAL, "SAP blocks may hold at most 256 sites");
    sg.bvol = (int)vol;
    sg.lstr[3] = 1;
    sg.lstr[2] = sg.b[3];
    sg.lstr[1] = sg.b[3] * sg.b[2];
    sg.lstr[0] = sg.b[3] * sg.b[2] * sg.b[1];
    sg.nblocks = op->g.V / sg.bvol;
    return WDIRAC_OK;
}

size_t sap_workspace(const dirac_op *op, const sap_params *p, int nrhs) {
    return (p->additive && p->cycles > 1) ? field_rhs_bytes(WDIRAC_F64, op->g.V) * (size_t)nrhs : 0;
}

hipError_t sap_apply(const dirac_op *op, const sap_params &p, const SapGeom &sg, double2 *x, const double2 *b,
                     int nrhs, double2 *work, double bscale, hipStream_t st) {
    if (!p.additive) {
        for (int cyc = 0; cyc < p.cycles; cyc++)
            for (int c = 0; c < 2; c++) {
                const hipError_t e =
                    sap_pass(op, p, sg, c, b, x, x, cyc == 0 && c == 0, cyc == 0 && c == 1, nrhs, bscale, st);
                if (e != hipSuccess) return e;
            }
        return hipSuccess;
    }
    // additive: every block from the same x, so consecutive cycles alternate between x and the workspace, the
    // last one writing x
    double2 *bufs[2] = {x, work};
    int out = (p.cycles % 2) ? 0 : 1;
    const double2 *in = nullptr;
    for (int cyc = 0; cyc < p.cycles; cyc++) {
        const hipError_t e = sap_pass(op, p, sg, -1, b, in, bufs[out], cyc == 0, false, nrhs, bscale, st);
        if (e != hipSuccess) return e;
        in = bufs[out];
        out ^= 1;
    }
    return hipSuccess;
}

}  // namespace wd

using namespace wd;

extern "C" {

size_t dirac_sap_workspace_bytes(const dirac_op *op, const sap_params *p, int nrhs) {
    SapGeom sg;
    if (nrhs < 1 || sap_geometry(op, p, sg)) return 0;
    return sap_workspace(op, p, nrhs);
}

int dirac_sap(const dirac_op *op, double *x, const double *b, int nrhs, const sap_params *p, void *work,
              size_t work_bytes, void *stream) {
    SapGeom sg;
    int rc = sap_geometry(op, p, sg);
    if (rc) return rc;
    if (!x || !b) return fail(WDIRAC_EINVAL, "null field pointer");
    if (nrhs < 1) return fail(WDIRAC_EINVAL, "nrhs must be >= 1");
    const size_t n = field_rhs_bytes(WDIRAC_F64, op->g.V) * (size_t)nrhs;
    const char *xb = reinterpret_cast<const char *>(x), *bb = reinterpret_cast<const char *>(b);
    if (xb < bb + n && bb < xb + n) return fail(WDIRAC_EINVAL, "x overlaps b");
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(work)) & 15)
        return fail(WDIRAC_EINVAL, "field pointers must be 16-byte aligned");
    const size_t need = sap_workspace(op, p, nrhs);
    if (need && (!work || work_bytes < need)) return fail(WDIRAC_EINVAL, "SAP workspace too small");
    if (need) {
        const char *wb = static_cast<const char *>(work);
        if ((wb < xb + n && xb < wb + need) || (wb < bb + n && bb < wb + need))
            return fail(WDIRAC_EINVAL, "SAP workspace overlaps x or b");
    }
    const hipError_t e = sap_apply(op, *p, sg, reinterpret_cast<double2 *>(x), reinterpret_cast<const double2 *>(b),
                                   nrhs, static_cast<double2 *>(work), 1.0, (hipStream_t)stream);
    if (e != hipSuccess) return fail(WDIRAC_EHIP, std::string("SAP launch: ") + hipGetErrorString(e));
    return WDIRAC_OK;
}

}  // extern "C"

// Fused Wilson-clover stencil (Eq. (1.13); D = D_sc - D_nc of Eqs. (2.5)-(2.7)).
//
// One lane owns one lattice site and a register block of NR right-hand
// sides, and performs in registers what the paper splits into 16 kernel
// launches plus a self-coupling kernel (Algorithm 4 and the clover kernel):
// the self-coupling product A(x) psi(x), then for each of the 8 neighbours
// the spin projection to a half-spinor h = u + s B_mu d (the prp kernels of
// Listing 4.2), the SU(3) product with U_mu(x) or U_mu(x-mu)^H, and the
// reconstruction of the lower half as s B_mu^H (U h) (the back-substitution
// of Sec. 2.2).  Every link and clover entry is loaded once per site and
// register block and used for all NR right-hand sides; nothing but the
// result is written.  The count of right-hand sides and the link format are
// compile-time constants: with branches on either, a hop's spinor loads waited
// for its link and each right-hand side for the one before (site kernel, us,
// 64 x 32^3: FP64 678 -> 568, FP16S 4 RHS 543 -> 460; columns FP32 4 RHS
// 722 -> 686; FP64 48^3 x 96 2735 -> 2696, bound by fabric traffic).
//
// Gamma basis: gamma_mu = [[0, B_mu], [B_mu^H, 0]], B_T = 1, B_Z = -i s3,
// B_Y = -i s2, B_X = -i s1, so the projector (I + s gamma_mu) maps
// (u, d) -> (h, s B_mu^H h) with h = u + s B_mu d.  D uses s = -1 for the
// forward hop and s = +1 for the backward hop; D^H swaps them.
//
// Work decomposition: a work item is (tile of up to 256 consecutive sites,
// register block of right-hand sides).  Items are dealt so that the
// work-group running on XCD k (work-groups go to the 8 XCDs round-robin)
// always gets tiles of the same 1/8 of every T-slice, and all XCDs advance
// through the T-slices together: the T-neighbours of a slice are then read
// while the slice is still in the Infinity Cache, and the Z-neighbours
// mostly come from the same XCD's L2.  The register blocks of one tile are
// consecutive items on the same XCD, so their shared links and clover stay
// in that XCD's L2 while it can hold them.  With fewer work-groups than
// items (an optional persistent grid) each work-group strides through the
// item list.
#include "spinor_io.h"
#include "stencil.h"
#include "dslash.h"

namespace wd {

struct Nbr {
    int fwd[4], bwd[4];
    bool fwd_wrapT, bwd_wrapT;
};

__device__ __forceinline__ Nbr neighbours(const Geom &g, int s) {
    Nbr n;
    int c[4];
    int r = s;
    c[3] = r % g.n[3]; r /= g.n[3];
    c[2] = r % g.n[2]; r /= g.n[2];
    c[1] = r % g.n[1];
    c[0] = r / g.n[1];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        int st = g.stride[mu], L = g.n[mu];
        n.fwd[mu] = (c[mu] == L - 1) ? s - (L - 1) * st : s + st;
        n.bwd[mu] = (c[mu] == 0) ? s + (L - 1) * st : s - st;
    }
    n.fwd_wrapT = c[0] == g.n[0] - 1;
    n.bwd_wrapT = c[0] == 0;
    return n;
}

// acc += f (1 + S gamma_mu)-projected hop of the neighbour at site j of every right-hand side, through the link U
// (DAGU: its adjoint)
template <int P, int MU, int S, bool DAGU, int NR>
__device__ __forceinline__ void hop(const cx<typename Store<P>::T> U[9], const Chunk<NR> &ch, int V, int j,
                                    typename Store<P>::T f, cx<typename Store<P>::T> (&acc)[NR][12]) {
    using T = typename Store<P>::T;
#pragma unroll
    for (int r = 0; r < NR; r++) {
        Raw<P> x;
        cx<T> h[6], chi[6];
        x.load(ch.in[r], V, j);
        project_raw<MU, S>(x, h);
        su3_mul<DAGU>(U, h, chi);
        reconstruct_scaled<MU, S>(acc[r], chi, x.weight(f));
    }
}

// both hops of direction MU; FENCE: hops between two fences (1, 2, 4 or 8)
template <int P, int MU, bool DAG, int ROWS, int NR, int FENCE>
__device__ __forceinline__ void hop_pair(const Chunk<NR> &ch, const OpData &d, int V, int s, const Nbr &nb,
                                         bool apbc, cx<typename Store<P>::T> (&acc)[NR][12]) {
    using T = typename Store<P>::T;
    constexpr int SF = DAG ? +1 : -1;  // forward projector (I + SF gamma)
    constexpr int SB = -SF;            // backward projector
    cx<T> U[9];
    // forward: -1/2 (I + SF gamma) (x) U_mu(x) psi(x+mu)
    Store<P>::load_link(d.links, V, MU, s, U, ROWS);
    hop<P, MU, SF, false, NR>(U, ch, V, nb.fwd[MU], (MU == 0 && apbc && nb.fwd_wrapT) ? T(0.5) : T(-0.5), acc);
    if (FENCE == 1) hop_boundary<T, NR>(acc);
    // backward: -1/2 (I + SB gamma) (x) U_mu(x-mu)^H psi(x-mu)
    Store<P>::load_link(d.links, V, MU, nb.bwd[MU], U, ROWS);
    hop<P, MU, SB, true, NR>(U, ch, V, nb.bwd[MU], (MU == 0 && apbc && nb.bwd_wrapT) ? T(0.5) : T(-0.5), acc);
    if (MU == 3 || FENCE <= 2 || (MU == 1 && FENCE == 4)) hop_boundary<T, NR>(acc);
}

// acc = A(x) x of every right-hand side, x(r, b, v) giving chirality block b of the r-th
template <int P, int NR, typename X>
__device__ __forceinline__ void self_term(const OpData &d, int V, int s, X x,
                                          cx<typename Store<P>::T> (&acc)[NR][12]) {
    using T = typename Store<P>::T;
#pragma unroll
    for (int b = 0; b < 2; b++) {
        if (d.clover_compact) {
            T cr[28];
            Store<P>::load_clover_compact(d.clover, V, b, s, cr);
#pragma unroll
            for (int r = 0; r < NR; r++) {
                cx<T> p[6];
                x(r, b, p);
                clover_block_compact((T)d.diag, cr, p, &acc[r][6 * b]);
            }
        } else {
            T dd[6];
            cx<T> uu[15];
            Store<P>::load_clover(d.clover, V, b, s, dd, uu);
#pragma unroll
            for (int r = 0; r < NR; r++) {
                cx<T> p[6];
                x(r, b, p);
                clover_block(dd, uu, p, &acc[r][6 * b]);
            }
        }
    }
}

template <int P, bool DAG, int ROWS, int NR, int FENCE>
__device__ __forceinline__ void site_apply(const Chunk<NR> &ch, const OpData &d, const Geom &g, int s, bool apbc) {
    using T = typename Store<P>::T;
    const int V = g.V;
    cx<T> acc[NR][12];
    self_term<P, NR>(d, V, s, [&](int r, int b, cx<T> *p) { Store<P>::load_half(ch.in[r], V, s, b, p); }, acc);
    const Nbr nb = neighbours(g, s);
    hop_boundary<T, NR>(acc);
    hop_pair<P, 0, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, apbc, acc);
    hop_pair<P, 1, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, apbc, acc);
    hop_pair<P, 2, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, apbc, acc);
    hop_pair<P, 3, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, apbc, acc);
#pragma unroll
    for (int r = 0; r < NR; r++) Store<P>::store_spinor(ch.out[r], V, s, acc[r]);
}

// Register T-sweep (tile order 3): one lane walks the sites t0..t1-1 of one
// column (z, y, x).  psi(t+1) is loaded once as the forward T neighbour and
// kept as the next step's own spinor, and the backward T hop of site t+1,
// -1/2 (I + SB gamma_T) (x) U_T(t)^H psi(t), is formed at step t and carried
// in registers, so no T-neighbour spinor or backward T link is re-read.
template <int P, bool DAG, int ROWS, int NR, int FENCE>
__device__ __forceinline__ void column_sweep(const Chunk<NR> &ch, const OpData &d, const Geom &g, int c, int t0,
                                             int t1, bool apbc, cx<typename Store<P>::T> (*ut_lds)[9]) {
    using T = typename Store<P>::T;
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    const int V = g.V, S = g.stride[0], nT = g.n[0];
    // neighbour columns in Z, Y, X
    int cf[4], cb[4];
    {
        int r = c, q[4];
        q[3] = r % g.n[3]; r /= g.n[3];
        q[2] = r % g.n[2];
        q[1] = r / g.n[2];
#pragma unroll
        for (int mu = 1; mu < 4; mu++) {
            const int st = g.stride[mu], L = g.n[mu];
            cf[mu] = (q[mu] == L - 1) ? c - (L - 1) * st : c + st;
            cb[mu] = (q[mu] == 0) ? c + (L - 1) * st : c - st;
        }
    }
    Raw<P> self[NR];
    cx<T> chiT[NR][6];  // carried product and its weight
    T wT[NR];
    {
        const int tm = (t0 == 0) ? nT - 1 : t0 - 1;
        const T f = (apbc && t0 == 0) ? T(0.5) : T(-0.5);
        cx<T> U[9];
        Store<P>::load_link(d.links, V, 0, tm * S + c, U, ROWS);
#pragma unroll
        for (int r = 0; r < NR; r++) {
            Raw<P> x;
            cx<T> h[6];
            x.load(ch.in[r], V, tm * S + c);
            self[r].load(ch.in[r], V, t0 * S + c);
            project_raw<0, SB>(x, h);
            su3_mul<true>(U, h, chiT[r]);
            wT[r] = x.weight(f);
        }
    }
    for (int t = t0; t < t1; t++) {
        const int s = t * S + c;
        cx<T> acc[NR][12];
        self_term<P, NR>(d, V, s, [&](int r, int b, cx<T> *p) { self[r].half(b, p); }, acc);
        // backward T hop (carried), then the one for site t+1
        const bool last = (t == nT - 1);
        // U_T(s) serves both T hops of the step; the copy parked in the lane's LDS slot between them spares a
        // second load through the L2, which by then has often evicted it (measured: -75 B read per site)
        {
            const T f = (apbc && last) ? T(0.5) : T(-0.5);
            cx<T> U[9];
            Store<P>::load_link(d.links, V, 0, s, U, ROWS);
#pragma unroll
            for (int e = 0; e < 9; e++) ut_lds[threadIdx.x][e] = U[e];
#pragma unroll
            for (int r = 0; r < NR; r++) {
                reconstruct_scaled<0, SB>(acc[r], chiT[r], wT[r]);
                cx<T> h[6];
                project_raw<0, SB>(self[r], h);
                su3_mul<true>(U, h, chiT[r]);
                wT[r] = self[r].weight(f);
            }
        }
        hop_boundary<T, NR>(acc);
        Nbr nb;
#pragma unroll
        for (int mu = 1; mu < 4; mu++) {
            nb.fwd[mu] = t * S + cf[mu];
            nb.bwd[mu] = t * S + cb[mu];
        }
        nb.fwd[0] = nb.bwd[0] = s;
        nb.fwd_wrapT = nb.bwd_wrapT = false;
        hop_pair<P, 1, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, false, acc);
        hop_pair<P, 2, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, false, acc);
        hop_pair<P, 3, DAG, ROWS, NR, FENCE>(ch, d, V, s, nb, false, acc);
        // forward T hop; psi(t+1) becomes the next step's own spinor
        {
            const int sp = (last ? 0 : t + 1) * S + c;
            const T f = (apbc && last) ? T(0.5) : T(-0.5);
            cx<T> U[9];
#pragma unroll
            for (int e = 0; e < 9; e++) U[e] = ut_lds[threadIdx.x][e];
#pragma unroll
            for (int r = 0; r < NR; r++) {
                cx<T> h[6], chi[6];
                self[r].load(ch.in[r], V, sp);
                project_raw<0, SF>(self[r], h);
                su3_mul<false>(U, h, chi);
                reconstruct_scaled<0, SF>(acc[r], chi, self[r].weight(f));
            }
        }
#pragma unroll
        for (int r = 0; r < NR; r++) Store<P>::store_spinor(ch.out[r], V, s, acc[r]);
        hop_boundary<T, NR>(acc);
    }
}

// site range [lo, hi) of tile slot vb (see TileMap in dslash.h); hi may lie before lo
__device__ __forceinline__ void tile_range(const TileMap &m, int vb, int &lo, int &hi) {
    if (m.order == kOrderTSweep) {
        const int k = vb & 7, j = vb >> 3;
        const int t = j / m.tiles_per_range, tile = j - t * m.tiles_per_range;
        const int base = t * m.slice;
        const int r0 = base + (int)(((long long)k * m.slice) >> 3);
        const int r1 = base + (int)(((long long)(k + 1) * m.slice) >> 3);
        lo = r0 + tile * m.block;
        hi = min(lo + m.block, min(r1, m.V));
    } else if (m.order == kOrderZPlanes) {
        const int k = vb & 7, j = vb >> 3;
        const int q = j / m.plane_tiles, tile = j - q * m.plane_tiles;
        const int zb = q / m.nt, t = q - zb * m.nt;
        const int z = zb * 8 + k;
        const int plane = m.slice / m.nz;
        lo = hi = 0;
        if (z < m.nz) {
            const int base = (t * m.nz + z) * plane;
            lo = base + tile * m.block;
            hi = min(lo + m.block, base + plane);
        }
    } else {
        int tile = vb;
        if (m.order == kOrderXcdChunk) {
            // contiguous ranges of tiles per XCD
            const int q = m.ntiles >> 3, rr = m.ntiles & 7;
            const int k = vb & 7, j = vb >> 3;
            tile = k * q + (k < rr ? k : rr) + j;
        }
        lo = tile * m.block;
        hi = min(lo + m.block, m.V);
    }
}

// site of lane l of tile slot vb in kOrderZGroups (-1: no site): XCD k takes the groups of zw consecutive z-planes
// (zw p, ..., zw p + zw - 1) with p = k mod 8, group-block by group-block, each block's T-planes in order; a tile
// is 64 consecutive (y, x) sites, wave w of the work-group in plane zw p + w
__device__ __forceinline__ int zgroup_site(const TileMap &m, int vb, int l) {
    const int k = vb & 7, j = vb >> 3;
    const int nxyb = (m.plane_tiles + m.xyb - 1) / m.xyb;
    const int tl = j % m.xyb, q = j / m.xyb;
    const int t = q % m.nt, r = q / m.nt;
    const int xyb = r % nxyb, zb = r / nxyb;
    const int tile = xyb * m.xyb + tl;
    const int z = m.zw * (zb * 8 + k) + (l >> 6);
    const int plane = m.slice / m.nz;
    const int xy = tile * 64 + (l & 63);
    if (z >= m.nz || tile >= m.plane_tiles || xy >= plane) return -1;
    return (t * m.nz + z) * plane + xy;
}

// Hops between two fences and waves per SIMD the registers must allow, of the
// site kernel: FP64 keeps one hop's loads in flight (two: 568 -> 581 us at
// 64 x 32^3), FP32 and FP16S issue the loads of several hops together.
template <int P, int NR> constexpr int site_fence() {
    return (P == WDIRAC_F64 || NR == 4) ? 1 : (P == WDIRAC_F16S && NR == 1) ? 8 : 4;
}
template <int P, int NR> constexpr int occupancy() {
    return P == WDIRAC_F64 ? (NR == 4 ? 1 : 2) : P == WDIRAC_F32 ? (NR == 1 ? 4 : 2) : (NR == 4 ? 2 : 3);
}

template <int P, bool DAG, int ROWS, int NR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(occupancy<P, NR>())))
void dslash_kernel(ChunkTable<NR> tab, OpData d, Geom g, TileMap m, int apbc) {
    const int nitems = m.nslots * tab.nchunks;   // nslots is a multiple of 8
    for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
        // XCD-affine dealing: w % 8 == vb % 8, consecutive items of one XCD
        // walk through the register blocks of a tile before the next tile
        const int xcd = w & 7, q = w >> 3;
        const int vb = (q / tab.nchunks) * 8 + xcd;
        const int c = q - (q / tab.nchunks) * tab.nchunks;
        int lo, hi;
        tile_range(m, vb, lo, hi);
        const int s = lo + (int)threadIdx.x;
        if (s < hi) site_apply<P, DAG, ROWS, NR, site_fence<P, NR>()>(tab.c[c], d, g, s, apbc != 0);
    }
}

// right-hand sides k .. k + N of a register block as a block of their own
template <int N, int NR> __device__ __forceinline__ Chunk<N> sub_chunk(const Chunk<NR> &c, int k) {
    Chunk<N> o;
#pragma unroll
    for (int r = 0; r < N; r++) {
        o.in[r] = c.in[k + r];
        o.out[r] = c.out[k + r];
    }
    return o;
}

// dslash_kernel with a last register block of `rest` < NR right-hand sides, tab.c[tab.nchunks].  As launches of their own
// the last few left most of the chip idle (us, three right-hand sides, 16^4 FP32 25.6 -> 18.1, 24 x 16^2 x 24 FP32 59.5
// -> 51.3; seven at 12^4 FP64 43 -> 31).  FP64 and FP32 take it in its tile's turn (after all whole blocks: 51.4 -> 61.1),
// FP16S after all whole blocks (32^4, three: 183, in turn 200).  A kernel of its own, since the second path would change
// the whole blocks' registers.
template <int P, bool DAG, int ROWS, int NR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(occupancy<P, NR>())))
void dslash_rest_kernel(ChunkTable<NR> tab, OpData d, Geom g, TileMap m, int apbc, int rest) {
    constexpr bool in_turn = P != WDIRAC_F16S;
    const int blocks = tab.nchunks + (in_turn ? 1 : 0), nitems = m.nslots * (tab.nchunks + 1);
    for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
        const bool after = !in_turn && w >= m.nslots * blocks;  // nslots is a multiple of 8
        const int xcd = w & 7, q = w >> 3;
        const int vb = after ? w - m.nslots * blocks : (q / blocks) * 8 + xcd;
        const int c = after ? tab.nchunks : q - (q / blocks) * blocks;
        int lo, hi;
        tile_range(m, vb, lo, hi);
        const int s = lo + (int)threadIdx.x;
        if (s >= hi) continue;
        if (c < tab.nchunks) {
            site_apply<P, DAG, ROWS, NR, site_fence<P, NR>()>(tab.c[c], d, g, s, apbc != 0);
            continue;
        }
        const Chunk<NR> &ch = tab.c[tab.nchunks];
        if (NR == 4 && (rest & 2))
            site_apply<P, DAG, ROWS, 2, site_fence<P, 2>()>(sub_chunk<2>(ch, 0), d, g, s, apbc != 0);
        if (rest & 1)
            site_apply<P, DAG, ROWS, 1, site_fence<P, 1>()>(sub_chunk<1>(ch, rest - 1), d, g, s, apbc != 0);
    }
}

// the same for the column kernel, which carries psi(t+1) and the T half-spinors
template <int P, int NR> constexpr int column_fence() {
    return P == WDIRAC_F64 ? (NR == 1 ? 2 : 4) : P == WDIRAC_F32 ? 4 : 8;
}
template <int P, int NR> constexpr int occupancy_col() { return NR == 1 ? 2 : 1; }
// One FP32 right-hand side with two-row links: two hops between fences and three waves per SIMD at most.  Its registers
// allow four, whose columns displace each other's neighbours from the L2; two are too few where the columns are just more
// than two per SIMD (us, four hops and four waves, this, four hops and two waves: 48^3 x 96 T-chunk 2 1385 / 1348 / 1339,
// 64 x 32^3 286 / 273 / 265, 48 x 24^3 82 / 84 / 93).  With full links it gains nothing (32^4 170 / 172 / 182).
template <int P, int ROWS, int NR> constexpr bool column_few() { return P == WDIRAC_F32 && ROWS == 2 && NR == 1; }
// column and T range of a lane of tile slot vb: the columns of XCD k's 1/8 of a slice (or of its patches), T-chunk tc;
// -1: none
__device__ __forceinline__ int tile_column(const TileMap &m, const Geom &g, int vb, int &t0, int &t1) {
    const int k = vb & 7, j = vb >> 3;
    const int tc = j / m.tiles_per_range, tile = j - tc * m.tiles_per_range;
    t0 = tc * m.tchunk;
    t1 = min(t0 + m.tchunk, g.n[0]);
    int col = -1;
    if (m.order == kOrderPatch) {
        const int p0 = (int)(((long long)k * m.patches) >> 3), p1 = (int)(((long long)(k + 1) * m.patches) >> 3);
        const int pi = p0 + tile;
        const int lx = (int)threadIdx.x % kPatchX, ly = ((int)threadIdx.x / kPatchX) % kPatchY,
                  lz = (int)threadIdx.x / (kPatchX * kPatchY);
        const int px = pi % m.npx, py = (pi / m.npx) % m.npy, pzi = pi / (m.npx * m.npy);
        const int x = px * kPatchX + lx, y = py * kPatchY + ly, z = pzi * m.pz + lz;
        if (pi < p1 && x < g.n[3] && y < g.n[2] && z < g.n[1]) col = (z * g.n[2] + y) * g.n[3] + x;
    } else {
        const int r0 = (int)(((long long)k * m.slice) >> 3), r1 = (int)(((long long)(k + 1) * m.slice) >> 3);
        const int cc = r0 + tile * m.block + (int)threadIdx.x;
        if (cc < r1) col = cc;
    }
    return t0 < t1 ? col : -1;
}

template <int P, bool DAG, int ROWS, int NR>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(occupancy_col<P, NR>(), column_few<P, ROWS, NR>() ? 3 : 8)))
void dslash_column_kernel(ChunkTable<NR> tab, OpData d, Geom g, TileMap m, int apbc) {
    __shared__ cx<typename Store<P>::T> ut_lds[256][9];
    const int nitems = m.nslots * tab.nchunks;
    for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
        const int xcd = w & 7, q = w >> 3;
        const int vb = (q / tab.nchunks) * 8 + xcd;
        const int c = q - (q / tab.nchunks) * tab.nchunks;
        int t0, t1;
        const int col = tile_column(m, g, vb, t0, t1);
        if (col >= 0)
            column_sweep<P, DAG, ROWS, NR, column_few<P, ROWS, NR>() ? 2 : column_fence<P, NR>()>(
                tab.c[c], d, g, col, t0, t1, apbc != 0, ut_lds);
    }
}

// the same with a lone last right-hand side, tab.c[tab.nchunks], after all pairs: its work-groups fill the pairs' last
// round (us, as a launch of its own and now: 48 x 24^3 five FP64 751 -> 697, FP32 396 -> 321)
template <int P, bool DAG, int ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(occupancy_col<P, 2>())))
void dslash_column_rest_kernel(ChunkTable<2> tab, OpData d, Geom g, TileMap m, int apbc) {
    __shared__ cx<typename Store<P>::T> ut_lds[256][9];
    const int pairs = m.nslots * tab.nchunks, nitems = pairs + m.nslots;  // nslots is a multiple of 8
    for (int w = blockIdx.x; w < nitems; w += gridDim.x) {
        const int xcd = w & 7, q = w >> 3;
        const bool lone = w >= pairs;
        const int vb = lone ? w - pairs : (q / tab.nchunks) * 8 + xcd;
        int t0, t1;
        const int col = tile_column(m, g, vb, t0, t1);
        if (col < 0) continue;
        if (lone)
            column_sweep<P, DAG, ROWS, 1, column_fence<P, 1>()>(sub_chunk<1>(tab.c[tab.nchunks], 0), d, g, col, t0, t1,
                                                                apbc != 0, ut_lds);
        else
            column_sweep<P, DAG, ROWS, 2, column_fence<P, 2>()>(tab.c[q - (q / tab.nchunks) * tab.nchunks], d, g, col,
                                                                t0, t1, apbc != 0, ut_lds);
    }
}

// Link-stationary multi-RHS stencil (FP32 compute, two-row links): a lane
// loads the 8 links it needs (rows 0 and 1 of U_mu(x) and U_mu(x-mu), 96
// registers) and stages its own clover blocks in LDS once, then walks every
// right-hand side of the launch reading only spinors.  Links and clover
// are thus read from memory once per launch instead of once per register
// block, which a 4 MB L2 per XCD cannot provide when many right-hand sides
// stream through.  The LDS slots are private to their lane (no barrier).
// Per right-hand side the arithmetic is that of dslash_kernel (same order).
template <int P, bool DAG>
__global__ __launch_bounds__(kStationaryBlock) __attribute__((amdgpu_waves_per_eu(2)))
void dslash_stationary_kernel(RhsTable tab, OpData d, Geom g, TileMap m, int apbc) {
    using T = typename Store<P>::T;
    static_assert(P != WDIRAC_F64, "FP64 links do not fit in registers");
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    __shared__ float4 lds[18][kStationaryBlock];
    int s;
    if (m.order == kOrderZGroups) {
        s = zgroup_site(m, blockIdx.x, threadIdx.x);
        if (s < 0) return;
    } else {
        int lo, hi;
        tile_range(m, blockIdx.x, lo, hi);
        s = lo + (int)threadIdx.x;
        if (s >= hi) return;
    }
    const int V = g.V;
    const int tid = threadIdx.x;
    const bool compact = d.clover_compact != 0;
#pragma unroll
    for (int b = 0; b < 2; b++) {
        if (compact) {
            T cr[28];
            Store<P>::load_clover_compact(d.clover, V, b, s, cr);
#pragma unroll
            for (int k = 0; k < 7; k++)
                lds[7 * b + k][tid] = make_float4(-2 * cr[4 * k], -2 * cr[4 * k + 1], -2 * cr[4 * k + 2], -2 * cr[4 * k + 3]);
        } else {
            T dd[6];
            cx<T> uu[15];
            Store<P>::load_clover(d.clover, V, b, s, dd, uu);
            lds[9 * b + 0][tid] = make_float4(-2 * dd[0], -2 * dd[1], -2 * dd[2], -2 * dd[3]);
            lds[9 * b + 1][tid] = make_float4(-2 * dd[4], -2 * dd[5], -2 * uu[0].r, -2 * uu[0].i);
#pragma unroll
            for (int k = 0; k < 7; k++)
                lds[9 * b + 2 + k][tid] = make_float4(-2 * uu[1 + 2 * k].r, -2 * uu[1 + 2 * k].i, -2 * uu[2 + 2 * k].r,
                                                      -2 * uu[2 + 2 * k].i);
        }
    }
    const T dg = T(-2) * (T)d.diag;
    const Nbr nb = neighbours(g, s);
    cx<T> Lf[4][6], Lb[4][6];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        cx<T> U[9];
        Store<P>::load_link(d.links, V, mu, s, U, 2);
#pragma unroll
        for (int e = 0; e < 6; e++) Lf[mu][e] = U[e];
        Store<P>::load_link(d.links, V, mu, nb.bwd[mu], U, 2);
#pragma unroll
        for (int e = 0; e < 6; e++) Lb[mu][e] = U[e];
    }
    // everything up to the store is accumulated scaled by -2 (exact): the clover
    // blocks were staged times -2, the hop projections drop their factor -1/2
    // (an anti-periodic T wrap keeps a sign), and -1/2 is applied once at the end
    const T ffT = (apbc && nb.fwd_wrapT) ? T(-1) : T(1);
    const T fbT = (apbc && nb.bwd_wrapT) ? T(-1) : T(1);
    for (int r = 0; r < tab.n; r++) {
        const void *in = tab.in[r];
        cx<T> accs[1][12];
        cx<T>(&acc)[12] = accs[0];
        {
            cx<T> self[12];
            Store<P>::load_spinor(in, V, s, self);
#pragma unroll
            for (int b = 0; b < 2; b++) {
                if (compact) {
                    T cr[28];
#pragma unroll
                    for (int k = 0; k < 7; k++) {
                        const float4 q = lds[7 * b + k][tid];
                        cr[4 * k] = q.x; cr[4 * k + 1] = q.y; cr[4 * k + 2] = q.z; cr[4 * k + 3] = q.w;
                    }
                    clover_block_compact(dg, cr, &self[6 * b], &acc[6 * b]);
                } else {
                    T dd[6];
                    cx<T> uu[15];
                    const float4 a0 = lds[9 * b][tid], a1 = lds[9 * b + 1][tid];
                    dd[0] = a0.x; dd[1] = a0.y; dd[2] = a0.z; dd[3] = a0.w; dd[4] = a1.x; dd[5] = a1.y;
                    uu[0] = {a1.z, a1.w};
#pragma unroll
                    for (int k = 0; k < 7; k++) {
                        const float4 q = lds[9 * b + 2 + k][tid];
                        uu[1 + 2 * k] = {q.x, q.y};
                        uu[2 + 2 * k] = {q.z, q.w};
                    }
                    clover_block(dd, uu, &self[6 * b], &acc[6 * b]);
                }
            }
        }
        hop_boundary<T, 1>(accs);
#define WD_STAT_HOP(MU)                                                         \
        {                                                                       \
            cx<T> U[9], h[6], chi[6];                                           \
            Raw<P> x;                                                           \
            _Pragma("unroll") for (int e = 0; e < 6; e++) U[e] = Lf[MU][e];     \
            third_row(U);                                                       \
            x.load(in, V, nb.fwd[MU]);                                          \
            project_raw<MU, SF>(x, h);                                          \
            su3_mul<false>(U, h, chi);                                          \
            reconstruct_scaled<MU, SF>(acc, chi, x.weight(MU == 0 ? ffT : T(1))); \
        }                                                                       \
        {                                                                       \
            cx<T> U[9], h[6], chi[6];                                           \
            Raw<P> x;                                                           \
            _Pragma("unroll") for (int e = 0; e < 6; e++) U[e] = Lb[MU][e];     \
            third_row(U);                                                       \
            x.load(in, V, nb.bwd[MU]);                                          \
            project_raw<MU, SB>(x, h);                                          \
            su3_mul<true>(U, h, chi);                                           \
            reconstruct_scaled<MU, SB>(acc, chi, x.weight(MU == 0 ? fbT : T(1))); \
        }                                                                       \
        hop_boundary<T, 1>(accs);
        WD_STAT_HOP(0)
        WD_STAT_HOP(1)
        WD_STAT_HOP(2)
        WD_STAT_HOP(3)
#undef WD_STAT_HOP
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = T(-0.5) * acc[k];
        Store<P>::store_spinor(tab.out[r], V, s, acc);
    }
}

// Small lattices: a launch of a few hundred waves is one long chain of loads, eight hops after one another, on a chip
// that is mostly idle.  Here a work-group of four waves takes 64 sites of one right-hand side; wave mu forms the two
// products of direction mu (waves 2 and 3 also one block each of A(x) psi(x)) and leaves them in LDS, then wave s adds
// spin s up in the site kernel's order, so the bits are the site kernel's.  us against the site kernel: 8^4 FP64
// 7.8 -> 6.3, FP32 6.6 -> 4.9, FP16S 6.6 -> 5.0; 10^4 9.0 -> 7.0, 7.4 -> 5.6, 7.3 -> 5.4; FP64 12^4 10.5 -> 9.8 but
// two right-hand sides 11.2 -> 16.3 (65 KB of LDS: two work-groups per CU), FP32 14^4 9.0 -> 8.7, two 11.6 -> 13.0.
template <int P> struct SplitLds {
    using T = typename Store<P>::T;
    cx<T> chi[8][6][64];  // hop 2 mu (forward), 2 mu + 1 (backward)
    T f[8][64];           // its factor times the neighbour's scale
    cx<T> res[12][64];
};

template <int P, int MU, int S, int SPIN>
__device__ __forceinline__ void split_add(const SplitLds<P> &m, int h, int l, cx<typename Store<P>::T> (&acc)[3]) {
    using T = typename Store<P>::T;
    const T f = m.f[h][l], w = (SPIN < 2 || S > 0) ? f : -f;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cx<T> c0 = m.chi[h][c][l], c1 = m.chi[h][3 + c][l];
        cx<T> v;
        if (SPIN == 0) v = c0;
        else if (SPIN == 1) v = c1;
        else if (SPIN == 2) v = MU == 0 ? c0 : MU == 1 ? times_i(c0) : MU == 2 ? c1 : times_i(c1);
        else v = MU == 0 ? c1 : MU == 1 ? times_mi(c1) : MU == 2 ? mk<T>(-c0.r, -c0.i) : times_i(c0);
        acc[c] = {fma(w, v.r, acc[c].r), fma(w, v.i, acc[c].i)};
    }
}

template <int P, bool DAG, int SPIN> __device__ __forceinline__ void split_spin(SplitLds<P> &m, int l) {
    using T = typename Store<P>::T;
    constexpr int SF = DAG ? +1 : -1, SB = -SF;
    cx<T> acc[3] = {m.res[3 * SPIN][l], m.res[3 * SPIN + 1][l], m.res[3 * SPIN + 2][l]};
    split_add<P, 0, SF, SPIN>(m, 0, l, acc);
    split_add<P, 0, SB, SPIN>(m, 1, l, acc);
    split_add<P, 1, SF, SPIN>(m, 2, l, acc);
    split_add<P, 1, SB, SPIN>(m, 3, l, acc);
    split_add<P, 2, SF, SPIN>(m, 4, l, acc);
    split_add<P, 2, SB, SPIN>(m, 5, l, acc);
    split_add<P, 3, SF, SPIN>(m, 6, l, acc);
    split_add<P, 3, SB, SPIN>(m, 7, l, acc);
#pragma unroll
    for (int c = 0; c < 3; c++) m.res[3 * SPIN + c][l] = acc[c];
}

template <int P, int MU, bool DAG, int ROWS>
__device__ __forceinline__ void split_hops(SplitLds<P> &m, const void *in, const OpData &d, const Geom &g, int s, int l,
                                           const Nbr &nb, bool apbc) {
    using T = typename Store<P>::T;
    constexpr int SF = DAG ? +1 : -1, SB = -SF;
    cx<T> U[9], B[9], h[6], chi[6];
    Raw<P> x, y;
    Store<P>::load_link(d.links, g.V, MU, s, U, ROWS);
    x.load(in, g.V, nb.fwd[MU]);
    Store<P>::load_link(d.links, g.V, MU, nb.bwd[MU], B, ROWS);
    y.load(in, g.V, nb.bwd[MU]);
    project_raw<MU, SF>(x, h);
    su3_mul<false>(U, h, chi);
#pragma unroll
    for (int k = 0; k < 6; k++) m.chi[2 * MU][k][l] = chi[k];
    m.f[2 * MU][l] = x.weight((MU == 0 && apbc && nb.fwd_wrapT) ? T(0.5) : T(-0.5));
    project_raw<MU, SB>(y, h);
    su3_mul<true>(B, h, chi);
#pragma unroll
    for (int k = 0; k < 6; k++) m.chi[2 * MU + 1][k][l] = chi[k];
    m.f[2 * MU + 1][l] = y.weight((MU == 0 && apbc && nb.bwd_wrapT) ? T(0.5) : T(-0.5));
}

template <int P, int B>
__device__ __forceinline__ void split_self(SplitLds<P> &m, const void *in, const OpData &d, int V, int s, int l) {
    using T = typename Store<P>::T;
    cx<T> p[6], y[6];
    Store<P>::load_half(in, V, s, B, p);
    if (d.clover_compact) {
        T cr[28];
        Store<P>::load_clover_compact(d.clover, V, B, s, cr);
        clover_block_compact((T)d.diag, cr, p, y);
    } else {
        T dd[6];
        cx<T> uu[15];
        Store<P>::load_clover(d.clover, V, B, s, dd, uu);
        clover_block(dd, uu, p, y);
    }
#pragma unroll
    for (int k = 0; k < 6; k++) m.res[6 * B + k][l] = y[k];
}

template <int P, bool DAG, int ROWS>
__global__ __launch_bounds__(256) void dslash_split_kernel(ChunkTable<1> tab, OpData d, Geom g, TileMap m, int apbc) {
    using T = typename Store<P>::T;
    __shared__ SplitLds<P> lds;
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int vb = (q / tab.nchunks) * 8 + xcd;
    const int c = q - (q / tab.nchunks) * tab.nchunks;
    int lo, hi;
    tile_range(m, vb, lo, hi);
    if (lo >= hi) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int s = min(lo + l, hi - 1);  // idle lanes repeat the last site and store nothing
    const void *in = tab.c[c].in[0];
    const Nbr nb = neighbours(g, s);
    switch (wave) {
    case 0: split_hops<P, 0, DAG, ROWS>(lds, in, d, g, s, l, nb, apbc != 0); break;
    case 1: split_hops<P, 1, DAG, ROWS>(lds, in, d, g, s, l, nb, apbc != 0); break;
    case 2:
        split_self<P, 0>(lds, in, d, g.V, s, l);
        split_hops<P, 2, DAG, ROWS>(lds, in, d, g, s, l, nb, apbc != 0);
        break;
    default:
        split_self<P, 1>(lds, in, d, g.V, s, l);
        split_hops<P, 3, DAG, ROWS>(lds, in, d, g, s, l, nb, apbc != 0);
    }
    __syncthreads();
    switch (wave) {
    case 0: split_spin<P, DAG, 0>(lds, l); break;
    case 1: split_spin<P, DAG, 1>(lds, l); break;
    case 2: split_spin<P, DAG, 2>(lds, l); break;
    default: split_spin<P, DAG, 3>(lds, l);
    }
    __syncthreads();
    if (lo + l >= hi) return;
    cx<T> v[12];
#pragma unroll
    for (int k = 0; k < 12; k++) v[k] = lds.res[k][l];
    Store<P>::store_part(tab.c[c].out[0], g.V, s, v, wave);
}

// ---------------------------------------------------------------------------
// host side

TileMap make_tilemap(const Geom &g, int order, int block, int tchunk) {
    TileMap m;
    m.order = order;
    m.block = block;
    m.V = g.V;
    m.slice = g.V / g.n[0];
    m.tchunk = tchunk < 1 ? 1 : (tchunk > g.n[0] ? g.n[0] : tchunk);
    m.patches = m.npx = m.npy = 0;
    m.pz = block / (kPatchX * kPatchY);
    m.nt = g.n[0];
    m.nz = g.n[1];
    m.zw = 1;
    m.xyb = 1;
    m.plane_tiles = 0;
    if (order == kOrderColumn) {
        const int per_range = (m.slice + 7) / 8;
        m.tiles_per_range = (per_range + block - 1) / block;
        m.ntiles = (g.n[0] + m.tchunk - 1) / m.tchunk * 8 * m.tiles_per_range;
    } else if (order == kOrderPatch) {
        m.npx = (g.n[3] + kPatchX - 1) / kPatchX;
        m.npy = (g.n[2] + kPatchY - 1) / kPatchY;
        m.patches = m.npx * m.npy * ((g.n[1] + m.pz - 1) / m.pz);
        m.tiles_per_range = (m.patches + 7) / 8;
        m.ntiles = (g.n[0] + m.tchunk - 1) / m.tchunk * 8 * m.tiles_per_range;
    } else if (order == kOrderZGroups) {
        m.zw = block / 64;
        m.plane_tiles = (m.slice / m.nz + 63) / 64;
        m.xyb = (tchunk >= 1 && tchunk < m.plane_tiles) ? tchunk : m.plane_tiles;
        const int nxyb = (m.plane_tiles + m.xyb - 1) / m.xyb;
        m.ntiles = ((m.nz + m.zw - 1) / m.zw + 7) / 8 * nxyb * m.nt * m.xyb * 8;
    } else if (order == kOrderZPlanes) {
        m.plane_tiles = (m.slice / m.nz + block - 1) / block;
        m.ntiles = (m.nz + 7) / 8 * m.nt * m.plane_tiles * 8;
    } else if (order == kOrderTSweep) {
        // an eighth of a slice below 48 sites: slabs of as many T-slices as keep an eighth within one wave (us, 1024 x
        // 4^3, one right-hand side, by slices and in slabs: FP64 67 -> 19, FP32 37 -> 9.8)
        const int q = m.slice < 384 ? slab_slices(g.n[0], m.slice, 512) : 1;
        m.slice *= q;
        const int per_range = (m.slice + 7) / 8;
        m.tiles_per_range = (per_range + block - 1) / block;
        m.ntiles = (g.n[0] + q - 1) / q * 8 * m.tiles_per_range;
    } else {
        m.tiles_per_range = 0;
        m.ntiles = (g.V + block - 1) / block;
    }
    m.nslots = (m.ntiles + 7) / 8 * 8;
    return m;
}

static Tuning g_tuning;
static std::mutex g_tuning_mu;

std::mutex &tuning_mutex() { return g_tuning_mu; }
Tuning &tuning_unlocked() { return g_tuning; }
Tuning tuning_snapshot() {
    std::lock_guard<std::mutex> lk(g_tuning_mu);
    return g_tuning;
}

// Work-groups of one kernel instance that fit on the device at once.
template <auto Kernel> static int resident_blocks(int block) {
    static int cached[5] = {0, 0, 0, 0, 0};
    const int slot = block / 64;
    if (!cached[slot]) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, Kernel, block, 0) != hipSuccess || cus * per_cu < 8) {
            (void)hipGetLastError();
            return 8;
        }
        cached[slot] = cus * per_cu / 8 * 8;
    }
    return cached[slot];
}

// One launch of `blocks` register blocks over the tiles of m.  A persistent grid has at most the resident work-groups,
// each striding through the item list (by default the hardware dispatcher hands out one work-group per item in order,
// which measured faster).
template <auto Kernel, typename Tab, typename... Rest>
static hipError_t launch_items(int blocks, const Tab &tab, const OpData &d, const Geom &g, const TileMap &m, int apbc,
                               bool persistent, const LaunchCfg &cfg, hipStream_t st, Rest... rest) {
    const Tuning tu = tuning_snapshot();
    long long grid = (long long)m.nslots * blocks;
    if ((persistent && tu.persistent_blocks > 0) || cfg.persistent) {
        long long cap = resident_blocks<Kernel>(cfg.block);
        if (tu.persistent_blocks > 0 && tu.persistent_blocks < cap) cap = tu.persistent_blocks / 8 * 8;
        if (cap < 8) cap = 8;
        if (grid > cap) grid = cap;
    }
    if (grid > (1LL << 30)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(Kernel, dim3((unsigned)grid), dim3(cfg.block), 0, st, tab, d, g, m, apbc, rest...);
    return hipGetLastError();
}

// Group the right-hand sides of all batches, in order, into register blocks
// of NR (a block may span batches), the remainder into a smaller last one.
template <int P, bool DAG, int ROWS, int NR>
static hipError_t launch_nr(const std::pair<const void *, void *> *rhs, size_t n, const OpData &d, const Geom &g,
                            int apbc, bool persistent, const LaunchCfg &cfg, hipStream_t st) {
    constexpr int NRC = NR > 2 ? 2 : NR;  // the column kernels take at most two right-hand sides per lane
    const TileMap m = make_tilemap(g, cfg.order, cfg.block, cfg.tchunk);
    const bool column = is_column_order(m.order);
    if (column && NR != NRC) return hipErrorInvalidValue;
    size_t rest = n % NR;
    for (size_t k = 0; k + NR <= n;) {
        ChunkTable<NR> tab;
        tab.nchunks = (int)std::min((n - k) / NR, (size_t)kMaxChunks);
        for (int i = 0; i < tab.nchunks * NR; i++, k++) {
            tab.c[i / NR].in[i % NR] = rhs[k].first;
            tab.c[i / NR].out[i % NR] = rhs[k].second;
        }
        hipError_t e = hipSuccess;
        if constexpr (NR > 1) {
            if (rest && k + rest == n && tab.nchunks < kMaxChunks) {
                for (size_t i = 0; i < rest; i++) {
                    tab.c[tab.nchunks].in[i] = rhs[k + i].first;
                    tab.c[tab.nchunks].out[i] = rhs[k + i].second;
                }
                if (!column)
                    return launch_items<&dslash_rest_kernel<P, DAG, ROWS, NR>>(tab.nchunks + 1, tab, d, g, m, apbc,
                                                                               persistent, cfg, st, (int)rest);
                if constexpr (NR == 2)
                    return launch_items<&dslash_column_rest_kernel<P, DAG, ROWS>>(tab.nchunks + 1, tab, d, g, m, apbc,
                                                                                  persistent, cfg, st);
            }
        }
        if (!column)
            e = launch_items<&dslash_kernel<P, DAG, ROWS, NR>>(tab.nchunks, tab, d, g, m, apbc, persistent, cfg, st);
        else if constexpr (NR == NRC)
            e = launch_items<&dslash_column_kernel<P, DAG, ROWS, NR>>(tab.nchunks, tab, d, g, m, apbc, persistent, cfg,
                                                                      st);
        if (e != hipSuccess) return e;
    }
    // fewer than one block, or the table was full
    if constexpr (NR > 1)
        if (rest)
            return launch_nr<P, DAG, ROWS, NR / 2>(rhs + (n - rest), rest, d, g, apbc, persistent, cfg, st);
    return hipSuccess;
}

template <int P, bool DAG, int ROWS>
static hipError_t launch_split(const std::vector<std::pair<const void *, void *>> &rhs, const OpData &d, const Geom &g,
                               int apbc, hipStream_t st) {
    const TileMap m = make_tilemap(g, kOrderTSweep, 64, 1);
    for (size_t c0 = 0; c0 < rhs.size(); c0 += kMaxChunks) {
        ChunkTable<1> tab;
        tab.nchunks = (int)std::min(rhs.size() - c0, (size_t)kMaxChunks);
        for (int i = 0; i < tab.nchunks; i++) {
            tab.c[i].in[0] = rhs[c0 + i].first;
            tab.c[i].out[0] = rhs[c0 + i].second;
        }
        hipLaunchKernelGGL((dslash_split_kernel<P, DAG, ROWS>), dim3(m.nslots * tab.nchunks), dim3(256), 0, st, tab, d,
                           g, m, apbc);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int P, bool DAG, int ROWS>
static hipError_t launch_rows(const std::vector<std::pair<const void *, void *>> &rhs, const OpData &d, const Geom &g,
                              int apbc, bool persistent, const LaunchCfg &cfg, hipStream_t st) {
    if (cfg.order == kOrderSplit) return launch_split<P, DAG, ROWS>(rhs, d, g, apbc, st);
    if (cfg.nr >= 4 && !is_column_order(cfg.order))
        return launch_nr<P, DAG, ROWS, 4>(rhs.data(), rhs.size(), d, g, apbc, persistent, cfg, st);
    if (cfg.nr >= 2)
        return launch_nr<P, DAG, ROWS, 2>(rhs.data(), rhs.size(), d, g, apbc, persistent, cfg, st);
    return launch_nr<P, DAG, ROWS, 1>(rhs.data(), rhs.size(), d, g, apbc, persistent, cfg, st);
}

// Link-stationary launch: all right-hand sides of all batches, in groups of
// `group` (2 .. kMaxStationaryRhs - 1; else kMaxStationaryRhs) per launch,
// one work-group of kStationaryBlock lanes per tile.  Measurements below are
// FP32 and FP16S, 41 RHS at 48^3 x 96, all results bit-identical.
// - Plane tiles (zw = 1: 128 consecutive sites of one (t, z) plane; each XCD
//   walks the T-planes of every eighth z in T order) keep a site's
//   T-neighbours in work-groups that run at the same time, a few right-hand
//   sides apart; with T-slice tiles the next slice only started after the
//   current one had walked every right-hand side (FP32 44.0 -> 39.5 ms, FP16S
//   27.5 -> 25.7 ms).  Both z-neighbours are planes of other XCDs.
// - Z-pair tiles (zw >= 2: the two waves take the same 64 (y, x) sites of
//   planes z and z + 1) read one of the two z-neighbours inside the
//   work-group (FP32 groups of 12: 33.7 ms; four z-planes in 256-lane
//   work-groups were slower, 41 ms).  With zw = 4 an XCD walks its z-pairs
//   along T in blocks of about eight x-rows before the next block, so a
//   T-neighbour's tile ran only a few work-groups earlier (FP32 groups of
//   16: 30.3 ms; FP16S in one launch 24.3 ms; blocks of whole rows measured
//   faster than ragged ones).
// - Smaller groups re-read the links and clover once per launch but shorten
//   the time between the uses of a neighbour spinor (FP32 plane tiles: groups
//   of 6 36.4 ms, all in one launch 39.7 ms; FP16S is fastest in one launch).
template <int P, bool DAG>
static hipError_t launch_stationary(const dirac_batch *batches, int nbatch, const OpData &d, const Geom &g,
                                    int apbc, int group, int zw, hipStream_t st) {
    const size_t rb = field_rhs_bytes(P, g.V);
    std::vector<std::pair<const void *, void *>> rhs;
    for (int b = 0; b < nbatch; b++)
        for (int r = 0; r < batches[b].nrhs; r++)
            rhs.emplace_back(static_cast<const char *>(batches[b].in) + r * rb,
                             static_cast<char *>(batches[b].out) + r * rb);
    static_assert(kStationaryBlock == 128, "z-pair tiles are two waves");
    // zw = 4: z-pair tiles walked along T in (y, x) blocks of about eight x-rows (0: whole planes)
    const int xyb = zw == 4 ? (8 * g.n[3] + 63) / 64 : 0;
    const TileMap m = make_tilemap(g, zw >= 2 ? kOrderZGroups : kOrderZPlanes, kStationaryBlock, xyb);
    const size_t grp = (group >= 2 && group < kMaxStationaryRhs) ? (size_t)group : (size_t)kMaxStationaryRhs;
    for (size_t r0 = 0; r0 < rhs.size(); r0 += grp) {
        RhsTable tab;
        tab.n = (int)std::min(grp, rhs.size() - r0);
        for (int i = 0; i < kMaxStationaryRhs; i++) {
            const size_t k = r0 + std::min(i, tab.n - 1);
            tab.in[i] = rhs[k].first;
            tab.out[i] = rhs[k].second;
        }
        hipLaunchKernelGGL((dslash_stationary_kernel<P, DAG>), dim3((unsigned)m.nslots), dim3(kStationaryBlock), 0, st,
                           tab, d, g, m, apbc);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int P, bool DAG>
static hipError_t launch_p(const dirac_batch *batches, int nbatch, const OpData &d, const Geom &g, int apbc,
                           bool persistent, LaunchCfg cfg, hipStream_t st) {
    int total = 0;
    for (int b = 0; b < nbatch; b++) total += batches[b].nrhs;
    if (cfg.order == kOrderStationary) {
        if constexpr (P != WDIRAC_F64) {
            if (d.rows == 2)
                return launch_stationary<P, DAG>(batches, nbatch, d, g, apbc, cfg.tchunk, cfg.nr, st);
        }
        cfg.order = kOrderTSweep;  // FP64 or full links: the register-blocked site kernel
    }
    if (total == 1) cfg.nr = 1;
    if (is_column_order(cfg.order) && cfg.nr > 2) cfg.nr = 2;  // register budget
    const size_t rb = field_rhs_bytes(P, g.V);
    std::vector<std::pair<const void *, void *>> rhs;
    for (int b = 0; b < nbatch; b++)
        for (int r = 0; r < batches[b].nrhs; r++)
            rhs.emplace_back(static_cast<const char *>(batches[b].in) + r * rb,
                             static_cast<char *>(batches[b].out) + r * rb);
    return d.rows == 2 ? launch_rows<P, DAG, 2>(rhs, d, g, apbc, persistent, cfg, st)
                       : launch_rows<P, DAG, 3>(rhs, d, g, apbc, persistent, cfg, st);
}

hipError_t dslash_launch_cfg(const dirac_batch *batches, int nbatch, int prec, bool dagger, const OpData &d,
                             const Geom &g, int apbc, bool persistent, const LaunchCfg &cfg, hipStream_t st) {
    switch (prec) {
    case WDIRAC_F64:
        return dagger ? launch_p<WDIRAC_F64, true>(batches, nbatch, d, g, apbc, persistent, cfg, st)
                      : launch_p<WDIRAC_F64, false>(batches, nbatch, d, g, apbc, persistent, cfg, st);
    case WDIRAC_F32:
        return dagger ? launch_p<WDIRAC_F32, true>(batches, nbatch, d, g, apbc, persistent, cfg, st)
                      : launch_p<WDIRAC_F32, false>(batches, nbatch, d, g, apbc, persistent, cfg, st);
    case WDIRAC_F16S:
        return dagger ? launch_p<WDIRAC_F16S, true>(batches, nbatch, d, g, apbc, persistent, cfg, st)
                      : launch_p<WDIRAC_F16S, false>(batches, nbatch, d, g, apbc, persistent, cfg, st);
    }
    return hipErrorInvalidValue;
}

// Launch configuration of n right-hand sides where none was tuned or set.  Measured best of the site kernel (T-slice
// order) against the column sweep, us, 16^4 / 32 x 16^2 x 32 / 48 x 24^3 / 32^4 / 64 x 32^3, two-row links:
//   FP64 1 RHS   site 16 / 77 / 194 / 290 / 568   column 23 / 68 / 190 / 285 / 567
//   FP64 4 RHS   site 62 / 227 / 555 / 956 / 1922  column 46 / 210 / 500 / 764 / 1533
//   FP32 1 RHS   site 9.5 / 35 / 82 / 129 / 275   column 16 / 35 / 82 / 124 / 283
//   FP32 4 RHS   site 23 / 104 / 259 / 403 / 784   column 25 / 91 / 239 / 352 / 686
//   FP16S 4 RHS  site 18 / 62 / 149 / 232 / 460    column 21 / 62 / 154 / 245 / 477
// The column sweep adds the hops in another order, so its last bits differ from the site kernel's; the choice between
// the two goes by the lattice alone, so that a result does not depend on how many right-hand sides are applied
// together: FP64 walks columns past 2^17 sites (the lanes fill the chip), FP32 from 2^18, FP16S never.  Pairs per
// lane halve the waves: site kernel from 2^17 site-right-hand-sides (FP32 16^4, two: one per lane 12.9, four: pairs
// 22.8; 8^4: pairs 11.9 against 8), FP64 columns from 2^21 (48 x 24^3, two: one per lane 307, pairs 316; 32^4, two:
// pairs 445; three 64 x 32^3 1349 against 1360).  T-chunks of 8 for one or two FP32 right-hand sides from 2^21 on (32^4
// one 119 against 134, two 200 against 206), else 4 (48 x 24^3 four 238 against 291).  The link-stationary kernel (the site kernel's order and bits) takes six and more FP32 right-hand sides
// between 16^4 and 2^18 sites: 12 at 16^4 67 -> 54; at 12^4 25 against 49.  Up to 2^14 site-right-hand-sides at FP64,
// 2^15 else, the small-lattice kernel (measured there; same bits as the site kernel).
// The FP64 site kernel takes two or three right-hand sides and, with full links, any odd count one per lane (us, one per
// lane against pairs: 16 x 12 x 24^2 two 55 / 58, 20 x 32 x 20 x 24 two 138 / 159; 16^4 three 43 / 50, full links seven
// 99 / 122; 64 x 4 x 12^2 full links five 54 / 63).
// Columns whose waves, four sites long, are just more than the chip's 1024 SIMDs leave half of them idle in the second
// round: the site kernel then (us, site kernel against columns, 20 x 32 x 20 x 24, 1200 waves: FP64 one 84 / 91, full links
// 98 / 113, FP32 full links one 47 / 56, four 125 / 142; 28 x 24^3, 1512: FP64 one 116 / 103, FP32 full links 65 / 61).
// Thin lattices: columns and z-pairs only where the maps keep the lanes busy.  4096 x 4^3 has eight columns an XCD (FP64,
// us, one right-hand side: columns 349, site kernel in slabs 95); 512 x 8^3 has 64, one wave of a work-group whose LDS is
// for four, which pairs, one wave per SIMD, do not make up for (eight: pairs 967, one per lane 449); 64 x 4 x 16^2 has two
// z-pairs for eight XCDs (FP32 of eight: link-stationary 105, site kernel 52).
LaunchCfg untuned_cfg(const Geom &g, int prec, int n, int rows) {
    const int V = g.V;
    const long long w = (long long)V * n;
    if (w <= (prec == WDIRAC_F64 ? 1 << 14 : 1 << 15)) return {kOrderSplit, 256, 1, 1};
    // whether work-groups of `lanes` lanes keep three quarters of them busy
    const auto full = [&](const TileMap &m, int lanes) { return 4LL * V >= 3LL * m.ntiles * lanes; };
    const auto columns = [&] {
        const int waves = make_tilemap(g, kOrderColumn, 64, 4).ntiles;  // per right-hand side
        return full(make_tilemap(g, kOrderColumn, 64, 1), 64) && (waves <= 1024 || waves >= 1400);
    };
    if (prec == WDIRAC_F64 && V > 1 << 17 && columns())
        return {kOrderColumn, 256, 4,
                w >= (n == 3 ? 1 << 24 : 1 << 21) && full(make_tilemap(g, kOrderColumn, 256, 1), 256) ? 2 : 1};
    if (prec == WDIRAC_F32 && V >= 1 << 18 && columns())
        return {kOrderColumn, 256, w >= 1 << 21 && n < 3 ? 8 : 4, n > 1 ? 2 : 1};
    if (prec == WDIRAC_F32 && rows == 2 && n >= 6 && V >= 1 << 16 &&
        full(make_tilemap(g, kOrderZGroups, kStationaryBlock, 0), kStationaryBlock))
        return {kOrderStationary, kStationaryBlock, 1, 2};
    const bool single = prec == WDIRAC_F64 && (n < 4 || (n % 2 && rows == 3));
    return {kOrderTSweep, 256, 4, w > 1 << 17 && !single ? 2 : 1};
}

// The configuration of a launch: the autotuned one for this lattice,
// precision, right-hand-side count and link format if there is one, the
// process-wide values once one of them was set, else the rule above.
hipError_t dslash_launch_batches(const dirac_batch *batches, int nbatch, int prec, bool dagger, const OpData &d,
                                 const Geom &g, int apbc, bool persistent, hipStream_t st) {
    int total = 0;
    for (int b = 0; b < nbatch; b++) total += batches[b].nrhs;
    const Tuning tu = tuning_snapshot();
    LaunchCfg cfg{tu.order, tu.block, tu.tchunk, (prec >= 0 && prec < 3) ? tu.nr[prec] : 1};
    if (!tu.explicit_launch && !tuned_cfg(g, prec, total, d.rows, d.clover_compact, cfg))
        cfg = untuned_cfg(g, prec, total, d.rows);
    return dslash_launch_cfg(batches, nbatch, prec, dagger, d, g, apbc, persistent, cfg, st);
}

}  // namespace wd

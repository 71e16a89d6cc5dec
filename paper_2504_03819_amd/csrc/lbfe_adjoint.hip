// Discrete adjoint of the D3Q27 free-energy LB step: lambda(t) =
// (d f(t+1) / d f(t))^T lambda(t+1) for the forward map of lbfe_kernels.hip,
// plus the adjoint of the initialiser and the parameter gradients
// dL/dkappa, dL/d(wet_value), dL/dnu.  (The adjoint is not part of the
// paper; it differentiates the paper's discrete update exactly.)
//
// Per adjoint step, after the forward auxiliary fields of f(t) have been
// recomputed (launch_aux):
//   k_adj_collide   pull-gather lambda*(x) = lambda(t+1)(x + c_i) (or the
//                   bounce-back slot), local collision adjoint in central-
//                   moment space; writes the direct part of lambda(t) and
//                   the adjoints of u, F, Q, p_m (and rho, nu via omega_1)
//   k_adj_wall_move (moving walls) the wall-velocity term of the reflected
//                   populations transposed into rho_bar and p_m_bar
//   k_adj_phimu     transposed Q stencil -> adjoint of phi; back through
//                   phi = (p_m - rho/3) u, u = (j + F/2)/rho, F = (1/3-rho) G;
//                   then the transposed gradient stencil -> adjoint of mu
//                   (all nodes), in one z-march with G_bar kept in LDS
//   k_adj_wall_gather (walls) wall average of Eq. (36) transposed
//   k_adj_rho       mu0'(rho) and the (symmetric) Laplacian transposed;
//                   kappa and nu gradients
//   k_adj_tail      (walls) limiter/window of Eqs. (37)-(38) transposed, wet
//                   value gradient; (rho_bar_total, j_bar) per node, for the
//                   next step's gather
//   k_adj_final     lambda_i(t) += rho_bar + c_i . j_bar, applied when lambda
//                   is read out; between adjoint steps this term is added by
//                   the next step's gather instead
//   k_adj_reduce*   deterministic parameter-gradient accumulation
// With a solid voxel mask the collision adjoint takes its bounce-back links
// from the neighbour words, solid nodes hold no lambda and no source
// adjoints, and the wall averages and window of every solid node are
// transposed per node (k_adj_wall_gather_m, k_adj_wall_rho_solid_m).  With
// moving walls k_adj_wall_move transposes the wall-velocity term of the
// reflected populations.
#include <type_traits>

#include "lbfe_device.h"
#include "lbfe_dpp.h"
#include "lbfe_factored.h"

namespace lbfe {
namespace {

template <int P> using real_t = typename Pol<P>::real;

constexpr unsigned kSelfBit = 1u << kRest;  // neighbour word: the node itself is solid
// a fluid node: inside the fluid planes, and not solid in a voxel mask
__device__ inline bool fluid_node(const KP &kp, const Bufs &b, size_t n) {
    if (kp.masked) return !(b.nbr[n] & kSelfBit);
    const int z = (int)(n / kp.plane);
    return z >= kp.z0 && z < kp.z1;
}

// Adjoint auxiliary arrays inside Bufs::abuf, in slots of N doubles.  The
// slots marked (real) hold planes in the compute precision (three float
// planes use half of their three slots): those values are formed in that
// precision, so keeping them narrower loses nothing.
enum : int {
    A_UB = 0,    // 3 (real): u_bar
    A_FB = 3,    // 3 (real): F_bar
    A_QB = 6,    // 3 (real): Q_bar (after folding the fourth-order terms)
    A_PMB = 9,   // p_m bar
    A_RHOB = 10, // rho bar (local part)
    A_JB = 11,   // 3 (real): j bar, rounded to the compute precision
    A_MUB = 14,  // mu bar (all nodes; the wall and mask transposes)
    A_KAPC = 15, // dL/dkappa, a partial sum per workgroup of k_adj_rho
    A_NUC = 16,  // per-node dL/dnu contribution
    A_WETC = 17, // dL/d(wet): a partial sum per workgroup of k_adj_tail, or (mask) per node
    A_RAVEB = 18,// mask: rho_ave bar at solid nodes; else dL/dnu, a partial sum per workgroup of k_adj_rho
    A_RHOBT = 19,// rho bar total (all nodes)
    A_MUBT = 20, // mu bar total (all nodes)
    A_PACK = 21, // 4 planes: (rho_bar_total, j_bar) per node as 4 compute-precision values
    A_COUNT = 25
};

// Adjoint (lambda) storage: same row-blocked layout as the populations, in
// the compute precision.
template <class real> struct Lam {
    real *p;
    unsigned nx;
    __device__ Lam(void *q, const KP &kp) : p((real *)q), nx((unsigned)kp.nx) {}
    __device__ size_t off(int i, unsigned row, unsigned x) const { return ((size_t)row * 27 + i) * nx + x; }
    __device__ real ld(int i, unsigned row, unsigned x) const { return p[off(i, row, x)]; }
    __device__ real ld_nt(int i, unsigned row, unsigned x) const { return ldnt(p + off(i, row, x)); }
    __device__ void st(int i, unsigned row, unsigned x, real v) const { p[off(i, row, x)] = v; }
    __device__ void st_nt(int i, unsigned row, unsigned x, real v) const {
        __builtin_nontemporal_store(v, p + off(i, row, x));
    }
};

// Sum of v over the workgroup's NT threads, in a fixed order, on thread 0.
template <int NT> __device__ inline double block_sum(double v) {
    __shared__ double w[NT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63u) == 0) w[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int q = 0; q < NT / 64; ++q) t += w[q];
    __syncthreads();
    return t;
}

// Plane c of a (real) slot group.
template <class real> __device__ inline real *aplane(void *abuf, int slot, int c, size_t N) {
    return (real *)((double *)abuf + (size_t)slot * N) + (size_t)c * N;
}

// ---- transposed 1-D transforms -------------------------------------------
// Transpose of the inverse map (k0,k1,k2) -> (f-,f0,f+) (see inv3).
template <class real> __device__ inline void inv3_T(real &lm, real &l0, real &lp, real u) {
    const real s = lp + lm, d = lp - lm;
    const real k0 = l0 + u * u * ((real)0.5 * s - l0) + (real)0.5 * u * d;
    const real k1 = u * (s - (real)2 * l0) + (real)0.5 * d;
    const real k2 = (real)0.5 * s - l0;
    lm = k0;
    l0 = k1;
    lp = k2;
}
// Transpose of the forward map (f-,f0,f+) -> (k0,k1,k2): g_c = m0 + (c-u) m1 + (c-u)^2 m2.
template <class real> __device__ inline void fwd3_T(real &a, real &b, real &c, real u) {
    const real m0 = a, m1 = b, m2 = c;
    const real em = (real)-1 - u, e0 = -u, ep = (real)1 - u;
    a = m0 + em * m1 + em * em * m2;
    b = m0 + e0 * m1 + e0 * e0 * m2;
    c = m0 + ep * m1 + ep * ep * m2;
}
// lambda_hat = T(u)^{-T} lambda*  (slots: directions in, central moments out)
template <class real> __device__ inline void cm_inverse_T(real (&l)[27], real ux, real uy, real uz) {
#pragma unroll
    for (int p = 0; p < 9; ++p) inv3_T(l[3 * p], l[3 * p + 1], l[3 * p + 2], uz);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int g = 0; g < 3; ++g) inv3_T(l[9 * a + g], l[9 * a + 3 + g], l[9 * a + 6 + g], uy);
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int g = 0; g < 3; ++g) inv3_T(l[3 * b + g], l[9 + 3 * b + g], l[18 + 3 * b + g], ux);
}
// g = T(u)^T m  (slots: central moments in, directions out)
template <class real> __device__ inline void cm_forward_T(real (&m)[27], real ux, real uy, real uz) {
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int g = 0; g < 3; ++g) fwd3_T(m[3 * b + g], m[9 + 3 * b + g], m[18 + 3 * b + g], ux);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int g = 0; g < 3; ++g) fwd3_T(m[9 * a + g], m[9 * a + 3 + g], m[9 * a + 6 + g], uy);
#pragma unroll
    for (int p = 0; p < 9; ++p) fwd3_T(m[3 * p], m[3 * p + 1], m[3 * p + 2], uz);
}

// sum_{abg} lam_{abg} (S_x k)_{abg} with (S_x k)_{abg} = a k_{(a-1)bg}; S_y, S_z alike.
template <class real>
__device__ inline void shift_dot(const real (&lam)[27], const real (&k)[27], real &sx, real &sy, real &sz) {
    real ax = 0, ay = 0, az = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
            for (int g = 0; g < 3; ++g) {
                if (a > 0) ax += (real)a * lam[K(a, b, g)] * k[K(a - 1, b, g)];
                if (b > 0) ay += (real)b * lam[K(a, b, g)] * k[K(a, b - 1, g)];
                if (g > 0) az += (real)g * lam[K(a, b, g)] * k[K(a, b, g - 1)];
            }
    sx = ax;
    sy = ay;
    sz = az;
}

// Transpose of the collision's linear part D (Eqs. (21)-(26) at zero
// sources), in place on lambda_hat -> D^T lambda_hat, with the adjoints of
// the sources: F, the six Q terms, p_m and omega_1 (which also multiplies
// pre-collision moments k).
template <class real> struct SrcBar {
    real F[3], Q[6], pm, om1;
};

template <class real>
__device__ inline void collide_T(real (&l)[27], const real (&k)[27], const Rates<real> &R, real q200, real q020,
                                 real q002, SrcBar<real> &sb) {
    const real one = 1, half = 0.5, third = (real)(1.0 / 3.0), ninth = (real)(1.0 / 9.0);
    const real *w = R.w;
    for (int a = 0; a < 3; ++a) sb.F[a] = 0;
    for (int a = 0; a < 6; ++a) sb.Q[a] = 0;
    sb.pm = 0;
    sb.om1 = 0;
    // first order
    {
        const real r0 = one - w[0], c0 = one - half * w[0];
        sb.F[0] += c0 * l[K(1, 0, 0)];
        sb.F[1] += c0 * l[K(0, 1, 0)];
        sb.F[2] += c0 * l[K(0, 0, 1)];
        l[K(1, 0, 0)] *= r0;
        l[K(0, 1, 0)] *= r0;
        l[K(0, 0, 1)] *= r0;
    }
    // second order, off-diagonal
    sb.om1 -= l[K(1, 1, 0)] * k[K(1, 1, 0)] + l[K(0, 1, 1)] * k[K(0, 1, 1)] + l[K(1, 0, 1)] * k[K(1, 0, 1)];
    l[K(1, 1, 0)] *= (one - w[1]);
    l[K(0, 1, 1)] *= (one - w[1]);
    l[K(1, 0, 1)] *= (one - w[1]);
    // second order, diagonal: (A, B, S) combinations
    {
        const real l200 = l[K(2, 0, 0)], l020 = l[K(0, 2, 0)], l002 = l[K(0, 0, 2)];
        const real Ab = third * (l200 - (real)2 * l020 + l002);
        const real Bb = third * (l200 + l020 - (real)2 * l002);
        const real Sb = third * (l200 + l020 + l002);
        const real A = k[K(2, 0, 0)] - k[K(0, 2, 0)], B = k[K(2, 0, 0)] - k[K(0, 0, 2)];
        sb.om1 += Ab * (-A - half * (q200 - q020)) + Bb * (-B - half * (q200 - q002));
        const real c1 = one - half * w[1], c2 = one - half * w[2];
        sb.Q[0] += c1 * (Ab + Bb) + c2 * Sb;
        sb.Q[1] += -c1 * Ab + c2 * Sb;
        sb.Q[2] += -c1 * Bb + c2 * Sb;
        sb.pm += (real)3 * w[2] * Sb;
        const real Ap = (one - w[1]) * Ab, Bp = (one - w[1]) * Bb, Sp = (one - w[2]) * Sb;
        l[K(2, 0, 0)] = Ap + Bp + Sp;
        l[K(0, 2, 0)] = -Ap + Sp;
        l[K(0, 0, 2)] = -Bp + Sp;
    }
    // third order
    {
        const real r3 = one - w[3], r4 = one - w[4], c3 = (one - half * w[3]) * (real)(2.0 / 3.0);
        auto pair = [&](int ia, int ib, int comp) {
            const real Pb = half * (l[ia] + l[ib]), Mb = half * (l[ia] - l[ib]);
            sb.F[comp] += c3 * Pb;
            l[ia] = r3 * Pb + r4 * Mb;
            l[ib] = r3 * Pb - r4 * Mb;
        };
        pair(K(1, 2, 0), K(1, 0, 2), 0);
        pair(K(2, 1, 0), K(0, 1, 2), 1);
        pair(K(2, 0, 1), K(0, 2, 1), 2);
        l[K(1, 1, 1)] *= (one - w[5]);
    }
    // fourth order: (D1, D2, S4) combinations
    {
        const real l220 = l[K(2, 2, 0)], l202 = l[K(2, 0, 2)], l022 = l[K(0, 2, 2)];
        const real D1b = third * (l220 - l202), D2b = third * (l220 - l022), S4b = third * (l220 + l202 + l022);
        const real c6 = one - half * w[6], c7 = one - half * w[7];
        sb.Q[3] += c6 * (D1b + D2b) + c7 * S4b;
        sb.Q[4] += c6 * (-(real)2 * D1b + D2b) + c7 * S4b;
        sb.Q[5] += c6 * (D1b - (real)2 * D2b) + c7 * S4b;
        sb.pm += w[7] * S4b;
        const real D1p = (one - w[6]) * D1b, D2p = (one - w[6]) * D2b, S4p = (one - w[7]) * S4b;
        l[K(2, 2, 0)] = D1p + D2p + S4p;
        l[K(2, 0, 2)] = -(real)2 * D1p + D2p + S4p;
        l[K(0, 2, 2)] = D1p - (real)2 * D2p + S4p;
        l[K(2, 1, 1)] *= (one - w[8]);
        l[K(1, 2, 1)] *= (one - w[8]);
        l[K(1, 1, 2)] *= (one - w[8]);
    }
    // fifth order
    {
        const real c9 = (one - half * w[9]) * ninth, r9 = one - w[9];
        sb.F[0] += c9 * l[K(1, 2, 2)];
        sb.F[1] += c9 * l[K(2, 1, 2)];
        sb.F[2] += c9 * l[K(2, 2, 1)];
        l[K(1, 2, 2)] *= r9;
        l[K(2, 1, 2)] *= r9;
        l[K(2, 2, 1)] *= r9;
    }
    // sixth order
    sb.pm += w[10] * ninth * l[K(2, 2, 2)];
    l[K(2, 2, 2)] *= (one - w[10]);
}

// The last term of lambda(t): lambda_i(x) = direct part + rho_bar_total(x)
// + c_i . j_bar(x) at fluid nodes.  It is either applied in place
// (k_adj_final) or, while the next adjoint step follows, added to each value
// as that step gathers it (k_adj_collide with PEND): the same expression in
// the same order, so both give lambda bit for bit.
template <class real> __device__ inline real final_term(real rb, real jx, real jy, real jz, int i) {
    real add = rb;
    if (cxi(i)) add += (real)cxi(i) * jx;
    if (cyi(i)) add += (real)cyi(i) * jy;
    if (czi(i)) add += (real)czi(i) * jz;
    return add;
}
// the same four values packed per node (k_adj_tail), one vector load
template <class real> using Pack4 = std::conditional_t<std::is_same_v<real, double>, double4, float4>;
template <class real> __device__ inline real final_term(const Pack4<real> *pk, int i, size_t m) {
    const Pack4<real> t = pk[m];
    return final_term<real>(t.x, t.y, t.z, t.w, i);
}

// Adjoint sources that the stencils and sums read at solid nodes too: zero
// there, written by the seed (wall planes) or by k_adj_collide (masks), so that
// a sweep does not depend on what its workspace held.
template <class real> __device__ inline void zero_sources(void *abuf, size_t N, size_t n) {
#pragma unroll
    for (int c = 0; c < 3; ++c) aplane<real>(abuf, A_QB, c, N)[n] = (real)0;
    ((double *)abuf)[A_NUC * N + n] = 0.0;
}

template <class real> __device__ inline void store_pack(void *abuf, size_t N, size_t n, double rhobt) {
    Pack4<real> t;
    t.x = (real)rhobt;
    t.y = aplane<real>(abuf, A_JB, 0, N)[n];
    t.z = aplane<real>(abuf, A_JB, 1, N)[n];
    t.w = aplane<real>(abuf, A_JB, 2, N)[n];
    ((Pack4<real> *)((double *)abuf + A_PACK * N))[n] = t;
}

// ---------------------------------------------------------------------------
// PEND: lam_in holds only the direct part of lambda(t+1); its last term is
// added during the gather from the (rho_bar_total, j_bar) pack that the
// previous adjoint step left (this kernel does not write it).
// NT: f, lambda, F, Q and mu are read once and the node's own lambda row is
// written once, so from 2^20 nodes, where the lattices exceed the caches, they
// go non-temporal (192x192x96 in FP32: 342 -> 320 us); a small box keeps them
// in the caches (48x40x32 in FP64: 17.2 us, 19.2 non-temporal).
template <int P, bool PEND, bool MASK, bool NT>
__global__ __launch_bounds__(kBlock) void k_adj_collide(KP kp, Bufs b, const void *ft, const void *lam_in,
                                                        void *lam_out) {
    using real = real_t<P>;
    const unsigned idx = tile_id(kp) * kBlock + threadIdx.x;
    if (idx >= kp.nfluid) return;
    const unsigned n = (unsigned)kp.z0 * kp.plane + idx;
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    const unsigned row = nb.row(0, 0);
    const Pops<P, NT> fin(ft, kp);
    const Lam<real> lin(const_cast<void *>(lam_in), kp), lout(lam_out, kp);
    // solid mask: bit i of the neighbour word marks a link that ends on a
    // solid node (bounce-back); a solid node holds no lambda
    auto ld = [&](const auto *p) { return NT ? ldnt(p) : *p; };
    auto ldl = [&](int i, unsigned r, unsigned xx) { return NT ? lin.ld_nt(i, r, xx) : lin.ld(i, r, xx); };
    auto stl = [&](int i, real v) { NT ? lout.st_nt(i, row, (unsigned)x, v) : lout.st(i, row, (unsigned)x, v); };
    const unsigned wm = MASK ? b.nbr[n] : 0u;
    if (MASK && (wm & kSelfBit)) {
#pragma unroll
        for (int i = 0; i < 27; ++i) stl(i, (real)0);
        zero_sources<real>(b.abuf, kp.N, n);
        return;
    }

    // forward recomputation at x: the moments, kinematics and collision of
    // k_collide (the same device functions, so the same roundings)
    real k[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) k[i] = fin.ld(i, row, (unsigned)x);
    double rd;
    real jx, jy, jz;
    moments(k, rd, jx, jy, jz);
    const real *F = (const real *)b.F;
    const real Fx = ld(F + n), Fy = ld(F + kp.N + n), Fz = ld(F + 2 * (size_t)kp.N + n);
    const Kin<real> kin = kinematics(kp, rd, jx, jy, jz, Fx, Fy, Fz, ld(b.mu + n));
    const real ux = kin.ux, uy = kin.uy, uz = kin.uz, pm = kin.pm;
    const real *Qa = (const real *)b.Q;
    const real q200 = ld(Qa + n), q020 = ld(Qa + kp.N + n), q002 = ld(Qa + 2 * (size_t)kp.N + n);
    real q220 = 0, q202 = 0, q022 = 0;
    const real third = (real)(1.0 / 3.0);
    if (kp.corr4) {
        q220 = (q200 + q020) * third;
        q202 = (q200 + q002) * third;
        q022 = (q020 + q002) * third;
    }
    Rates<real> R;
#pragma unroll
    for (int q = 0; q < 11; ++q) R.w[q] = (real)kp.om[q];
    const real om1 = kin.om1;
    R.w[1] = om1;
    cm_forward(k, ux, uy, uz);  // k: pre-collision central moments
    real ks[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) ks[i] = k[i];
    collide(ks, R, Fx, Fy, Fz, pm, q200, q020, q002, q220, q202, q022);

    // reverse streaming: lambda*_i(x) = lambda_i(t+1)(x + c_i), or the
    // bounce-back partner at x when x + c_i is solid
    const bool wall_lo = kp.walls && z == 1;
    const bool wall_hi = kp.walls && z == kp.nz - 2;
    real l[27];
    const Pack4<real> *pk = (const Pack4<real> *)((const double *)b.abuf + A_PACK * (size_t)kp.N);
    auto bounce = [&](int i) {
        const int cz = czi(i);
        if constexpr (MASK) return ((wm >> i) & 1u) != 0;
        return (cz < 0 && wall_lo) || (cz > 0 && wall_hi);
    };
    if constexpr (PEND && (sizeof(real) == 8 || MASK)) {
        // FP64: the pending (rho_bar_total, j_bar) of each link's neighbour
        // with one vector load per link, beside the link's lambda (the
        // lane-shift form below needs more registers than an FP64 wave has
        // at two waves per SIMD)
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int cz = czi(i);
            if (bounce(i))
                l[i] = ldl(26 - i, row, (unsigned)x) + final_term<real>(pk, 26 - i, n);
            else
                l[i] = ldl(i, nb.row(cyi(i), cz), nb.xo(cxi(i))) +
                       final_term<real>(pk, i, nb.at(cxi(i), cyi(i), cz));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int cz = czi(i);
            if (bounce(i))
                l[i] = ldl(26 - i, row, (unsigned)x);
            else
                l[i] = ldl(i, nb.row(cyi(i), cz), nb.xo(cxi(i)));
        }
    }
    if constexpr (PEND && sizeof(real) == 4 && !MASK) {
        // The pending (rho_bar_total, j_bar) of the 27 neighbours, one row
        // (cy, cz) at a time: the x - 1 and x + 1 values are those of the
        // adjacent lanes (a wave holds consecutive nodes), loaded only by
        // the lanes at a wave's or a row's ends.  The last active lane of
        // a partial wave has x = nx - 1 (fluid rows are whole).
        const unsigned lane = threadIdx.x & 63u;
        const bool own_m = lane == 0u || x == 0, own_p = lane == 63u || x == kp.nx - 1;
        const Pack4<real> c0 = pk[n];
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const int cy = r / 3 - 1, cz = r % 3 - 1;
            const Pack4<real> c = pk[nb.at(0, cy, cz)];
            Pack4<real> m, p;
            m.x = shr1(c.x), m.y = shr1(c.y), m.z = shr1(c.z), m.w = shr1(c.w);
            p.x = shl1(c.x), p.y = shl1(c.y), p.z = shl1(c.z), p.w = shl1(c.w);
            if (own_m) m = pk[nb.at(-1, cy, cz)];
            if (own_p) p = pk[nb.at(1, cy, cz)];
            const bool bb = (cz < 0 && wall_lo) || (cz > 0 && wall_hi);
#pragma unroll
            for (int cx = -1; cx <= 1; ++cx) {
                const int i = 9 * (cx + 1) + 3 * (cy + 1) + (cz + 1);
                const Pack4<real> t = cx < 0 ? m : (cx > 0 ? p : c);
                l[i] += bb ? final_term<real>(c0.x, c0.y, c0.z, c0.w, 26 - i)
                           : final_term<real>(t.x, t.y, t.z, t.w, i);
            }
        }
    }
    // (moving walls: the wall term's adjoint is added by k_adj_wall_move)
    cm_inverse_T(l, ux, uy, uz);  // l = lambda_hat (adjoint of k*)
    real ubx, uby, ubz;
    shift_dot(l, ks, ubx, uby, ubz);  // lambda_hat . S k*
    SrcBar<real> sb;
    collide_T(l, k, R, q200, q020, q002, sb);  // l = D^T lambda_hat
    real tx, ty, tz;
    shift_dot(l, k, tx, ty, tz);  // (D^T lambda_hat) . S k
    ubx -= tx;
    uby -= ty;
    ubz -= tz;
    cm_forward_T(l, ux, uy, uz);  // direct part of lambda(t)
#pragma unroll
    for (int i = 0; i < 27; ++i) stl(i, l[i]);

    // fold the fourth-order correction (Eq. (28)) into Q_bar
    real qb0 = sb.Q[0], qb1 = sb.Q[1], qb2 = sb.Q[2];
    if (kp.corr4) {
        qb0 += third * (sb.Q[3] + sb.Q[4]);
        qb1 += third * (sb.Q[3] + sb.Q[5]);
        qb2 += third * (sb.Q[4] + sb.Q[5]);
    }
    // omega_1 = 1 / (rho nu / p_m + 1/2)
    const double o = (double)om1, dpm = (double)pm, rr = rd;
    const double om1b = (double)sb.om1;
    const double rhob = -om1b * o * o * kp.nu / dpm;
    const double pmb = (double)sb.pm + om1b * o * o * rr * kp.nu / (dpm * dpm);
    const double nub = -om1b * o * o * rr / dpm;
    const size_t N = kp.N;
    double *A = (double *)b.abuf;
    aplane<real>(A, A_UB, 0, N)[n] = ubx;
    aplane<real>(A, A_UB, 1, N)[n] = uby;
    aplane<real>(A, A_UB, 2, N)[n] = ubz;
    aplane<real>(A, A_FB, 0, N)[n] = sb.F[0];
    aplane<real>(A, A_FB, 1, N)[n] = sb.F[1];
    aplane<real>(A, A_FB, 2, N)[n] = sb.F[2];
    aplane<real>(A, A_QB, 0, N)[n] = qb0;
    aplane<real>(A, A_QB, 1, N)[n] = qb1;
    aplane<real>(A, A_QB, 2, N)[n] = qb2;
    A[A_PMB * N + n] = pmb;
    A[A_RHOB * N + n] = rhob;
    A[A_NUC * N + n] = nub;
}

// Moving walls: a reflected population carries -[f^eq_i - f^eq_opp(i)](rho,
// p_m, u_w) (k_wall_move), which is linear in (rho, p_m) at a given u_w; its
// adjoint adds to rho_bar and p_m_bar of the wall-adjacent nodes, from the
// lambda* that k_adj_collide gathered on the reflected links (a kernel of its
// own, after k_adj_collide: the wall equilibria would raise the collision
// adjoint's register count past two waves per SIMD in FP64).
template <int P, bool PEND>
__global__ __launch_bounds__(kBlock) void k_adj_wall_move(KP kp, Bufs b, const void *lam_in) {
    using real = real_t<P>;
    const unsigned idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= 2 * kp.plane) return;
    const int side = idx >= kp.plane;
    if (side && kp.nz - 2 == 1) return;  // one fluid plane: both walls by side 0
    const unsigned p = idx - (side ? kp.plane : 0u);
    const int y = (int)(p / (unsigned)kp.nx), x = (int)(p - (unsigned)y * kp.nx);
    const int z = side ? kp.nz - 2 : 1;
    const size_t n = (size_t)z * kp.plane + p;
    const Nb nb(kp, x, y, z);
    const unsigned row = nb.row(0, 0);
    const Lam<real> lin(const_cast<void *>(lam_in), kp);
    const Pack4<real> *pk = (const Pack4<real> *)((const double *)b.abuf + A_PACK * (size_t)kp.N);
    const bool wall_lo = z == 1, wall_hi = z == kp.nz - 2;
    double wrb = 0.0, wpb = 0.0;
    for (int w = 0; w < 2; ++w) {
        if (!(w == 0 ? wall_lo : wall_hi)) continue;
        real ea[27], eb[27];
        const real uwx = (real)kp.wall_u[2 * w], uwy = (real)kp.wall_u[2 * w + 1];
        wall_equilibrium((real)1, (real)0, uwx, uwy, ea);
        wall_equilibrium((real)0, (real)1, uwx, uwy, eb);
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const int cz = czi(i);
            if ((w == 0 && cz < 0) || (w == 1 && cz > 0)) {
                // lambda*_i at a reflected link: the node's own value of the
                // opposite direction, plus its pending last term
                real li = lin.ld(26 - i, row, (unsigned)x);
                if constexpr (PEND) li = li + final_term<real>(pk, 26 - i, n);
                wrb -= (double)li * (double)(ea[i] - ea[26 - i]);
                wpb -= (double)li * (double)(eb[i] - eb[26 - i]);
            }
        }
    }
    double *A = (double *)b.abuf;
    A[A_RHOB * kp.N + n] += wrb;
    A[A_PMB * kp.N + n] += wpb;
}

// The transposed Q and gradient stencils, factored (lbfe_factored.h), in one
// z-march:
//   phi part, at fluid nodes: phi_bar_a = transpose of Q_a = -9 sum_i w_i
//     c_ia phi_a(x + c_i) = 9 sum_i w_i c_ia Q_bar_a(x + c_i), then back
//     through phi = (p_m - rho/3) u, u = (j + F/2)/rho, F = (1/3 - rho) G:
//     j_bar, rho_bar (local part), G_bar and the local part of mu_bar;
//   mu part, at every node: mu_bar(y) = local part (fluid) - 3 sum_i w_i
//     c_i . G_bar(y + c_i) (G_bar is zero at solid nodes), into A_MUBT.
// A workgroup owns a PTX x PTY tile of mu_bar planes [zs, ze); the phi part
// runs on the tile and its one-node ring, one node per thread.  Iteration t
// stages Q_bar and mu of plane t (two-node halo), takes the in-plane parts of
// plane t-1 and the phi part of plane t-2, whose G_bar goes to LDS, then the
// in-plane parts of G_bar(t-3) and mu_bar(t-4).  Each stage reads what the
// iteration before wrote (two slots per LDS plane), so one barrier per plane
// suffices.  G_bar never goes to HBM; the owned node's j_bar and rho_bar do,
// the ring nodes only give G_bar.  Bound by its loads (128 B per node without
// the halos) and their latency: at 192x192x96 in FP32 133 us, 3.4 TB/s on
// those bytes, where reading every 27-point sum from LDS took 192 us; at
// 48x40x32 in FP64 18 against 62 us.
template <int P, bool MASK, int PTX, int PTY, int PNT>
__global__ __launch_bounds__(PNT, 4) void k_adj_phimu(KP kp, Bufs b, int cz) {
    using real = real_t<P>;
    constexpr int PWX = PTX + 4, PNR = PWX * (PTY + 4);  // Q_bar and mu region: tile + 2-node halo
    constexpr int GWX = PTX + 2, GNR = GWX * (PTY + 2);  // G_bar region: tile + 1-node ring
    constexpr int PPT = (PNR + PNT - 1) / PNT;           // Q_bar / mu region points per thread
    static_assert(GNR <= PNT && PTX * PTY <= PNT, "one G_bar node, one owned column per thread");
    __shared__ double sq[2][4][PNR];  // Q_bar x, y, z and mu of plane p (slot p & 1)
    __shared__ double sg[2][3][GNR];  // G_bar of plane p (slot p & 1)
    __shared__ double sl[3][GNR];     // local part of mu_bar of plane p (slot p mod 3)
    const int ntx = (kp.nx + PTX - 1) / PTX;
    int tile, chunk;
    xcd_tile(tile, chunk);
    const int x0 = tile % ntx * PTX, y0 = tile / ntx * PTY;
    const int zs = chunk * cz, ze = min(zs + cz, kp.nz);
    const size_t N = kp.N;
    const unsigned plane = kp.plane;
    double *A = (double *)b.abuf;
    const real *j = (const real *)b.j, *F = (const real *)b.F;
    const int tid = threadIdx.x;
    constexpr unsigned S = sizeof(real);

    // Q_bar / mu region points of this thread, in-plane node index
    unsigned qoff[PPT];
#pragma unroll
    for (int m = 0; m < PPT; ++m) {
        const int r = tid + m * PNT;
        qoff[m] = r < PNR ? (unsigned)zwrap(y0 + r / PWX - 2, kp.ny) * kp.nx + zwrap(x0 + r % PWX - 2, kp.nx) : kNone;
    }
    // phi node (ga, gb) of the G_bar region, owned when inside the tile and grid
    const int ga = tid % GWX, gb = tid / GWX;
    const bool hasg = tid < GNR;
    const unsigned noff =
        hasg ? (unsigned)zwrap(y0 + gb - 1, kp.ny) * kp.nx + zwrap(x0 + ga - 1, kp.nx) : kNone;
    const bool owng = hasg && ga >= 1 && ga <= PTX && gb >= 1 && gb <= PTY && x0 + ga - 1 < kp.nx && y0 + gb - 1 < kp.ny;
    const int cq = hasg ? (gb + 1) * PWX + ga + 1 : PWX + 1;  // the node in the Q_bar / mu region
    // owned column (ta, tb) of the mu part
    const int ta = tid % PTX, tb = tid / PTX;
    const bool own = tid < PTX * PTY && x0 + ta < kp.nx && y0 + tb < kp.ny;
    const unsigned ooff = own ? (unsigned)(y0 + tb) * kp.nx + (x0 + ta) : kNone;
    const int cg = tid < PTX * PTY ? (tb + 1) * GWX + ta + 1 : GWX + 1;

    auto next = [&](int g) { return g + 1 == kp.nz ? 0 : g + 1; };
    // loads run one iteration ahead of their use
    real qpre[3][PPT];
    double mpre[PPT];
    auto load_q = [&](int g, bool ok) {  // ok false: a plane the chunk does not need
        const size_t f = (size_t)g * plane;
#pragma unroll
        for (int m = 0; m < PPT; ++m) {
            const unsigned o = ok ? qoff[m] : kNone;
#pragma unroll
            for (int c = 0; c < 3; ++c) pld(qpre[c][m], plane_of(aplane<real>(A, A_QB, c, N), f, plane, S), o);
            pld(mpre[m], plane_of(b.mu, f, plane, 8), o);
        }
    };
    double rpre, ppre, bpre;
    real jpre[3], fpre[3], upre[3], gpre[3];
    unsigned wpre = 0;
    auto load_node = [&](int g, bool ok) {
        const size_t f = (size_t)g * plane;
        const unsigned o = ok ? noff : kNone, oo = ok && owng ? noff : kNone;
        pld(rpre, plane_of(b.rho, f, plane, 8), o);
        pld(ppre, plane_of(A + A_PMB * N, f, plane, 8), oo);
        pld(bpre, plane_of(A + A_RHOB * N, f, plane, 8), oo);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            pld(jpre[c], plane_of(j + c * N, f, plane, S), o);
            pld(fpre[c], plane_of(F + c * N, f, plane, S), o);
            pld(upre[c], plane_of(aplane<real>(A, A_UB, c, N), f, plane, S), o);
            pld(gpre[c], plane_of(aplane<real>(A, A_FB, c, N), f, plane, S), o);
        }
        if constexpr (MASK) wpre = hasg ? b.nbr[f + noff] : kSelfBit;
    };

    Ring3 rq, rm, rg;  // in-plane parts of Q_bar, grad mu, G_bar
    double mc = 0.0;   // mu of the phi node's newest plane
    int t = zs - 2;
    int g4 = zwrap(t - 4, kp.nz), g3 = zwrap(t - 3, kp.nz), g2 = zwrap(t - 2, kp.nz), g1 = zwrap(t - 1, kp.nz),
        gn = zwrap(t, kp.nz);
    int s2 = (t - 2 + 6) % 3;  // (t - 2) mod 3; t >= -2
    load_q(gn, true);
    load_node(g2, false);
    for (; t <= ze + 3; ++t) {
#pragma unroll
        for (int m = 0; m < PPT; ++m)
            if (tid + m * PNT < PNR) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sq[t & 1][c][tid + m * PNT] = (double)qpre[c][m];
                sq[t & 1][3][tid + m * PNT] = mpre[m];
            }
        gn = next(gn);
        load_q(gn, t + 1 <= ze + 1);

        if (t - 1 >= zs - 2 && t - 2 <= ze) {
            const int p = t - 2;
            const double(*q)[PNR] = sq[(t - 1) & 1];
            const Part3 qn{dx_wy<PWX>(q[0], cq), wx_dy<PWX>(q[1], cq), smooth2<PWX>(q[2], cq)};
            const Part3 mn{dx_wy<PWX>(q[3], cq), wx_dy<PWX>(q[3], cq), smooth2<PWX>(q[3], cq)};
            double jb[3] = {0, 0, 0}, Gb[3] = {0, 0, 0}, rhob = 0.0, mloc = 0.0;
            const bool fplane = p >= zs - 1 && g2 >= kp.z0 && g2 < kp.z1;
            const bool fl = fplane && !(MASK && (wpre & kSelfBit));
            if (fl) {
                const double pb[3] = {1.5 * wz(rq.a.x, rq.b.x, qn.x), 1.5 * wz(rq.a.y, rq.b.y, qn.y), 1.5 * (qn.z - rq.a.z)};
                const double g[3] = {0.5 * wz(rm.a.x, rm.b.x, mn.x), 0.5 * wz(rm.a.y, rm.b.y, mn.y), 0.5 * (mn.z - rm.a.z)};
                const double r = rpre, rinv = 1.0 / r;
                const real ir = (real)1 / (real)r;
                const double c1 = 1.0 / 3.0 - r, c2 = (double)(real)((1.0 + mc - r) * (1.0 / 3.0));
                double pu = 0.0, uu = 0.0, fg = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double u = (double)((jpre[c] + (real)0.5 * fpre[c]) * ir);
                    const double ut = (double)upre[c] + c2 * pb[c];
                    // u = (j + F/2)/rho: j_bar = u_tilde/rho, F_bar += j_bar/2
                    jb[c] = ut * rinv;
                    const double Fb = (double)gpre[c] + 0.5 * jb[c];
                    Gb[c] = c1 * Fb;
                    pu += pb[c] * u;
                    uu += ut * u;
                    fg += Fb * g[c];
                }
                rhob = bpre - pu * (1.0 / 3.0) - uu * rinv - fg;
                mloc = (ppre + pu) * (1.0 / 3.0);  // p_m = (1 + mu)/3
            }
            if (hasg && p >= zs - 1) {  // (solid: no G_bar, no local mu_bar)
#pragma unroll
                for (int c = 0; c < 3; ++c) sg[p & 1][c][tid] = Gb[c];
                sl[s2][tid] = mloc;
            }
            // the fill planes at both ends belong to the neighbouring chunks
            const unsigned o = fl && owng && p >= zs && p < ze ? noff : kNone;
            const size_t f = (size_t)g2 * plane;
#pragma unroll
            for (int c = 0; c < 3; ++c) pst((real)jb[c], plane_of(aplane<real>(A, A_JB, c, N), f, plane, S), o);
            pst(rhob, plane_of(A + A_RHOB * N, f, plane, 8), o);
            rq.push(qn);
            rm.push(mn);
            mc = q[3][cq];
        }
        load_node(g1, t - 1 >= zs - 1 && t - 1 <= ze);

        if (t - 3 >= zs - 1) {
            const int p3 = t - 3, p = t - 4;
            const double(*g)[GNR] = sg[p3 & 1];
            const Part3 n{dx_wy<GWX>(g[0], cg), wx_dy<GWX>(g[1], cg), smooth2<GWX>(g[2], cg)};
            const double d = 0.5 * wz(rg.a.x, rg.b.x, n.x) + 0.5 * wz(rg.a.y, rg.b.y, n.y) + 0.5 * (n.z - rg.a.z);
            const double v = sl[s2 == 2 ? 0 : s2 + 1][cg] - d;  // slot (t - 4) mod 3
            pst(v, plane_of(A + A_MUBT * N, (size_t)g4 * plane, plane, 8), p >= zs ? ooff : kNone);
            rg.push(n);
        }
        __syncthreads();
        g4 = g3;
        g3 = g2;
        g2 = g1;
        g1 = next(g1);
        s2 = s2 == 2 ? 0 : s2 + 1;
    }
}

// Normalising weight sum of the wall average at solid node (x, y, zs).
__device__ inline double wall_den(const KP &kp, int zs) {
    double den = 0.0;
    for (int cz = -1; cz <= 1; ++cz) {
        const int zz = zs + cz;
        if (zz < 1 || zz > kp.nz - 2) continue;
        for (int cy = -1; cy <= 1; ++cy)
            for (int cx = -1; cx <= 1; ++cx) den += wq(cx, cy, cz);
    }
    return den;
}

// Transpose of a wall average (Eqs. (36)/(37)) for the fluid first layers:
// dst(y) += sum over solid neighbours s of w(y - s) / den(s) * src(s).
__global__ __launch_bounds__(kBlock) void k_adj_wall_gather(KP kp, const double *src, double *dst) {
    const unsigned idx = blockIdx.x * kBlock + threadIdx.x;
    if (idx >= 2 * kp.plane) return;
    const int side = idx >= kp.plane;
    if (side && kp.nz - 2 == 1) return;  // one fluid layer: both walls handled by side 0
    const unsigned p = idx - (side ? kp.plane : 0u);
    const int y = (int)(p / (unsigned)kp.nx), x = (int)(p - (unsigned)y * kp.nx);
    const int zf = side ? kp.nz - 2 : 1;  // fluid layer next to a wall
    const Nb nb(kp, x, y, zf);
    double acc = 0.0;
    for (int cz = -1; cz <= 1; ++cz) {
        const int zs = zf + cz;
        if (zs != 0 && zs != kp.nz - 1) continue;  // only solid neighbours
        const double inv = 1.0 / wall_den(kp, zs);
        for (int cy = -1; cy <= 1; ++cy)
            for (int cx = -1; cx <= 1; ++cx) acc += wq(cx, cy, cz) * inv * src[nb.at(cx, cy, cz)];
    }
    dst[(size_t)zf * kp.plane + p] += acc;
}

// rho_bar_total(y) = [fluid: rho_bar + mu_bar mu0'(rho)] - kappa L[mu_bar_fluid](y), in a
// z-march like k_adj_phimu's (plane t staged, in-plane parts of t-1, node t-2);
// dL/dkappa = -mu_bar L[rho] and, with nuc, the nodes' dL/dnu are summed per
// workgroup here (the separate pass that read both from memory took 3.7 us of a
// 48x40x32 step, 16 of a 192x192x96 one).  `mub` is the total mu_bar (solid
// entries are ignored: the Laplacian's adjoint sees fluid mu_bar only).
constexpr int RTX = 32, RTY = 16, RNT = RTX * RTY;
constexpr int RWX = RTX + 2, RNR = RWX * (RTY + 2), RPT = (RNR + RNT - 1) / RNT;
template <bool MASK>
__global__ __launch_bounds__(RNT) void k_adj_rho(KP kp, const double *mub, const double *rhob_local,
                                                 const double *rho, const double *nuc, double *rhobt, double *kap,
                                                 double *nu, int cz, const unsigned *nbr) {
    __shared__ double sd[2][2][RNR];  // mu_bar (0 on solid planes) and rho of plane p (slot p & 1)
    const int ntx = (kp.nx + RTX - 1) / RTX;
    int tile, chunk;
    xcd_tile(tile, chunk);
    const int x0 = tile % ntx * RTX, y0 = tile / ntx * RTY;
    const int zs = chunk * cz, ze = min(zs + cz, kp.nz);
    const unsigned plane = kp.plane;
    const int tid = threadIdx.x, ta = tid % RTX, tb = tid / RTX;
    const bool own = x0 + ta < kp.nx && y0 + tb < kp.ny;
    const unsigned ooff = own ? (unsigned)(y0 + tb) * kp.nx + (x0 + ta) : kNone;
    const int c = (tb + 1) * RWX + ta + 1;
    unsigned off[RPT];
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
        const int r = tid + m * RNT;
        off[m] = r < RNR ? (unsigned)zwrap(y0 + r / RWX - 1, kp.ny) * kp.nx + zwrap(x0 + r % RWX - 1, kp.nx) : kNone;
    }
    auto next = [&](int g) { return g + 1 == kp.nz ? 0 : g + 1; };
    auto fluid_plane = [&](int g) { return g >= kp.z0 && g < kp.z1; };
    // loads run one iteration ahead of their use
    double pre[2][RPT], lpre, npre = 0.0;
    unsigned wpre = 0;
    auto load = [&](int g, bool ok) {  // ok false: a plane the chunk does not need
        const size_t f = (size_t)g * plane;
        const bool fl = ok && fluid_plane(g);
#pragma unroll
        for (int m = 0; m < RPT; ++m) {
            pld(pre[0][m], plane_of(mub, f, plane, 8), fl ? off[m] : kNone);
            pld(pre[1][m], plane_of(rho, f, plane, 8), ok ? off[m] : kNone);
        }
    };
    auto load_node = [&](int g, bool ok) {
        const size_t f = (size_t)g * plane;
        pld(lpre, plane_of(rhob_local, f, plane, 8), ok ? ooff : kNone);
        if (nuc) pld(npre, plane_of(nuc, f, plane, 8), ok ? ooff : kNone);
        if constexpr (MASK) wpre = own ? nbr[f + ooff] : kSelfBit;
    };
    double ksum = 0, nsum = 0;
    double ma = 0, mb = 0, ra = 0, rb = 0, m0 = 0, r0 = 0;  // Wx Wy of two planes back, one back; values one back
    int t = zs - 1;
    int g2 = zwrap(t - 2, kp.nz), g1 = zwrap(t - 1, kp.nz), gn = zwrap(t, kp.nz);
    load(gn, true);
    load_node(g2, false);
    for (; t <= ze + 1; ++t) {
#pragma unroll
        for (int m = 0; m < RPT; ++m)
            if (tid + m * RNT < RNR) {
                sd[t & 1][0][tid + m * RNT] = pre[0][m];
                sd[t & 1][1][tid + m * RNT] = pre[1][m];
            }
        gn = next(gn);
        load(gn, t + 1 <= ze);
        if (t - 1 >= zs - 1) {
            const double(*d)[RNR] = sd[(t - 1) & 1];
            const double mn = smooth2<RWX>(d[0], c), rn = smooth2<RWX>(d[1], c);
            const double lm = 6.0 * (wz(ma, mb, mn) - m0), lr = 6.0 * (wz(ra, rb, rn) - r0);
            const bool fluid = fluid_plane(g2) && !(MASK && (wpre & kSelfBit));
            double out = -kp.kappa * lm;
            if (fluid) {
                const double q = 1.0 - kp.b * r0;
                const double dmu0 = kp.RT / (r0 * q * q) - 2.0 * kp.a;
                out += lpre + m0 * dmu0;
                if (own && t - 2 >= zs) ksum -= m0 * lr;
            }
            nsum += npre;  // 0 outside the chunk and the box
            load_node(g1, t - 1 >= zs && t - 1 < ze);
            const unsigned o = t - 2 >= zs ? ooff : kNone;
            const size_t f = (size_t)g2 * plane;
            pst(out, plane_of(rhobt, f, plane, 8), o);
            ma = mb, mb = mn, ra = rb, rb = rn;
            m0 = d[0][c];
            r0 = d[1][c];
        } else {
            load_node(g1, t - 1 >= zs && t - 1 < ze);
        }
        __syncthreads();
        g2 = g1;
        g1 = next(g1);
    }
    ksum = block_sum<RNT>(ksum);
    nsum = block_sum<RNT>(nsum);
    if (tid == 0) {
        const size_t i = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
        kap[i] = ksum;
        nu[i] = nsum;
    }
}

// rho_ave_bar = W'(rho_ave) rho_bar(x_s) of a solid node with wall average rave
// and rho_bar g; wet receives dL/d(wet_value) = dW/d(wet)
// rho_bar(x_s) (active branch of Eq. (38)).
__device__ inline double wall_rho_bar(const KP &kp, double rave, double g, double &wet) {
    double dW = 1.0, dwet = 0.0;
    if (rave >= kp.lo && rave <= kp.hi) {
        if (kp.wet_mode == LBFE_WET_PHI) {
            const double v = kp.wet_value * rave;
            const bool inside = v >= kp.lo && v <= kp.hi;
            dW = inside ? kp.wet_value : 0.0;
            dwet = inside ? rave : 0.0;
        } else if (kp.wet_mode == LBFE_WET_DELTA) {
            const double v = rave - kp.wet_value;
            const bool inside = v >= kp.lo && v <= kp.hi;
            dW = inside ? 1.0 : 0.0;
            dwet = inside ? -1.0 : 0.0;
        }
    }
    wet = dwet * g;
    return dW * g;
}

// The end of an adjoint step at a fluid node.  WALLS: beside a wall,
// rho_bar_total takes the transposed wall average of rho_ave_bar over the
// node's nine solid neighbours, whose rho_bar k_adj_rho left in the solid
// planes; each is formed again for every neighbour, from the 5 x 5 densities
// around the node, loaded together: no launches of their own (two of 4 us).
// PACK: the (rho_bar_total, j_bar) pack of the next step.
template <int P, bool PACK, bool WALLS>
__global__ __launch_bounds__(kBlock) void k_adj_tail(KP kp, Bufs b) {
    using real = real_t<P>;
    const unsigned idx = tile_id(kp) * kBlock + threadIdx.x;
    const size_t N = kp.N;
    double *A = (double *)b.abuf, *rhobt = A + A_RHOBT * N;
    double wet = 0.0;
    if (idx < kp.nfluid) {
        const unsigned n = (unsigned)kp.z0 * kp.plane + idx;
        double rb = rhobt[n];
        if constexpr (WALLS) {
            int x, y, z;
            decompose(kp, n, x, y, z);
            if (z == 1 || z == kp.nz - 2) {
                unsigned X[5], Y[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    X[k] = (unsigned)zwrap(x + k - 2, kp.nx);
                    Y[k] = (unsigned)zwrap(y + k - 2, kp.ny) * (unsigned)kp.nx;
                }
                // densities of the plane beside the wall and their wall averages
                double r[5][5], acc = 0.0;
#pragma unroll
                for (int v = 0; v < 5; ++v)
#pragma unroll
                    for (int u = 0; u < 5; ++u) r[v][u] = b.rho[(size_t)z * kp.plane + Y[v] + X[u]];
                for (int side = 0; side < 2; ++side) {
                    if (side ? z != kp.nz - 2 : z != 1) continue;
                    const int zs = side ? kp.nz - 1 : 0;
                    double g[3][3];
#pragma unroll
                    for (int v = 0; v < 3; ++v)
#pragma unroll
                        for (int u = 0; u < 3; ++u) g[v][u] = rhobt[(size_t)zs * kp.plane + Y[v + 1] + X[u + 1]];
                    const double inv = 1.0 / wall_den(kp, zs);
#pragma unroll
                    for (int cy = -1; cy <= 1; ++cy)
#pragma unroll
                        for (int cx = -1; cx <= 1; ++cx) {
                            double num = 0.0, den = 0.0, w;
#pragma unroll
                            for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
                                for (int dx = -1; dx <= 1; ++dx) {
                                    num += wq(dx, dy, 1) * r[cy + dy + 2][cx + dx + 2];
                                    den += wq(dx, dy, 1);
                                }
                            acc += wq(cx, cy, 1) * inv * wall_rho_bar(kp, num / den, g[cy + 1][cx + 1], w);
                            if (cx == 0 && cy == 0) wet += w;
                        }
                }
                rb += acc;
                rhobt[n] = rb;
            }
        }
        if constexpr (PACK) store_pack<real>(b.abuf, N, n, rb);
    }
    if constexpr (WALLS) {
        wet = block_sum<kBlock>(wet);
        if (threadIdx.x == 0) A[A_WETC * N + blockIdx.x] = wet;
    }
}

// ---- solid voxel masks ------------------------------------------------------
// The transposes of the mask path's wall averages (Eqs. (36)-(37) at every
// solid node with a fluid neighbour, weights w_i of its fluid neighbours in
// direction order) and of the window of Eq. (38), per node.

// dst = src at fluid nodes, 0 at solid nodes (mu_bar as the Laplacian's
// adjoint sees it)
__global__ __launch_bounds__(kBlock) void k_adj_fluid_copy_m(KP kp, const unsigned *nbr, const double *src,
                                                           double *dst) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    dst[n] = (nbr[n] & kSelfBit) ? 0.0 : src[n];
}

// weight sum of the wall average at solid node n (0: no fluid neighbour)
__device__ inline double mask_den(unsigned w) {
    double den = 0.0;
#pragma unroll
    for (int i = 0; i < 27; ++i)
        if (!(w & (1u << i))) den += wi(i);
    return den;
}

// dst(y) += sum over the solid neighbours s = y + c_i of fluid y of
// w_i / den(s) src(s)
__global__ __launch_bounds__(kBlock) void k_adj_wall_gather_m(KP kp, const unsigned *nbr, const double *src,
                                                            double *dst) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned w = nbr[n];
    if ((w & kSelfBit) || w == 0u) return;
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        if (!(w & (1u << i))) continue;
        const unsigned s = nb.at(cxi(i), cyi(i), czi(i));
        acc += wi(i) / mask_den(nbr[s]) * src[s];
    }
    dst[n] += acc;
}

// Solid nodes: rho_ave_bar = W'(rho_ave) rho_bar(x_s) and the per-node
// dL/d(wet_value) (active branch of Eq. (38)); 0 elsewhere.
__global__ __launch_bounds__(kBlock) void k_adj_wall_rho_solid_m(KP kp, const unsigned *nbr, const double *rho,
                                                               const double *rhobt, double *raveb, double *wetc) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned w = nbr[n];
    double rb = 0.0, wc = 0.0;
    if (w & kSelfBit) {
        int x, y, z;
        decompose(kp, n, x, y, z);
        const Nb nb(kp, x, y, z);
        double num = 0.0, den = 0.0;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            if (w & (1u << i)) continue;
            const double wt = wi(i);
            num += wt * rho[nb.at(cxi(i), cyi(i), czi(i))];
            den += wt;
        }
        if (den > 0.0) {
            rb = wall_rho_bar(kp, num / den, rhobt[n], wc);
        }
    }
    raveb[n] = rb;
    wetc[n] = wc;
}

// lambda_i(t) = direct part + rho_bar_total + c_i . j_bar at fluid nodes.
template <int P> __global__ __launch_bounds__(kBlock) void k_adj_final(KP kp, Bufs b, void *lam) {
    using real = real_t<P>;
    const unsigned idx = tile_id(kp) * kBlock + threadIdx.x;
    if (idx >= kp.nfluid) return;
    const unsigned n = (unsigned)kp.z0 * kp.plane + idx;
    if (kp.masked && (b.nbr[n] & kSelfBit)) return;
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const Pack4<real> *pk = (const Pack4<real> *)((const double *)b.abuf + A_PACK * (size_t)kp.N);
    const Lam<real> L(lam, kp);
#pragma unroll
    for (int i = 0; i < 27; ++i) L.st(i, row, x, L.ld(i, row, x) + final_term<real>(pk, i, n));
}

// Per-block sums of n values (a fixed grid-stride assignment: the same sums in
// the same order on every call).
__global__ __launch_bounds__(kBlock) void k_adj_reduce_part(unsigned n, const double *a, double *part) {
    double v = 0.0;
    for (unsigned i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) v += a[i];
    v = block_sum<kBlock>(v);
    if (threadIdx.x == 0) part[blockIdx.x] = v;
}

// The partial sums of a step, in a fixed order, onto acc[0..2] = kappa, wet
// value, nu (one workgroup).
constexpr int kFinal = 1024;
__global__ __launch_bounds__(kFinal) void k_adj_reduce_final(unsigned nk, const double *kap, const double *nu,
                                                             unsigned nw, const double *wet, double *acc) {
    double v[3] = {0, 0, 0};
    for (unsigned q = threadIdx.x; q < nk; q += kFinal) {
        v[0] += kap[q];
        v[2] += nu[q];
    }
    for (unsigned q = threadIdx.x; q < nw; q += kFinal) v[1] += wet[q];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[k] = block_sum<kFinal>(v[k]);
        if (threadIdx.x == 0) acc[k] += v[k];
    }
}

// ---- seed and initialiser ---------------------------------------------------
// lambda(T), zero gradient accumulators and zero sources at the solid nodes
__device__ inline void zero_grads(const Bufs &b) {
    if (blockIdx.x == 0 && threadIdx.x < 8) b.agrad[threadIdx.x] = 0.0;
}

template <int P> __global__ __launch_bounds__(kBlock) void k_adj_seed(KP kp, Bufs b, const double *g, void *lam) {
    using real = real_t<P>;
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    zero_grads(b);
    if (n >= kp.N) return;
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const bool fluid = fluid_node(kp, b, n);
    if (!fluid) zero_sources<real>(b.abuf, kp.N, n);
    const real v = fluid ? (real)g[n] : (real)0;
    const Lam<real> L(lam, kp);
#pragma unroll
    for (int i = 0; i < 27; ++i) L.st(i, row, x, v);
}

template <int P>
__global__ __launch_bounds__(kBlock) void k_adj_seed_pop(KP kp, Bufs b, const double *g, void *lam) {
    using real = real_t<P>;
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    zero_grads(b);
    if (n >= kp.N) return;
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const bool fluid = fluid_node(kp, b, n);
    if (!fluid) zero_sources<real>(b.abuf, kp.N, n);
    const Lam<real> L(lam, kp);
#pragma unroll
    for (int i = 0; i < 27; ++i) L.st(i, row, x, fluid ? (real)g[(size_t)i * kp.N + n] : (real)0);
}

template <int P>
__global__ __launch_bounds__(kBlock) void k_adj_get(KP kp, Bufs b, const void *lam, double *out) {
    using real = real_t<P>;
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const bool fluid = fluid_node(kp, b, n);
    const Lam<real> L(const_cast<void *>(lam), kp);
#pragma unroll
    for (int i = 0; i < 27; ++i) out[(size_t)i * kp.N + n] = fluid ? (double)L.ld(i, row, x) : 0.0;
}

// Initialiser f = T(u0)^{-1} k_eq(rho0, p_m): k_eq_bar = T(u0)^{-T} lambda(0);
// rho_bar_local = k_eq_bar_000, mu_bar = p_m_bar / 3 (fluid), 0 at solid.
// PEND: the last term of lambda(0) is added as it is read (k_adj_final would
// read and write the lattice for it: 224 us at 192x192x96 in FP32).
template <int P, bool PEND>
__global__ __launch_bounds__(kBlock) void k_adj_init_local(KP kp, Bufs b, const void *lam, const double *u0) {
    using real = real_t<P>;
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const bool fluid = fluid_node(kp, b, n);
    const size_t N = kp.N;
    double *A = (double *)b.abuf;
    if (!fluid) {
        A[A_RHOB * N + n] = 0.0;
        A[A_MUB * N + n] = 0.0;
        return;
    }
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const Lam<real> L(const_cast<void *>(lam), kp);
    real l[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) l[i] = L.ld(i, row, x);
    if constexpr (PEND) {
        const Pack4<real> *pk = (const Pack4<real> *)((const double *)b.abuf + A_PACK * N);
#pragma unroll
        for (int i = 0; i < 27; ++i) l[i] += final_term<real>(pk, i, n);
    }
    real ux = 0, uy = 0, uz = 0;
    if (u0) {
        ux = (real)u0[n];
        uy = (real)u0[N + n];
        uz = (real)u0[2 * N + n];
    }
    cm_inverse_T(l, ux, uy, uz);
    const double third = 1.0 / 3.0, ninth = 1.0 / 9.0;
    const double pmb = (double)l[K(2, 0, 0)] + (double)l[K(0, 2, 0)] + (double)l[K(0, 0, 2)] +
                       third * ((double)l[K(2, 2, 0)] + (double)l[K(2, 0, 2)] + (double)l[K(0, 2, 2)]) +
                       ninth * (double)l[K(2, 2, 2)];
    A[A_RHOB * N + n] = (double)l[K(0, 0, 0)];
    A[A_MUB * N + n] = pmb / 3.0;
}

__global__ __launch_bounds__(kBlock) void k_adj_init_out(KP kp, Bufs b, const double *rhobt, double *out) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    out[n] = fluid_node(kp, b, n) ? rhobt[n] : 0.0;
}

template <int P, bool MASK>
void adj_collide(hipStream_t s, const KP &kp, const Bufs &b, const void *ft, int lcur, bool pending) {
    auto go = [&](auto pend, auto nt) {
        k_adj_collide<P, decltype(pend)::value, MASK, decltype(nt)::value>
            <<<nblocks(kp.nfluid), kBlock, 0, s>>>(kp, b, ft, b.lam[lcur], b.lam[1 - lcur]);
    };
    const bool nt = kp.N >= (1u << 20);
    if (pending)
        nt ? go(std::true_type{}, std::true_type{}) : go(std::true_type{}, std::false_type{});
    else
        nt ? go(std::false_type{}, std::true_type{}) : go(std::false_type{}, std::false_type{});
}

// From 2^20 nodes the wide tile, one workgroup per CU: fewer ring nodes and
// halo lines (192x192x96 in FP32: 133 against 147 us); below, the narrow one,
// whose two workgroups per CU cover a small grid in more pieces (48x40x32 in
// FP64: 18 against 28 us).
template <int P, bool MASK> void phimu(hipStream_t s, const KP &kp, const Bufs &b) {
    auto go = [&](auto tx, auto ty, auto nt) {
        constexpr int TX = decltype(tx)::value, TY = decltype(ty)::value, NT = decltype(nt)::value;
        const unsigned tiles = (kp.nx + TX - 1) / TX * ((kp.ny + TY - 1) / TY);
        const int cz = march_chunk(tiles, kp.nz, 256 * (1024 / NT), 6);
        k_adj_phimu<P, MASK, TX, TY, NT><<<dim3(tiles, (kp.nz + cz - 1) / cz), NT, 0, s>>>(kp, b, cz);
    };
    using std::integral_constant;
    if (kp.N >= (1u << 20))
        go(integral_constant<int, 64>{}, integral_constant<int, 13>{}, integral_constant<int, 1024>{});
    else
        go(integral_constant<int, 32>{}, integral_constant<int, 12>{}, integral_constant<int, 512>{});
}

template <class Fn> hipError_t dispatch(int prec, Fn &&fn) {
    switch (prec) {
        case LBFE_FP64: return fn(std::integral_constant<int, LBFE_FP64>{});
        case LBFE_FP32: return fn(std::integral_constant<int, LBFE_FP32>{});
        case LBFE_FP16_DEV: return fn(std::integral_constant<int, LBFE_FP16_DEV>{});
        default: return fn(std::integral_constant<int, LBFE_FP16_DEV_F0FP32>{});
    }
}

constexpr unsigned kReduceBlocks = 1024;  // blocks of the gradient reduction

// The chain from mu_bar to rho_bar_total (A_RHOBT) with walls, the kappa, wet
// and nu sums and, in a step, the pack of the next one.  STEP: mu_bar from
// k_adj_phimu (A_MUBT); otherwise the initialiser's adjoint, its local part
// (A_MUB).
template <int P, bool STEP> hipError_t chain_tail(hipStream_t s, const KP &kp, const Bufs &b) {
    const size_t N = kp.N;
    double *A = (double *)b.abuf;
    const unsigned gN = nblocks(N), gf = nblocks(kp.nfluid), gw = nblocks(2 * (size_t)kp.plane);
    double *mub_tot = A + (STEP ? A_MUBT : A_MUB) * N;
    const unsigned tiles = (kp.nx + RTX - 1) / RTX * ((kp.ny + RTY - 1) / RTY);
    const int cz = march_chunk(tiles, kp.nz, 256 * 3, 3);
    const dim3 gall(tiles, (kp.nz + cz - 1) / cz);
    const double *wet = A + A_WETC * N, *nuc = STEP ? A + A_NUC * N : nullptr;
    // one slot each holds the partial sums: no more workgroups than nodes
    double *kap = A + A_KAPC * N, *nu = A + (kp.masked ? A_MUBT : A_RAVEB) * N;
    unsigned nwet = 0;
    if (kp.masked) {
        // mu_bar of the solid nodes back to their fluid neighbours (Eq. (36)),
        // then the Laplacian's adjoint with mu_bar zero at solid nodes
        k_adj_wall_gather_m<<<gN, kBlock, 0, s>>>(kp, b.nbr, mub_tot, mub_tot);
        k_adj_fluid_copy_m<<<gN, kBlock, 0, s>>>(kp, b.nbr, mub_tot, A + A_MUB * N);
        k_adj_rho<true><<<gall, RNT, 0, s>>>(kp, A + A_MUB * N, A + A_RHOB * N, b.rho, nuc, A + A_RHOBT * N, kap,
                                             nu, cz, b.nbr);
        k_adj_wall_rho_solid_m<<<gN, kBlock, 0, s>>>(kp, b.nbr, b.rho, A + A_RHOBT * N, A + A_RAVEB * N,
                                                     A + A_WETC * N);
        k_adj_wall_gather_m<<<gN, kBlock, 0, s>>>(kp, b.nbr, A + A_RAVEB * N, A + A_RHOBT * N);
        nwet = gN < kReduceBlocks ? gN : kReduceBlocks;
        k_adj_reduce_part<<<nwet, kBlock, 0, s>>>((unsigned)N, wet, b.agrad + 8);
        wet = b.agrad + 8;
    } else {
        if (kp.walls) k_adj_wall_gather<<<gw, kBlock, 0, s>>>(kp, mub_tot, mub_tot);
        k_adj_rho<false><<<gall, RNT, 0, s>>>(kp, mub_tot, A + A_RHOB * N, b.rho, nuc, A + A_RHOBT * N, kap, nu,
                                              cz, nullptr);
        if (kp.walls) nwet = gf;
    }
    if (kp.walls)
        k_adj_tail<P, STEP, true><<<gf, kBlock, 0, s>>>(kp, b);
    else if (STEP)
        k_adj_tail<P, STEP, false><<<gf, kBlock, 0, s>>>(kp, b);
    k_adj_reduce_final<<<1, kFinal, 0, s>>>(gall.x * gall.y, kap, nu, nwet, wet, b.agrad);
    return hipGetLastError();
}

}  // namespace

size_t adjoint_aux_bytes(int, size_t N) { return (size_t)A_COUNT * 8 * N; }
size_t adjoint_grad_slots() { return 3; }

hipError_t launch_adj_seed(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur, const double *g) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_adj_seed<P><<<nblocks(kp.N), kBlock, 0, s>>>(kp, b, g, b.lam[lcur]);
        return hipGetLastError();
    });
}

hipError_t launch_adj_seed_pop(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur, const double *g) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_adj_seed_pop<P><<<nblocks(kp.N), kBlock, 0, s>>>(kp, b, g, b.lam[lcur]);
        return hipGetLastError();
    });
}

hipError_t launch_adj_get(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur, double *out) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_adj_get<P><<<nblocks(kp.N), kBlock, 0, s>>>(kp, b, b.lam[lcur], out);
        return hipGetLastError();
    });
}

hipError_t launch_adj_step(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur, const void *ft,
                           bool recompute, bool pending) {
    if (recompute) {
        Bufs fb = b;
        fb.f[0] = const_cast<void *>(ft);
        hipError_t e = launch_aux(s, prec, kp, fb, 0, true);
        if (e != hipSuccess) return e;
    }
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        if (kp.masked) {
            adj_collide<P, true>(s, kp, b, ft, lcur, pending);
            phimu<P, true>(s, kp, b);
        } else {
            adj_collide<P, false>(s, kp, b, ft, lcur, pending);
            if (kp.moving) {
                const unsigned gw = nblocks(2 * (size_t)kp.plane);
                if (pending)
                    k_adj_wall_move<P, true><<<gw, kBlock, 0, s>>>(kp, b, b.lam[lcur]);
                else
                    k_adj_wall_move<P, false><<<gw, kBlock, 0, s>>>(kp, b, b.lam[lcur]);
            }
            phimu<P, false>(s, kp, b);
        }
        return chain_tail<P, true>(s, kp, b);  // lambda(t) = direct part; its last term is pending
    });
}

hipError_t launch_adj_finalize(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        k_adj_final<P><<<nblocks(kp.nfluid), kBlock, 0, s>>>(kp, b, b.lam[lcur]);
        return hipGetLastError();
    });
}

hipError_t launch_adj_init(hipStream_t s, int prec, const KP &kp, const Bufs &b, int lcur, bool pending,
                           const double *rho0, const double *u0, double *out) {
    // forward initialiser quantities: rho (with wall densities) and mu
    const unsigned gN = nblocks(kp.N);
    hipError_t e = launch_init_aux(s, kp, b, rho0);
    if (e != hipSuccess) return e;
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        if (pending)
            k_adj_init_local<P, true><<<gN, kBlock, 0, s>>>(kp, b, b.lam[lcur], u0);
        else
            k_adj_init_local<P, false><<<gN, kBlock, 0, s>>>(kp, b, b.lam[lcur], u0);
        hipError_t r = chain_tail<P, false>(s, kp, b);
        if (r != hipSuccess) return r;
        k_adj_init_out<<<gN, kBlock, 0, s>>>(kp, b, (const double *)b.abuf + A_RHOBT * (size_t)kp.N, out);
        return hipGetLastError();
    });
}

}  // namespace lbfe

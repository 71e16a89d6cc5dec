// Arbitrary solid voxel masks (curved or patterned substrates) on gfx950:
// the halfway bounce-back of Eq. (10) and the wetting boundary of
// Eqs. (36)-(38) at every solid node x_s of a mask, which the paper writes
// for a general x_s (Sec. III C).  The flat walls of the z-plane path are the
// special case of a mask holding the two planes.
//
// Every node carries one 32-bit neighbour word: bit i (i = 0..26) is set
// when x + c_i is solid, so bit 13 tells whether the node itself is solid.
// It is built once per mask; all kernels below work per node over the whole
// grid and read it (the _m kernels gather their neighbours through L1/L2,
// the _z stencils stage their input field in the z-marching LDS ring of
// lbfe_zring.h):
//   k_moments_m     rho, j of the fluid nodes (order of moments())
//   k_wall_rho_m    rho at solid nodes with a fluid neighbour, Eqs. (37)-(38)
//   k_mu_z / k_mu_f mu = mu0(rho) - kappa lap_h rho at fluid nodes, Eq. (32)
//                   (narrow forms / FP64; k_mu_m for the initialiser)
//   k_wall_mu_m     mu at solid nodes, Eq. (36)
//   k_fphi_z        G = grad_h mu, F = (1/3 - rho) G, u = (j + F/2)/rho,
//                   phi = (p_m - rho/3) u at fluid nodes, Eqs. (11)-(12), (27)
//   k_q_m           Q_aa = -3 d_a phi_a at fluid nodes, Eq. (27)
//                   (k_fq_f: both at once, in FP64)
//   k_collide_m     collision and push-streaming; a link that ends on a
//                   solid node returns into slot opp(i) of its own node
// Solid nodes hold no populations (their slots stay zero) and zero j, F,
// phi, Q; a solid node with no fluid neighbour gets rho = mu = 0 and is read
// by no fluid stencil.
#include <type_traits>

#include "lbfe_device.h"
#include "lbfe_factored.h"

namespace lbfe {
namespace {

template <int P> using real_t = typename Pol<P>::real;

constexpr unsigned kSelf = 1u << kRest;

__device__ inline bool solid_at(unsigned w) { return (w & kSelf) != 0; }

__global__ __launch_bounds__(kBlock) void k_mask_prep(KP kp, const uint8_t *solid, unsigned *nbr) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    unsigned w = 0;
#pragma unroll
    for (int i = 0; i < 27; ++i)
        if (solid[nb.at(cxi(i), cyi(i), czi(i))]) w |= 1u << i;
    nbr[n] = w;
}

template <int P, bool NT>
__global__ __launch_bounds__(kBlock) void k_moments_m(KP kp, const unsigned *nbr, const void *fq, double *rho,
                                                      void *jq, int *flag) {
    using real = real_t<P>;
    // (against the order of k_collide_m, as in k_moments)
    const unsigned n = tile_id(kp, true) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    // the population loads do not wait for the neighbour word (a solid
    // node's slots hold zeros); only the stores depend on it
    const unsigned w = nbr[n];
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    const Pops<P, NT> f(fq, kp);
    real v[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) v[i] = f.ld(i, row, x);
    double r;
    real jx, jy, jz;
    moments(v, r, jx, jy, jz);
    if (solid_at(w)) return;
    rho[n] = r;
    real *j = (real *)jq;
    j[n] = jx;
    j[kp.N + n] = jy;
    j[2 * (size_t)kp.N + n] = jz;
    if (!(r > 0.0 && kp.b * r < 1.0)) *flag = 1;
}

// Weighted average over the fluid neighbours of a solid node (Eqs. (36),
// (37)), in direction order; 0 when there is none.
__device__ inline double fluid_average(const KP &kp, unsigned w, const double *g, unsigned n) {
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    double num = 0.0, den = 0.0;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        if (w & (1u << i)) continue;
        const double wt = wi(i);
        num += wt * g[nb.at(cxi(i), cyi(i), czi(i))];
        den += wt;
    }
    return den > 0.0 ? num / den : 0.0;
}

__global__ __launch_bounds__(kBlock) void k_wall_rho_m(KP kp, const unsigned *nbr, double *rho) {
    const unsigned n = tile_id(kp) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned w = nbr[n];
    if (!solid_at(w)) return;
    rho[n] = window_rho(kp, fluid_average(kp, w, rho, n));
}

// mu = mu0(rho) - kappa lap_h rho, lap_h g = 6 sum_i w_i (g(x+c_i) - g(x))
__global__ __launch_bounds__(kBlock) void k_mu_m(KP kp, const unsigned *nbr, const double *rho, double *mu) {
    const unsigned n = tile_id(kp) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const bool solid = solid_at(nbr[n]);
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    const double r0 = rho[n];
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        if (i == kRest) continue;
        s += wi(i) * (rho[nb.at(cxi(i), cyi(i), czi(i))] - r0);
    }
    if (solid) return;
    mu[n] = mu_bulk(kp, r0) - kp.kappa * 6.0 * s;
}

__global__ __launch_bounds__(kBlock) void k_wall_mu_m(KP kp, const unsigned *nbr, double *mu) {
    const unsigned n = tile_id(kp) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned w = nbr[n];
    if (!solid_at(w)) return;
    mu[n] = fluid_average(kp, w, mu, n);
}

// Q_aa = -3 d_a,h phi_a = -9 sum_i w_i c_ia phi_a(x + c_i)
template <int P>
__global__ __launch_bounds__(kBlock) void k_q_m(KP kp, const unsigned *nbr, const void *phiq, void *Qq) {
    using real = real_t<P>;
    const unsigned n = tile_id(kp) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const size_t N = kp.N;
    real *Q = (real *)Qq;
    const bool solid = solid_at(nbr[n]);
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    const real *phi = (const real *)phiq;
    real sx = 0, sy = 0, sz = 0;
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        if (i == kRest) continue;
        const unsigned m = nb.at(cxi(i), cyi(i), czi(i));
        const real wt = (real)wi(i);
        if (cxi(i)) sx += (real)cxi(i) * wt * phi[m];
        if (cyi(i)) sy += (real)cyi(i) * wt * phi[N + m];
        if (czi(i)) sz += (real)czi(i) * wt * phi[2 * N + m];
    }
    const real h = (real)(-9.0);
    Q[n] = solid ? (real)0 : h * sx;
    Q[N + n] = solid ? (real)0 : h * sy;
    Q[2 * N + n] = solid ? (real)0 : h * sz;
}

template <int P, bool NT>
__global__ __launch_bounds__(kBlock) void k_collide_m(KP kp, const unsigned *nbr, const void *fin_q, void *fout_q,
                                                      const double *mu, const void *Fq, const void *Qq) {
    using real = real_t<P>;
    const unsigned n = tile_id(kp) * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const unsigned w = nbr[n];
    int x, y, z;
    decompose(kp, n, x, y, z);
    const Nb nb(kp, x, y, z);
    const Pops<P, NT> fin(fin_q, kp);
    const Pops<P> fout(fout_q, kp);
    const unsigned row = nb.row(0, 0);
    real f[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) f[i] = fin.ld(i, row, (unsigned)x);
    if (solid_at(w)) return;
    const real *F = (const real *)Fq, *Qa = (const real *)Qq;
    constexpr bool nt = NT && (P == LBFE_FP64 || P == LBFE_FP32);  // the aux fields are read once, as in k_collide
    auto ld = [&](const auto *p) { return nt ? ldnt(p) : *p; };
    collide_node(kp, f, ld(mu + n), ld(F + n), ld(F + kp.N + n), ld(F + 2 * (size_t)kp.N + n), ld(Qa + n),
                 ld(Qa + kp.N + n), ld(Qa + 2 * (size_t)kp.N + n));
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        if (w & (1u << i))
            fout.st(26 - i, row, (unsigned)x, f[i]);
        else
            fout.st(i, nb.row(cyi(i), czi(i)), nb.xo(cxi(i)), f[i]);
    }
}

// Initial populations of the fluid nodes (Eq. (20) equilibrium at rho0, u0,
// p_m(mu)); solid nodes get zeros.
template <int P>
__global__ __launch_bounds__(kBlock) void k_init_m(KP kp, const unsigned *nbr, const double *rho0, const double *u0,
                                                   const double *mu, void *fq) {
    using real = real_t<P>;
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    const Pops<P> f(fq, kp);
    const unsigned row = n / (unsigned)kp.nx, x = n - row * (unsigned)kp.nx;
    real k[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) k[i] = 0;
    if (!solid_at(nbr[n])) {
        const real pm = (real)((1.0 + mu[n]) / 3.0);
        k[K(0, 0, 0)] = (real)rho0[n];
        k[K(2, 0, 0)] = k[K(0, 2, 0)] = k[K(0, 0, 2)] = pm;
        k[K(2, 2, 0)] = k[K(2, 0, 2)] = k[K(0, 2, 2)] = pm * (real)(1.0 / 3.0);
        k[K(2, 2, 2)] = pm * (real)(1.0 / 9.0);
        real ux = 0, uy = 0, uz = 0;
        if (u0) {
            ux = (real)u0[n];
            uy = (real)u0[kp.N + n];
            uz = (real)u0[2 * (size_t)kp.N + n];
        }
        cm_inverse(k, ux, uy, uz);
#pragma unroll
        for (int i = 0; i < 27; ++i) f.st(i, row, x, k[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 27; ++i) f.st(i, row, x, (real)0);
    }
}

__global__ __launch_bounds__(kBlock) void k_copy_fluid_m(KP kp, const unsigned *nbr, const double *src, double *dst) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N) return;
    dst[n] = solid_at(nbr[n]) ? 0.0 : src[n];
}

__global__ __launch_bounds__(kBlock) void k_check_rho_m(KP kp, const unsigned *nbr, const double *rho, int *flag) {
    const unsigned n = blockIdx.x * kBlock + threadIdx.x;
    if (n >= kp.N || solid_at(nbr[n])) return;
    const double r = rho[n];
    if (!(r > 0.0 && kp.b * r < 1.0)) *flag = 1;
}

// The step's mu (the sums of k_mu_m, in the same order) and its force,
// velocity and phi, with the stencil field (rho, mu) staged in an LDS ring:
// grad_h mu = 3 sum_i w_i c_i mu(x + c_i), F = (1/3 - rho) grad_h mu,
// u = (j + F/2)/rho, phi = (p_m - rho/3) u; F = phi = 0 at solid nodes.
__global__ __launch_bounds__(ZCB) void k_mu_z(KP kp, const unsigned *nbr, const double *rho, double *mu, int cz) {
    __shared__ double lds[4][ZNR];
    int x0, y0, zs, ze;
    ztile(kp, cz, x0, y0, zs, ze);
    ZRing R;
    R.init(kp, lds, rho, x0, y0);
    R.march(zs, ze, [&](int k) {
        if (!R.own) return;
        const size_t n = (size_t)k * kp.plane + R.node;
        if (solid_at(nbr[n])) return;
        const double r0 = R.at(k, 0, 0);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            if (i == kRest) continue;
            s += wi(i) * (R.at(k + czi(i), cxi(i), cyi(i)) - r0);
        }
        mu[n] = mu_bulk(kp, r0) - kp.kappa * 6.0 * s;
    });
}

template <int P>
__global__ __launch_bounds__(ZCB) void k_fphi_z(KP kp, const unsigned *nbr, const double *rho, const void *jq,
                                                const double *mu, void *Fq, void *phiq, int cz) {
    using real = real_t<P>;
    __shared__ double lds[4][ZNR];
    int x0, y0, zs, ze;
    ztile(kp, cz, x0, y0, zs, ze);
    const size_t N = kp.N;
    real *F = (real *)Fq, *phi = (real *)phiq;
    const real *j = (const real *)jq;
    ZRing R;
    R.init(kp, lds, mu, x0, y0);
    R.march(zs, ze, [&](int k) {
        if (!R.own) return;
        const size_t n = (size_t)k * kp.plane + R.node;
        if (solid_at(nbr[n])) {
            for (int a = 0; a < 3; ++a) F[a * N + n] = phi[a * N + n] = (real)0;
            return;
        }
        double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            if (i == kRest) continue;
            const double v = 3.0 * wi(i) * R.at(k + czi(i), cxi(i), cyi(i));
            if (cxi(i)) gx += cxi(i) * v;
            if (cyi(i)) gy += cyi(i) * v;
            if (czi(i)) gz += czi(i) * v;
        }
        const double rd = rho[n];
        const double c1 = 1.0 / 3.0 - rd;
        const real Fx = (real)(c1 * gx), Fy = (real)(c1 * gy), Fz = (real)(c1 * gz);
        const real ir = (real)1 / (real)rd;
        const real ux = (j[n] + (real)0.5 * Fx) * ir;
        const real uy = (j[N + n] + (real)0.5 * Fy) * ir;
        const real uz = (j[2 * N + n] + (real)0.5 * Fz) * ir;
        const real c2 = (real)((1.0 + R.at(k, 0, 0) - rd) * (1.0 / 3.0));  // p_m - rho/3
        F[n] = Fx;
        F[N + n] = Fy;
        F[2 * N + n] = Fz;
        phi[n] = c2 * ux;
        phi[N + n] = c2 * uy;
        phi[2 * N + n] = c2 * uz;
    });
}

// ---- the FP64 stencils -------------------------------------------------------
// In FP64 the three stencils are factored (lbfe_factored.h; the narrow forms
// still have the point-by-point sums above): mu in one march, then F, phi and Q in another that keeps phi in
// LDS.  At 192x192x96 the two take 29 and 66 us (20 and 120 B per node without
// the halos), where the three point-by-point passes took 39, 66 and 79 us.

// mu = mu0(rho) - kappa 6 (Wz Wx Wy rho - rho) at fluid nodes.  Iteration t
// stages rho(t), takes the in-plane part of plane t-1 and the node of plane
// t-2; loads run one iteration ahead.
constexpr int UTX = 32, UTY = 16, UNT = UTX * UTY;
__global__ __launch_bounds__(UNT) void k_mu_f(KP kp, const unsigned *nbr, const double *rho, double *mu, int cz) {
    constexpr int W = UTX + 2, NR = W * (UTY + 2), PT = (NR + UNT - 1) / UNT;
    __shared__ double sd[2][NR];  // rho of plane p (slot p & 1)
    int tile, chunk;
    xcd_tile(tile, chunk);
    const int ntx = (kp.nx + UTX - 1) / UTX, x0 = tile % ntx * UTX, y0 = tile / ntx * UTY;
    const int zs = chunk * cz, ze = min(zs + cz, kp.nz);
    const unsigned plane = kp.plane;
    const int tid = threadIdx.x, ta = tid % UTX, tb = tid / UTX;
    const bool own = x0 + ta < kp.nx && y0 + tb < kp.ny;
    const unsigned ooff = own ? (unsigned)(y0 + tb) * kp.nx + (x0 + ta) : kNone;
    const int c = (tb + 1) * W + ta + 1;
    unsigned off[PT];
#pragma unroll
    for (int m = 0; m < PT; ++m) {
        const int r = tid + m * UNT;
        off[m] = r < NR ? (unsigned)zwrap(y0 + r / W - 1, kp.ny) * kp.nx + zwrap(x0 + r % W - 1, kp.nx) : kNone;
    }
    auto next = [&](int g) { return g + 1 == kp.nz ? 0 : g + 1; };
    double pre[PT];
    unsigned wpre = kSelf;
    auto load = [&](int g, bool ok) {  // ok false: a plane the chunk does not need
#pragma unroll
        for (int m = 0; m < PT; ++m) pld(pre[m], plane_of(rho, (size_t)g * plane, plane, 8), ok ? off[m] : kNone);
    };
    double a = 0, b = 0, r0 = 0;  // Wx Wy rho two planes back, one back; rho one back
    int t = zs - 1;
    int g2 = zwrap(t - 2, kp.nz), g1 = zwrap(t - 1, kp.nz), gn = zwrap(t, kp.nz);
    load(gn, true);
    for (; t <= ze + 1; ++t) {
#pragma unroll
        for (int m = 0; m < PT; ++m)
            if (tid + m * UNT < NR) sd[t & 1][tid + m * UNT] = pre[m];
        gn = next(gn);
        load(gn, t + 1 <= ze);
        const unsigned w = wpre;
        wpre = own && t - 1 >= zs && t - 1 < ze ? nbr[(size_t)g1 * plane + ooff] : kSelf;
        if (t - 1 >= zs - 1) {
            const double n = smooth2<W>(sd[(t - 1) & 1], c);
            if (!solid_at(w)) mu[(size_t)g2 * plane + ooff] = mu_bulk(kp, r0) - kp.kappa * 6.0 * (wz(a, b, n) - r0);
            a = b, b = n;
            r0 = sd[(t - 1) & 1][c];
        }
        __syncthreads();
        g2 = g1;
        g1 = next(g1);
    }
}

// G = grad_h mu, F = (1/3 - rho) G, u = (j + F/2)/rho, phi = (p_m - rho/3) u,
// Q_aa = -3 d_a phi_a.  The phi part runs on the tile and its one-node ring,
// one node per thread: iteration t stages mu(t) (two-node halo), takes the
// in-plane parts of plane t-1 and phi of plane t-2, then the in-plane parts of
// phi(t-3) and Q(t-4).  F = phi = Q = 0 at solid nodes.
template <int PTX, int PTY, int PNT>
__global__ __launch_bounds__(PNT, 4) void k_fq_f(KP kp, const unsigned *nbr, const double *rho, const double *j,
                                                 const double *mu, double *F, double *Q, int cz) {
    constexpr int PWX = PTX + 4, PNR = PWX * (PTY + 4);  // mu region
    constexpr int GWX = PTX + 2, GNR = GWX * (PTY + 2);  // phi region
    constexpr int PPT = (PNR + PNT - 1) / PNT;
    static_assert(GNR <= PNT && PTX * PTY <= PNT, "one phi node, one owned column per thread");
    __shared__ double sm[2][PNR];     // mu of plane p (slot p & 1)
    __shared__ double sp[2][3][GNR];  // phi of plane p (slot p & 1)
    int tile, chunk;
    xcd_tile(tile, chunk);
    const int ntx = (kp.nx + PTX - 1) / PTX, x0 = tile % ntx * PTX, y0 = tile / ntx * PTY;
    const int zs = chunk * cz, ze = min(zs + cz, kp.nz);
    const size_t N = kp.N;
    const unsigned plane = kp.plane;
    const int tid = threadIdx.x;
    unsigned moff[PPT];
#pragma unroll
    for (int m = 0; m < PPT; ++m) {
        const int r = tid + m * PNT;
        moff[m] = r < PNR ? (unsigned)zwrap(y0 + r / PWX - 2, kp.ny) * kp.nx + zwrap(x0 + r % PWX - 2, kp.nx) : kNone;
    }
    const int ga = tid % GWX, gb = tid / GWX;
    const bool hasg = tid < GNR;
    const unsigned noff = hasg ? (unsigned)zwrap(y0 + gb - 1, kp.ny) * kp.nx + zwrap(x0 + ga - 1, kp.nx) : kNone;
    const bool owng = hasg && ga >= 1 && ga <= PTX && gb >= 1 && gb <= PTY && x0 + ga - 1 < kp.nx && y0 + gb - 1 < kp.ny;
    const int cm = hasg ? (gb + 1) * PWX + ga + 1 : PWX + 1;
    const int ta = tid % PTX, tb = tid / PTX;
    const bool own = tid < PTX * PTY && x0 + ta < kp.nx && y0 + tb < kp.ny;
    const unsigned ooff = own ? (unsigned)(y0 + tb) * kp.nx + (x0 + ta) : kNone;
    const int cg = tid < PTX * PTY ? (tb + 1) * GWX + ta + 1 : GWX + 1;
    auto next = [&](int g) { return g + 1 == kp.nz ? 0 : g + 1; };
    // loads run one iteration ahead of their use
    double mpre[PPT], rpre, jpre[3];
    unsigned wpre = kSelf, qpre = kSelf;  // neighbour words of the phi node and of the owned column's Q node
    auto load_mu = [&](int g, bool ok) {  // ok false: a plane the chunk does not need
#pragma unroll
        for (int m = 0; m < PPT; ++m) pld(mpre[m], plane_of(mu, (size_t)g * plane, plane, 8), ok ? moff[m] : kNone);
    };
    auto load_node = [&](int g, bool ok) {
        const size_t f = (size_t)g * plane;
        const unsigned o = ok ? noff : kNone;
        pld(rpre, plane_of(rho, f, plane, 8), o);
#pragma unroll
        for (int c = 0; c < 3; ++c) pld(jpre[c], plane_of(j + c * N, f, plane, 8), o);
        wpre = ok && hasg ? nbr[f + noff] : kSelf;
    };
    Ring3 rm, rp;  // in-plane parts of grad mu, of the Q stencils
    double mc = 0.0;
    int t = zs - 2;
    int g4 = zwrap(t - 4, kp.nz), g3 = zwrap(t - 3, kp.nz), g2 = zwrap(t - 2, kp.nz), g1 = zwrap(t - 1, kp.nz),
        gn = zwrap(t, kp.nz);
    load_mu(gn, true);
    load_node(g2, false);
    for (; t <= ze + 3; ++t) {
#pragma unroll
        for (int m = 0; m < PPT; ++m)
            if (tid + m * PNT < PNR) sm[t & 1][tid + m * PNT] = mpre[m];
        gn = next(gn);
        load_mu(gn, t + 1 <= ze + 1);
        if (t - 1 >= zs - 2 && t - 2 <= ze) {
            const int p = t - 2;
            const double *q = sm[(t - 1) & 1];
            const Part3 n{dx_wy<PWX>(q, cm), wx_dy<PWX>(q, cm), smooth2<PWX>(q, cm)};
            double f[3] = {0, 0, 0}, ph[3] = {0, 0, 0};
            if (p >= zs - 1 && !solid_at(wpre)) {
                const double g[3] = {0.5 * wz(rm.a.x, rm.b.x, n.x), 0.5 * wz(rm.a.y, rm.b.y, n.y), 0.5 * (n.z - rm.a.z)};
                const double c1 = 1.0 / 3.0 - rpre, ir = 1.0 / rpre, c2 = (1.0 + mc - rpre) * (1.0 / 3.0);  // p_m - rho/3
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    f[c] = c1 * g[c];
                    ph[c] = c2 * ((jpre[c] + 0.5 * f[c]) * ir);
                }
            }
            if (hasg && p >= zs - 1) {
#pragma unroll
                for (int c = 0; c < 3; ++c) sp[p & 1][c][tid] = ph[c];
            }
            load_node(g1, t - 1 >= zs - 1 && t - 1 <= ze);
            // the fill planes at both ends belong to the neighbouring chunks
            const unsigned o = owng && p >= zs && p < ze ? noff : kNone;
#pragma unroll
            for (int c = 0; c < 3; ++c) pst_nt(f[c], plane_of(F + c * N, (size_t)g2 * plane, plane, 8), o);
            rm.push(n);
            mc = q[cm];
        }
        const unsigned w = qpre;
        qpre = own && t - 3 >= zs && t - 3 < ze ? nbr[(size_t)g3 * plane + ooff] : kSelf;
        if (t - 3 >= zs - 1) {
            const double(*g)[GNR] = sp[(t - 3) & 1];
            const Part3 n{dx_wy<GWX>(g[0], cg), wx_dy<GWX>(g[1], cg), smooth2<GWX>(g[2], cg)};
            const bool fl = !solid_at(w);
            const unsigned o = t - 4 >= zs ? ooff : kNone;
            const size_t f = (size_t)g4 * plane;
            pst_nt(fl ? -1.5 * wz(rp.a.x, rp.b.x, n.x) : 0.0, plane_of(Q, f, plane, 8), o);
            pst_nt(fl ? -1.5 * wz(rp.a.y, rp.b.y, n.y) : 0.0, plane_of(Q + N, f, plane, 8), o);
            pst_nt(fl ? -1.5 * (n.z - rp.a.z) : 0.0, plane_of(Q + 2 * N, f, plane, 8), o);
            rp.push(n);
        }
        __syncthreads();
        g4 = g3;
        g3 = g2;
        g2 = g1;
        g1 = next(g1);
    }
}

// the wide tile from 2^20 nodes, as for the adjoint's march (k_adj_phimu)
void fq_f(hipStream_t s, const KP &kp, const Bufs &b) {
    auto go = [&](auto tx, auto ty, auto nt) {
        constexpr int TX = decltype(tx)::value, TY = decltype(ty)::value, NT = decltype(nt)::value;
        const unsigned tiles = (kp.nx + TX - 1) / TX * ((kp.ny + TY - 1) / TY);
        const int cz = march_chunk(tiles, kp.nz, 256 * (1024 / NT), 6);
        k_fq_f<TX, TY, NT><<<dim3(tiles, (kp.nz + cz - 1) / cz), NT, 0, s>>>(
            kp, b.nbr, b.rho, (const double *)b.j, b.mu, (double *)b.F, (double *)b.Q, cz);
    };
    using std::integral_constant;
    if (kp.N >= (1u << 20))
        go(integral_constant<int, 64>{}, integral_constant<int, 13>{}, integral_constant<int, 1024>{});
    else
        go(integral_constant<int, 32>{}, integral_constant<int, 12>{}, integral_constant<int, 512>{});
}

template <int P> void chain_m(hipStream_t s, const KP &kp, const Bufs &b) {
    const unsigned g = nblocks(kp.N);
    if constexpr (P == LBFE_FP64) {
        const unsigned tiles = (kp.nx + UTX - 1) / UTX * ((kp.ny + UTY - 1) / UTY);
        const int cz = march_chunk(tiles, kp.nz, 256 * 3, 3);
        k_mu_f<<<dim3(tiles, (kp.nz + cz - 1) / cz), UNT, 0, s>>>(kp, b.nbr, b.rho, b.mu, cz);
        k_wall_mu_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.mu);
        fq_f(s, kp, b);
    } else {
        const dim3 gz = zgrid(kp);
        k_mu_z<<<gz, ZCB, 0, s>>>(kp, b.nbr, b.rho, b.mu, kZChunk);
        k_wall_mu_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.mu);
        k_fphi_z<P><<<gz, ZCB, 0, s>>>(kp, b.nbr, b.rho, b.j, b.mu, b.F, b.phi, kZChunk);
        k_q_m<P><<<g, kBlock, 0, s>>>(kp, b.nbr, b.phi, b.Q);
    }
}

template <class Fn> hipError_t dispatch(int prec, Fn &&fn) {
    switch (prec) {
        case LBFE_FP64: return fn(std::integral_constant<int, LBFE_FP64>{});
        case LBFE_FP32: return fn(std::integral_constant<int, LBFE_FP32>{});
        case LBFE_FP16_DEV: return fn(std::integral_constant<int, LBFE_FP16_DEV>{});
        default: return fn(std::integral_constant<int, LBFE_FP16_DEV_F0FP32>{});
    }
}

}  // namespace

hipError_t launch_mask_prep(hipStream_t s, const KP &kp, const Bufs &b, const uint8_t *solid) {
    k_mask_prep<<<nblocks(kp.N), kBlock, 0, s>>>(kp, solid, b.nbr);
    return hipGetLastError();
}

template <int P> static void moments_m(hipStream_t s, const KP &kp, const Bufs &b, int cur) {
    if (kp.keep1)
        k_moments_m<P, false><<<nblocks(kp.N), kBlock, 0, s>>>(kp, b.nbr, b.f[cur], b.rho, b.j, b.flag);
    else
        k_moments_m<P, true><<<nblocks(kp.N), kBlock, 0, s>>>(kp, b.nbr, b.f[cur], b.rho, b.j, b.flag);
}

hipError_t launch_aux_mask(hipStream_t s, int prec, const KP &kp, const Bufs &b, int cur) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        const unsigned g = nblocks(kp.N);
        moments_m<P>(s, kp, b, cur);
        k_wall_rho_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho);
        chain_m<P>(s, kp, b);
        return hipGetLastError();
    });
}

hipError_t launch_step_mask(hipStream_t s, int prec, const KP &kp, const Bufs &b, int cur, hipEvent_t *ev) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        const unsigned g = nblocks(kp.N);
        auto mark = [&](int k) {
            if (ev) (void)hipEventRecord(ev[k], s);
        };
        mark(0);
        moments_m<P>(s, kp, b, cur);
        k_wall_rho_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho);
        mark(1);
        chain_m<P>(s, kp, b);
        mark(2);
        if (kp.keep2)
            k_collide_m<P, false><<<g, kBlock, 0, s>>>(kp, b.nbr, b.f[cur], b.f[1 - cur], b.mu, b.F, b.Q);
        else
            k_collide_m<P, true><<<g, kBlock, 0, s>>>(kp, b.nbr, b.f[cur], b.f[1 - cur], b.mu, b.F, b.Q);
        mark(3);
        mark(4);
        return hipGetLastError();
    });
}

hipError_t launch_init_mask(hipStream_t s, int prec, const KP &kp, const Bufs &b, int cur, const double *rho0,
                            const double *u0) {
    return dispatch(prec, [&](auto pc) {
        constexpr int P = decltype(pc)::value;
        const unsigned g = nblocks(kp.N);
        k_copy_fluid_m<<<g, kBlock, 0, s>>>(kp, b.nbr, rho0, b.rho);
        k_wall_rho_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho);
        k_mu_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho, b.mu);
        k_init_m<P><<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho, u0, b.mu, b.f[cur]);
        return hipGetLastError();
    });
}

hipError_t launch_init_aux_mask(hipStream_t s, const KP &kp, const Bufs &b, const double *rho0) {
    const unsigned g = nblocks(kp.N);
    k_copy_fluid_m<<<g, kBlock, 0, s>>>(kp, b.nbr, rho0, b.rho);
    k_wall_rho_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho);
    k_mu_m<<<g, kBlock, 0, s>>>(kp, b.nbr, b.rho, b.mu);
    return hipGetLastError();
}

hipError_t launch_check_rho0_mask(hipStream_t s, const KP &kp, const Bufs &b, const double *rho0, int *flag) {
    k_check_rho_m<<<nblocks(kp.N), kBlock, 0, s>>>(kp, b.nbr, rho0, flag);
    return hipGetLastError();
}

}  // namespace lbfe
